"""The exchange of partial sums inside a table phase's launch: a block that has
waited long enough for another one's rows computes them itself, and a block that
starts late finds the rows it needs already there.

The library's build for this test (libedkm_exchange.so, EDKM_XW_WAIT = -1,
EDKM_XW_LATE = 3 ms) makes both happen in every launch: every second block
starts late, and no block waits.  Its results have to equal the product
build's bit for bit (blocks may mix rows of either origin, and decide the early
stop from them), whatever the launch shape."""
import os
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2309_00964_amd import build, edkm, inputs               # noqa: E402
import exchange_child                                              # noqa: E402

pytestmark = pytest.mark.gpu


def child(lib, out):
    env = dict(os.environ, EDKM_LIBRARY=lib, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, os.path.join(ROOT, "tests", "exchange_child.py"), str(out)], cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, (r.stdout[-1000:], r.stderr[-3000:])
    with np.load(out) as z:
        return {k: z[k] for k in z.files}


def same_bits(a, b):
    return a.dtype == b.dtype and a.shape == b.shape and np.array_equal(a.view(np.uint32), b.view(np.uint32))


def test_rows_computed_by_waiting_blocks_have_the_same_bits(tmp_path):
    if not os.path.exists(build.OUT_EXCHANGE):
        pytest.skip("the exchange build is not built")
    print("[gpu-case] exchange: product build, then the build whose blocks do not wait", flush=True)
    want = child(build.OUT, tmp_path / "product.npz")
    got = child(build.OUT_EXCHANGE, tmp_path / "exchange.npz")
    assert sorted(want) == sorted(got)
    # (the child's last forward updates the centroids in place: a block that
    # starts late still has to read C^(0))
    assert len({int(v[0]) for k, v in want.items() if k.startswith("11.it")}) > 1    # early stops differ
    bad = [k for k in want if not same_bits(want[k], got[k])]
    assert not bad, bad


@pytest.mark.parametrize("case", [c for c in exchange_child.CASES if c[1] > 1])
def test_a_batch_has_the_bits_of_single_calls(case):
    """Forward and backward: the launch shape decides only which block computes a
    row (sizes of one workgroup per N-sized pass, as exchange_child says)."""
    bits, count, iters, eps, fmt = case
    print("[gpu-case] exchange: batch against single calls", case, flush=True)
    sizes, keys, c0, g = exchange_child.case_inputs(bits, count, fmt)
    res = []
    for batches in ([range(count)], [[i] for i in range(count)]):
        o = exchange_child.outputs(sizes, 1 << bits)
        for ids in batches:
            take = lambda x: [x[i] for i in ids]
            plans = [edkm.Plan(sizes[i], bits, iters, key_format=fmt) for i in ids]
            edkm.init_unique_batch(plans, take(keys))
            edkm.forward_batch(plans, take(keys), inputs.TAU, eps, take(c0), take(o["c"]), take(o["wt"]), False,
                               take(o["it"]))
            edkm.backward_batch(plans, take(keys), take(g), take(o["gw"]), take(o["gc"]))
            torch.cuda.synchronize()
        res.append(o)
    for name in res[0]:
        for i in range(count):
            assert same_bits(res[0][name][i].cpu().numpy(), res[1][name][i].cpu().numpy()), (name, i)


@pytest.mark.parametrize("dense", [False, True])
def test_centroids_updated_in_place(dense):
    """c_out may be c_in: the same bits as with a buffer of its own."""
    print("[gpu-case] exchange: centroids in place", dense, flush=True)
    (n,), (keys,), (c0,), (g,) = exchange_child.case_inputs(3, 1, "fp16")
    res = []
    for in_place in (False, True):
        o = exchange_child.outputs([n], 8)
        c_in, c_out = c0.clone(), o["c"][0]
        if in_place:
            o["c"][0] = c_out = c_in
        plan = edkm.Plan(n, 3, 5)
        if dense:
            edkm.forward_dense(plan, keys, inputs.TAU, 0.0, c_in, c_out, o["wt"][0], False, o["it"][0])
            edkm.backward_dense(plan, keys, g, o["gw"][0], o["gc"][0])
        else:
            edkm.init_unique(plan, keys)
            edkm.forward(plan, keys, inputs.TAU, 0.0, c_in, c_out, o["wt"][0], False, o["it"][0])
            edkm.backward(plan, keys, g, o["gw"][0], o["gc"][0])
        torch.cuda.synchronize()
        res.append(o)
    assert not same_bits(res[1]["c"][0].cpu().numpy(), c0.cpu().numpy())
    for name in res[0]:
        assert same_bits(res[0][name][0].cpu().numpy(), res[1][name][0].cpu().numpy()), name

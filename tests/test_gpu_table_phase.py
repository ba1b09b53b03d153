"""The table phases' launch shapes: batches at the edges of one block per
virtual block, two virtual blocks per block and several launches give, bit for
bit, what single calls give (which one launch of 64 blocks computes), and a
forward or backward repeated after one init_unique, or after a failed forward,
starts from clean exchange rows."""
import os
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2309_00964_amd import edkm, inputs                     # noqa: E402
from paper_2309_00964_amd.runner import run                       # noqa: E402
from parity_util import assert_close                              # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("bits,count", [(1, 17), (2, 28), (3, 16), (3, 17), (4, 8), (4, 9), (4, 16), (4, 17)])
def test_batches_equal_single_calls(bits, count):
    print("[gpu-case] table phase bits", bits, "count", count, flush=True)
    sys.stdout.flush()
    k, iters = 1 << bits, 3
    sizes = [4001 + 37 * i for i in range(count)]
    keys_h = [inputs.fp16_weights(n, 700 + i) for i, n in enumerate(sizes)]
    keys = [torch.from_numpy(x.view(np.int16)).to(DEV) for x in keys_h]
    c0 = [torch.from_numpy(inputs.quantile_init(x, k)).to(DEV) for x in keys_h]
    g = [torch.from_numpy(inputs.upstream_grad(n, 800 + i)).to(DEV) for i, n in enumerate(sizes)]
    plans = [edkm.Plan(n, bits, iters, device=DEV) for n in sizes]
    co = [torch.empty(k, device=DEV) for _ in sizes]
    wt = [torch.empty(n, device=DEV) for n in sizes]
    gw = [torch.empty(n, device=DEV) for n in sizes]
    gc = [torch.empty(k, device=DEV) for _ in sizes]
    edkm.init_unique_batch(plans, keys)
    edkm.forward_batch(plans, keys, inputs.TAU, 0.0, c0, co, wt)
    edkm.backward_batch(plans, keys, g, gw, gc)
    torch.cuda.synchronize()
    for i in range(count):
        s = run(keys[i], c0[i], bits, inputs.TAU, iters, grad=g[i])
        torch.cuda.synchronize()
        assert torch.equal(co[i], s["c_out"]) and torch.equal(wt[i], s["w_tilde"]), i
        # bit for bit too: one workgroup takes all of a matrix in either call, and no
        # gradient is beyond the keyed sum's fixed-point range (those that are go to
        # G with float atomics, whose order is not fixed)
        assert torch.equal(gw[i], s["grad_w"]) and torch.equal(gc[i], s["grad_c"]), i


def test_forward_repeated_after_one_init():
    """The same plan: three forwards with other C^(0), tau and early stops (so
    that rows of later iterations stay unused in some), each equal to a fresh
    plan's, then the backward of the last."""
    n, iters = 30_011, 9
    kh = inputs.fp16_weights(n, 720)
    keys = torch.from_numpy(kh.view(np.int16)).to(DEV)
    c0 = torch.from_numpy(inputs.quantile_init(kh, 8)).to(DEV)
    g = torch.from_numpy(inputs.upstream_grad(n, 721)).to(DEV)
    plan = edkm.Plan(n, 3, iters, device=DEV)
    co, wt = torch.empty(8, device=DEV), torch.empty(n, device=DEV)
    it = torch.zeros(1, dtype=torch.int32, device=DEV)
    edkm.init_unique(plan, keys)
    for tau, eps, scale in ((2e-3, 0.0, 1.0), (4e-3, 1.0, 0.9), (2e-3, 1e-3, 1.1), (1e-3, 0.0, 0.8)):
        print("[gpu-case] repeated forward", tau, eps, scale, flush=True)
        c = c0 * scale
        edkm.forward(plan, keys, tau, eps, c, co, wt, False, it)
        s = run(keys, c, 3, tau, iters, eps=eps, grad=g)
        torch.cuda.synchronize()
        assert torch.equal(it, s["iters"]) and torch.equal(co, s["c_out"]) and torch.equal(wt, s["w_tilde"])
    gw, gc = torch.empty(n, device=DEV), torch.empty(8, device=DEV)
    edkm.backward(plan, keys, g, gw, gc)
    torch.cuda.synchronize()
    assert_close(gw.cpu().numpy(), s["grad_w"].cpu().numpy(), 1e-5, "grad_w")
    assert_close(gc.cpu().numpy(), s["grad_c"].cpu().numpy(), 1e-5, "grad_c")


@pytest.mark.parametrize("max_iter", [9, 1024])
def test_rows_of_the_iterations_run_are_emptied(max_iter):
    """One plan, forwards that stop after many, one, several iterations, a backward
    after each (twice after the last): every step gives a fresh plan's bits."""
    n = 15_001                                        # one workgroup per N-sized pass: no atomic's order matters
    kh = inputs.fp16_weights(n, 740)
    keys = torch.from_numpy(kh.view(np.int16)).to(DEV)
    c0 = torch.from_numpy(inputs.quantile_init(kh, 16)).to(DEV)
    g = torch.from_numpy(inputs.upstream_grad(n, 741)).to(DEV)
    plan = edkm.Plan(n, 4, max_iter, device=DEV)
    co, wt, gw, gc = (torch.empty(m, device=DEV) for m in (16, n, n, 16))
    it = torch.zeros(1, dtype=torch.int32, device=DEV)
    edkm.init_unique(plan, keys)
    seen = []
    for eps in (2e-4, 1.0, 1e-3, 2e-4):
        print("[gpu-case] rows emptied", max_iter, eps, flush=True)
        edkm.forward(plan, keys, inputs.TAU, eps, c0, co, wt, False, it)
        s = run(keys, c0, 4, inputs.TAU, max_iter, eps=eps, grad=g)
        for rep in range(2 if len(seen) == 3 else 1):
            edkm.backward(plan, keys, g, gw, gc)
            torch.cuda.synchronize()
            for name, x in (("iters", it), ("c_out", co), ("w_tilde", wt), ("grad_w", gw), ("grad_c", gc)):
                assert torch.equal(x, s[name]), (eps, rep, name)
        seen.append(int(it.item()))
    assert seen[1] == 1 and seen[0] > seen[2] > 1, seen


def forward_after_a_failed_one():
    import ctypes
    hip = ctypes.CDLL([x for x in edkm._hip_runtimes()][0])
    n, iters, k = 20_011, 4, 8
    kh = inputs.fp16_weights(n, 730)
    keys = torch.from_numpy(kh.view(np.int16)).to(DEV)
    c0 = torch.from_numpy(inputs.quantile_init(kh, k)).to(DEV)
    co, wt = torch.empty(k, device=DEV), torch.empty(n, device=DEV)
    plan = edkm.Plan(n, 3, iters, workspace=torch.zeros(edkm.workspace_bytes(n, 3, iters), dtype=torch.uint8, device=DEV))
    want = run(keys, c0, 3, inputs.TAU, iters)
    edkm.init_unique(plan, keys)
    # the rows: the words that init_unique emptied (all ones) in a workspace of zeros
    words = plan.workspace.view(torch.int32)
    at = torch.nonzero(words == -1).flatten()
    assert at.numel() == iters * 64 * 2 * k and int(at[-1] - at[0]) == at.numel() - 1
    rows = words[int(at[0]):int(at[-1]) + 1]

    def forward(stream):
        co.zero_(), wt.zero_()
        torch.cuda.synchronize()
        edkm.forward(plan, keys, inputs.TAU, 0.0, c0, co, wt, stream=stream)

    def check(what):
        torch.cuda.synchronize()
        assert torch.equal(co, want["c_out"]) and torch.equal(wt, want["w_tilde"]), what
        assert bool((rows == -1).all())

    s = torch.cuda.Stream()
    forward(s)
    check("before")
    print("[gpu-case] forward into an invalidated capture", flush=True)
    raw, graph = ctypes.c_void_p(), ctypes.c_void_p()      # a stream of its own: it stays invalidated
    assert hip.hipStreamCreateWithFlags(ctypes.byref(raw), 1) == 0
    assert hip.hipStreamBeginCapture(raw, 2) == 0          # relaxed
    assert hip.hipStreamSynchronize(raw) != 0              # not allowed: invalidates the capture
    with pytest.raises(edkm.EdkmError) as e:
        edkm.forward(plan, keys, inputs.TAU, 0.0, c0, co, wt, stream=raw.value)
    assert e.value.status == edkm.ERR_HIP
    assert hip.hipStreamEndCapture(raw, ctypes.byref(graph)) != 0
    hip.hipGetLastError()

    print("[gpu-case] forward on full rows", flush=True)
    full = torch.linspace(0.5, 2.0, rows.numel(), device=DEV).view(torch.int32)
    rows.copy_(full)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        edkm.forward(plan, keys, inputs.TAU, 0.0, c0, co, wt)
    forward(s)                                             # the graph has not run
    check("eager")
    for rep in range(3):
        rows.copy_(full)
        co.zero_(), wt.zero_()
        torch.cuda.synchronize()
        g.replay()
        check("replay %d" % rep)
    print("failed forward ok", flush=True)


def test_forward_after_one_that_failed_between_its_launches():
    """A failed forward may leave its exchange rows full.  The failure is a launch
    into a capture that has been invalidated (in a process of its own); what the
    launches before it would have left is written into the rows by hand.  A later
    forward empties them first, eagerly and captured, and a captured one that has
    not been replayed does not stand in for that."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.abspath(__file__)], cwd=root, capture_output=True, text=True,
                       timeout=110, env=dict(os.environ, PYTHONPATH=root))
    assert r.returncode == 0 and "failed forward ok" in r.stdout, (r.stdout[-1000:], r.stderr[-3000:])


if __name__ == "__main__":
    forward_after_a_failed_one()

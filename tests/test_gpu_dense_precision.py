"""The dense backward's rounding where map rows are nearly one-hot (small tau,
weights far outside the centroids): dL/dw and dL/dC^(0) of one iteration against
fp64.  Half the weights have no upstream gradient, so that their dL/dw_i is the
part through the centroids alone (the direct part g_i H_i is otherwise far
larger).  A row's deviations p_j - sum_i a_i p_i, p_j = gS_j (v - C_j), enter
divided by tau; taken as the difference of two numbers of size |p| they carry
about 2^-23 |p| / tau each, taken around a reference that the dominant entry
leaves at zero they carry a rounding of their own, smaller size."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import table                                           # noqa: E402
from paper_2309_00964_amd import inputs                            # noqa: E402
from paper_2309_00964_amd.runner import run                        # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda"
N = 40_000
# dL/dw_i here is about ten fp32 roundings (v - C, gS (v - C), the exponent and its
# power, the row's factor, the mean, the sum over j, 1/tau, the last addition) of
# at most 2^-24 of the result's size each; rel-L2 averages them.  Measured: rel-L2
# up to 3.3e-7, largest 4.5e-7.  With the deviations taken as the plain difference
# from the mean: largest 1.8e-6 to 7.1e-6 at tau = 2e-3, rel-L2 4.2e-7 to 5.3e-7
# at tau = 1e-4.  dL/dC^(0), a sum over all weights, cancels more (measured 1.9e-6).
U = 2.0 ** -24
BAR_L2, BAR_MAX, BAR_C = 7 * U, 10 * U, 1e-5


@pytest.mark.parametrize("tau", [2e-3, 5e-4, 1e-4])
@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_dense_gradients_of_nearly_one_hot_rows(bits, tau):
    print("[gpu-case] dense precision", bits, tau, flush=True)
    sys.stdout.flush()
    k = 1 << bits
    keys = inputs.fp16_weights(N, 300 + bits, True)                # 0.1% of the weights ten times wider
    c0 = np.asarray(inputs.quantile_init(keys, k), np.float32)
    g = inputs.upstream_grad(N, 310 + bits)
    g[::2] = 0
    o = run(torch.from_numpy(keys.view(np.int16)).to(DEV), torch.from_numpy(c0), bits, tau, 1,
            grad=torch.from_numpy(g), dense=True)
    torch.cuda.synchronize()
    f = table.forward(keys, c0.astype(np.float64), tau, 1)
    gw, gc = table.backward(keys, f, g.astype(np.float64))[:2]
    gw = gw[::2]
    ew = o["grad_w"].cpu().numpy().astype(np.float64)[::2] - gw
    ec = o["grad_c"].cpu().numpy().astype(np.float64) - gc
    l2w, mxw = np.linalg.norm(ew) / np.linalg.norm(gw), np.abs(ew).max() / np.abs(gw).max()
    l2c = np.linalg.norm(ec) / np.linalg.norm(gc)
    print("bits %d tau %.0e: dL/dw rel-L2 %.2e max %.2e, dL/dC rel-L2 %.2e" % (bits, tau, l2w, mxw, l2c), flush=True)
    assert l2w <= BAR_L2 and mxw <= BAR_MAX and l2c <= BAR_C

"""Forwards and backwards over the table phases' launch shapes, saved to the file
named on the command line: run once per build of the library (EDKM_LIBRARY)
and compared by test_gpu_exchange.py.  Every matrix is small enough for one
workgroup per N-sized pass and its gradients stay within the keyed sum's
fixed-point range, so that no result depends on the order of an atomic."""
import sys

import numpy as np
import torch

from paper_2309_00964_amd import edkm, inputs

DEV = "cuda"
# bits, matrices, iterations, eps, weight format.  A block runs one virtual block,
# two (from 17 matrices; the backward at 4 bits from 13) or four (the backward at 4
# bits from 17); full launch groups; early stops at different iterations in a batch
CASES = [(1, 1, 3, 0.0, "fp16"), (2, 1, 5, 0.0, "bf16"), (3, 1, 5, 0.0, "fp16"), (4, 1, 4, 0.0, "fp16"),
         (1, 28, 3, 0.0, "fp16"), (2, 17, 3, 0.0, "fp16"), (3, 28, 3, 0.0, "bf16"), (4, 9, 3, 0.0, "fp16"),
         (4, 16, 3, 0.0, "fp16"), (4, 17, 3, 0.0, "bf16"), (4, 28, 2, 0.0, "fp16"), (3, 5, 12, 5e-4, "fp16"),
         (4, 17, 12, 2e-4, "fp16")]


def case_inputs(bits, count, fmt):
    k = 1 << bits
    sizes = [4001 + 401 * i for i in range(count)]
    keys_h = [inputs.weights(n, 7000 + 100 * bits + i, False, fmt) for i, n in enumerate(sizes)]
    keys = [torch.from_numpy(x.view(np.int16)).to(DEV) for x in keys_h]
    c0 = [torch.from_numpy(np.asarray(inputs.quantile_init(x, k, fmt), np.float32) * np.float32(1 + 0.03 * i)).to(DEV)
          for i, x in enumerate(keys_h)]
    g = [torch.from_numpy(inputs.upstream_grad(n, 8000 + i)).to(DEV) for i, n in enumerate(sizes)]
    return sizes, keys, c0, g


def outputs(sizes, k):
    return dict(c=[torch.empty(k, device=DEV) for _ in sizes], wt=[torch.empty(n, device=DEV) for n in sizes],
                it=[torch.zeros(1, dtype=torch.int32, device=DEV) for _ in sizes],
                gw=[torch.empty(n, device=DEV) for n in sizes], gc=[torch.empty(k, device=DEV) for _ in sizes])


def main(out):
    res = {}
    for q, (bits, count, iters, eps, fmt) in enumerate(CASES):
        sizes, keys, c0, g = case_inputs(bits, count, fmt)
        o = outputs(sizes, 1 << bits)
        plans = [edkm.Plan(n, bits, iters, key_format=fmt) for n in sizes]
        print("[gpu-case] exchange", bits, count, iters, eps, fmt, flush=True)
        edkm.init_unique_batch(plans, keys)
        edkm.forward_batch(plans, keys, inputs.TAU, eps, c0, o["c"], o["wt"], False, o["it"])
        # the repeated forward starts from emptied rows; its centroids are updated in place
        for c, x in zip(o["c"], c0):
            c.copy_(x)
        edkm.forward_batch(plans, keys, inputs.TAU, eps, o["c"], o["c"], o["wt"], False, o["it"])
        edkm.backward_batch(plans, keys, g, o["gw"], o["gc"])
        torch.cuda.synchronize()
        for name, xs in o.items():
            for i, x in enumerate(xs):
                res["%d.%s.%d" % (q, name, i)] = x.cpu().numpy()
    np.savez(out, **res)


if __name__ == "__main__":
    main(sys.argv[1])

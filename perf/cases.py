"""The calls whose time matters to a user of the library, as cases that a timing
program can list, draw, prepare and run.

A case is a dict of plain values:

* ``kind``: which public calls one pass makes.
  - ``step``: init_unique, forward and backward through plans that the program
    keeps (the batched calls for more than one matrix): one training step's
    clustering;
  - ``autograd``: the same through ``function.dkm`` / ``dkm_batch`` and torch's
    autograd, which make their plans on each call;
  - ``forward``: init_unique and forward only, with early stop (clustering
    after training);
  - ``palettize``: the packed b-bit indices of the compressed model;
  - ``unique``: init_unique with counts, then the distinct patterns and the
    inverse index;
  - ``dense``: the comparison path, forward_dense and backward_dense.
* ``sizes``: weights per matrix, comma-separated; ``fmt`` of the weights;
  ``bits``; ``half``: W~, dL/dW~ and dL/dw in the weights' 16-bit format
  instead of fp32; ``iters`` and ``eps``: DKM iterations at most and the early
  stop; ``outliers``: 0.1% of the weights drawn ten times wider; ``flat``: the
  matrices lie one after another in flat buffers (from element 1 on), so that
  odd sizes leave most of them unaligned, as the pieces of a sharded flat
  parameter do.

Weights are N(0, 0.02^2) rounded to 16 bits, starting centroids the k evenly
spaced quantiles, dL/dW~ is N(0, 1), tau = 2e-3.
"""
import torch

from paper_2309_00964_amd import edkm, function, inputs

TAU = inputs.TAU
DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}

_BASE = dict(fmt="fp16", bits=3, half=False, iters=5, eps=0.0, outliers=False, flat=False)


def _case(name, kind, sizes, **kw):
    c = dict(_BASE, name=name, kind=kind, sizes=",".join(str(n) for n in sizes))
    c.update(kw)
    return c


_ATTN, _MLP = 4096 * 4096, 11008 * 4096
_LAYER = tuple(r * c for _, r, c in inputs.LLAMA7B_LAYER)


def listed():
    return [
        # the smallest whole step: a 256x256 matrix, all latency
        _case("step_256x256", "step", [256 * 256]),
        # one attention projection of LLaMA-7B
        _case("step_4096x4096", "step", [_ATTN]),
        # one MLP matrix with outliers, at the widest table
        _case("step_11008x4096_b4", "step", [_MLP], bits=4, outliers=True),
        # a whole LLaMA-7B decoder layer, seven matrices batched, fp32 W~ and gradients
        _case("step_layer", "step", _LAYER),
        # four decoder layers in one batch: the largest launch group of the 32-layer stack
        _case("step_4_layers_b2", "step", 4 * _LAYER, bits=2),
        # pieces of a sharded flat bf16 parameter: odd sizes, unaligned starts, 16-bit arrays
        _case("step_flat_shards", "step", [1000003, 262147, 65539], fmt="bf16", half=True, flat=True),
        # a decoder layer in a bf16 training step through autograd
        _case("autograd_layer_bf16", "autograd", _LAYER, fmt="bf16", half=True),
        # one module's weight through autograd, as a training script clusters it
        _case("autograd_1024x4096_b4", "autograd", [1024 * 4096], bits=4),
        # clustering a trained bf16 matrix until its centroids stand still
        _case("forward_eps_4096x4096", "forward", [_ATTN], fmt="bf16", bits=4, iters=30, eps=1e-4),
        # export of a clustered decoder layer
        _case("palettize_layer", "palettize", _LAYER),
        # the paper's two lists (distinct patterns, index per weight) of an MLP matrix
        _case("unique_11008x4096", "unique", [_MLP], outliers=True),
        # the comparison path: the map recomputed per weight in every iteration
        _case("dense_4096x4096", "dense", [_ATTN]),
    ]


def _size(rng, lo, hi):
    n = int(lo * (hi / lo) ** rng.random())
    return n | 1 if rng.random() < 0.5 else max(8, n & ~7)


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "autograd", "autograd", "forward", "palettize", "unique", "dense"])
    many = kind != "dense" and rng.random() < 0.4
    if many:
        m = rng.randint(2, 12)
        sizes = [_size(rng, 16384, _ATTN) for _ in range(m)]
    else:
        sizes = [_size(rng, 4096, 1 << 22 if kind == "dense" else _MLP)]
    return dict(
        kind=kind,
        sizes=",".join(str(n) for n in sizes),
        fmt=rng.choice(["fp16", "bf16"]),
        bits=rng.randint(1, 4),
        half=kind in ("step", "autograd", "forward") and rng.random() < 0.4,
        iters=30 if kind == "forward" else rng.randint(2, 8),
        eps=1e-4 if kind == "forward" else 0.0,
        outliers=rng.random() < 0.3,
        flat=many and kind == "step" and rng.random() < 0.3,
    )


def _sizes(case):
    return [int(s) for s in case["sizes"].split(",")]


def _pieces(sizes, flat, make):
    """One buffer holding all matrices, and a view per matrix.  Without ``flat``
    each matrix starts on a multiple of 64 elements."""
    at, starts = 1 if flat else 0, []
    for n in sizes:
        starts.append(at)
        at += n if flat else (n + 63) // 64 * 64
    buf = make(at)
    return buf, [buf[s:s + n] for s, n in zip(starts, sizes)]


def _keys_c0_grad(case, seed, dev):
    """Weights (their own 16-bit type), C^(0) and dL/dW~ of every matrix."""
    sizes, fmt, k = _sizes(case), case["fmt"], 1 << case["bits"]
    dt = DTYPES[fmt]
    _, ws = _pieces(sizes, case["flat"], lambda n: torch.zeros(n, dtype=dt, device=dev))
    c0 = []
    for i, w in enumerate(ws):
        keys = inputs.fp16_weights_device(w.numel(), 1000 * seed + i, dev, case["outliers"], fmt)
        w.copy_(keys.view(dt))
        c0.append(inputs.quantile_init_device(keys, k, fmt))
    gs = None
    if case["kind"] in ("step", "autograd", "dense"):
        gt = dt if case["half"] else torch.float32
        _, gs = _pieces(sizes, case["flat"], lambda n: torch.zeros(n, dtype=gt, device=dev))
        for i, g in enumerate(gs):
            g.copy_(inputs.upstream_grad_device(g.numel(), 1000 * seed + 500 + i, dev))
    return ws, c0, gs


def prepare(case, seed):
    dev = torch.device("cuda:0")
    sizes, kind, k = _sizes(case), case["kind"], 1 << case["bits"]
    ws, c0, gs = _keys_c0_grad(case, seed, dev)
    s = dict(case=case, ws=ws, c0=c0, gs=gs)
    if kind == "autograd":
        s["ws"] = [w.clone().requires_grad_(True) for w in ws]
        s["c0"] = [c.requires_grad_(True) for c in c0]
        return s
    m = len(sizes)
    s["keys"] = [w.view(torch.int16) for w in ws]
    s["plans"] = [edkm.Plan(n, case["bits"], case["iters"], device=dev, key_format=case["fmt"]) for n in sizes]
    out_t = DTYPES[case["fmt"]] if case["half"] else torch.float32

    def outputs(dtype):
        return _pieces(sizes, case["flat"], lambda n: torch.zeros(n, dtype=dtype, device=dev))

    if kind in ("step", "forward", "dense"):
        s["wt_buf"], s["wt"] = outputs(out_t)
        s["c_buf"] = torch.zeros(m, k, device=dev)
        s["iters_buf"] = torch.zeros(m, dtype=torch.int32, device=dev)
    if kind in ("step", "dense"):
        s["gw_buf"], s["gw"] = outputs(out_t)
        s["gc_buf"] = torch.zeros(m, k, device=dev)
    if kind == "palettize":
        s["lut"] = [c.contiguous() for c in c0]
        s["idx"] = [torch.zeros((n * case["bits"] + 7) // 8, dtype=torch.uint8, device=dev) for n in sizes]
    if kind == "unique":
        s["counts"] = torch.zeros(m, edkm.NKEYS, dtype=torch.int32, device=dev)
        s["nu"] = torch.zeros(m, dtype=torch.int32, device=dev)
        s["uniq"] = torch.zeros(m, edkm.NKEYS, dtype=torch.int16, device=dev)
        s["inv_buf"], s["inv"] = outputs(torch.int16)
    return s


def run(s):
    case = s["case"]
    kind, eps = case["kind"], case["eps"]
    if kind == "autograd":
        if len(s["ws"]) == 1:
            wt, c, it = function.dkm(s["ws"][0], s["c0"][0], TAU, case["iters"], eps, case["half"])
            wts, cs, its = [wt], [c], [it]
        else:
            wts, cs, its = function.dkm_batch(s["ws"], s["c0"], TAU, case["iters"], eps, case["half"])
        m = len(wts)
        g = torch.autograd.grad(wts, [*s["ws"], *s["c0"]], [x.view(w.shape) for x, w in zip(s["gs"], wts)])
        return dict(w_tilde=[w.detach() for w in wts], c_out=torch.stack(cs), iters=torch.cat(its),
                    grad_w=list(g[:m]), grad_c0=torch.stack(g[m:]))
    plans, keys = s["plans"], s["keys"]
    if kind == "palettize":
        edkm.palettize_batch(plans, keys, s["lut"], s["idx"])
        return s["idx"]
    if kind == "unique":
        edkm.init_unique_batch(plans, keys, list(s["counts"]), list(s["nu"].split(1)))
        edkm.unique_inverse_batch(plans, keys, list(s["uniq"]), s["inv"])
        return dict(counts=s["counts"], num_unique=s["nu"], unique=s["uniq"], inverse=s["inv_buf"])
    out = dict(w_tilde=s["wt_buf"], c_out=s["c_buf"], iters=s["iters_buf"])
    if kind == "dense":
        edkm.forward_dense(plans[0], keys[0], TAU, eps, s["c0"][0], s["c_buf"][0], s["wt"][0], case["half"],
                           s["iters_buf"])
        edkm.backward_dense(plans[0], keys[0], s["gs"][0], s["gw"][0], s["gc_buf"][0])
        return dict(out, grad_w=s["gw_buf"], grad_c0=s["gc_buf"])
    if len(plans) == 1:
        edkm.init_unique(plans[0], keys[0])
        edkm.forward(plans[0], keys[0], TAU, eps, s["c0"][0], s["c_buf"][0], s["wt"][0], case["half"],
                     s["iters_buf"])
        if kind == "step":
            edkm.backward(plans[0], keys[0], s["gs"][0], s["gw"][0], s["gc_buf"][0])
    else:
        edkm.init_unique_batch(plans, keys)
        edkm.forward_batch(plans, keys, TAU, eps, s["c0"], list(s["c_buf"]), s["wt"], case["half"],
                           list(s["iters_buf"].split(1)))
        if kind == "step":
            edkm.backward_batch(plans, keys, s["gs"], s["gw"], list(s["gc_buf"]))
    if kind == "step":
        out.update(grad_w=s["gw_buf"], grad_c0=s["gc_buf"])
    return out


def work(case):
    n, k, kind = sum(_sizes(case)), 1 << case["bits"], case["kind"]
    m = len(_sizes(case))
    e = 2 if case["half"] else 4
    if kind == "palettize":
        return {"bytes": n * (2 + case["bits"] / 8), "flops": m * edkm.NKEYS * 3 * k}
    if kind == "unique":
        return {"bytes": 4 * n + m * edkm.NKEYS * 6, "flops": 0}
    if kind == "forward":
        return {"bytes": n * (2 + e), "flops": m * edkm.NKEYS * 9 * k}
    rows = n if kind == "dense" else m * edkm.NKEYS     # rows of the map evaluated
    # 9 operations per map entry of a forward iteration, 15 of a backward one
    return {"bytes": n * (2 + 3 * e), "flops": rows * k * 24 * case["iters"]}


def tolerance(case):
    if case["kind"] in ("palettize", "unique"):
        return "exact"
    if case["half"]:
        return {"rel": 8e-3 if case["fmt"] == "bf16" else 1e-3}
    if case["kind"] == "autograd":                       # fp32 W~, dL/dw in the weights' type
        return {"rel": 8e-3 if case["fmt"] == "bf16" else 1e-3}
    return {"rel": 1e-5}


# ---------------------------------------------------------------------------
# the same results in 64 bits, by torch's own autograd on the distinct values


def _table64(keys, fmt, c0, iters, eps):
    """Distinct weight values, each weight's index among them, W~ per value,
    C^(T), T, and the graph's inputs (the values as the centroid sums see them,
    as the last map sees them, C^(0))."""
    u, inv, n = torch.unique(keys.to(torch.int32) & 0xFFFF, return_inverse=True, return_counts=True)
    v = u.to(torch.int16).view(DTYPES[fmt]).double()
    va, vb = v.clone().requires_grad_(True), v.clone().requires_grad_(True)
    c = c_start = c0.detach().double().clone().requires_grad_(True)
    nd = n.double()[:, None]
    t_done, prev = 0, c
    for t in range(1, iters + 1):
        a = torch.softmax(-(va[:, None] - c[None, :]).abs() / TAU, 1) * nd
        sj = a.sum(0)
        new = torch.where(sj > 0, (a * va[:, None]).sum(0) / torch.where(sj > 0, sj, torch.ones_like(sj)), c)
        prev, c, t_done = c, new, t
        if eps > 0 and float((c - prev).abs().max()) <= eps:
            break
    wt = torch.softmax(-(vb[:, None] - prev[None, :]).abs() / TAU, 1) @ c
    return inv, nd[:, 0], wt, c, t_done, va, vb, c_start


def exact(case, seed):
    kind, sizes = case["kind"], _sizes(case)
    if kind in ("palettize", "unique") or sum(sizes) > 250_000_000:
        return None
    dev = torch.device("cuda:0")
    ws, c0, gs = _keys_c0_grad(case, seed, dev)
    wt_buf, wts = _pieces(sizes, case["flat"], lambda n: torch.zeros(n, dtype=torch.float64, device=dev))
    gw_buf, gws = _pieces(sizes, case["flat"], lambda n: torch.zeros(n, dtype=torch.float64, device=dev))
    cs, gcs = [], []
    for i, w in enumerate(ws):
        inv, nd, tab, c, _, va, vb, cst = _table64(w.view(torch.int16), case["fmt"], c0[i], case["iters"], case["eps"])
        wts[i].copy_(tab.detach()[inv])
        cs.append(c.detach())
        if gs is None:
            continue
        g = gs[i].double()
        gsum = torch.zeros_like(nd).index_add_(0, inv, g)
        (h,) = torch.autograd.grad(tab.sum(), vb, retain_graph=True)
        ra, gc = torch.autograd.grad(tab, [va, cst], gsum)
        gws[i].copy_(g * h[inv] + (ra / nd)[inv])
        gcs.append(gc)
    if kind == "autograd":
        return dict(w_tilde=wts, c_out=torch.stack(cs), iters=None, grad_w=gws, grad_c0=torch.stack(gcs))
    out = dict(w_tilde=wt_buf, c_out=torch.stack(cs), iters=None)
    if gs is not None:
        out.update(grad_w=gw_buf, grad_c0=torch.stack(gcs))
    return out

"""How far values and gradients are from float64, problem by problem, with bars close to what the arithmetic gives.

The parity bars (1e-4, 1e-3) say that a result is right; they do not notice when it loses a digit or two.  Here
eighteen seeded problems, of the kinds that the entry points take, have bars of their own on the relative 2-norm of the
error.  A bar is four times the largest of three figures:
  - what float64 DP tables gave on the GPU (results are reproducible, so the factor is for other orders of the sums);
  - what float32 costs alone give: each is off by about COST_ERROR (||x||^2 + ||y||^2), which moves the weights of
    competing alignments by that over gamma (modelled on the CPU: the oracle on perturbed costs);
  - what storing the results in float32 costs.
A pair with two alignments of nearly equal weight can have 100 times the error of the others, whatever the arithmetic;
the median over the pairs is what tells one arithmetic from another.  Table entries with a 24-bit mantissa, whose
rounding differs between the two sweeps and adds up along the alignment, give 3.5e-7 to 7.2e-7 there in the problems
l256, l256_unfused, walk_*, bfloat16 and normalized, where float64 ones give 0.04e-7 to 1.5e-7, and miss the bars of all
of these but walk_rectangular's.
"""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from paper_2602_17206_amd import workloads

COST_ERROR = 8e-8  # rms error of a float32 cost over ||x||^2 + ||y||^2 (measured: 4.6e-8 to 7.9e-8, D = 2 ... 200)

# name: (entry point, B, N, M, D, gamma, mode, data, options)
PROBLEMS = {
    "tiny": ("grad", 4, 64, 64, 8, 1.0, "unfused", "normal", {}),
    "l256": ("grad", 8, 256, 256, 128, 0.1, "fused", "normal", {}),
    "l256_unfused": ("grad", 8, 256, 256, 128, 0.1, "unfused", "normal", {}),
    "l512_d128": ("grad", 4, 512, 512, 128, 1.0, "fused", "normal", {}),
    "l512_d32": ("grad", 4, 512, 512, 32, 1.0, "fused", "normal", {}),
    "walk_l1024": ("grad", 4, 1024, 1024, 128, 0.1, "fused", "walk", {}),
    "walk_l1024_unfused": ("grad", 4, 1024, 1024, 128, 0.1, "unfused", "walk", {}),
    "odd_unfused": ("grad", 5, 300, 237, 50, 0.1, "unfused", "normal", {}),
    "walk_rectangular": ("grad", 4, 700, 600, 64, 0.05, "fused", "walk", {}),
    "wide": ("grad", 4, 256, 256, 200, 1.0, "fused", "normal", {}),
    "dense": ("grad", 4, 512, 512, 2, 0.5, "fused", "walk", {}),
    "banded": ("grad", 4, 1024, 1024, 64, 0.1, "fused", "normal", {"bandwidth": 64}),
    "long_compact": ("grad", 2, 2048, 1900, 128, 0.01, "fused", "normal", {"min_memory": True}),
    "ragged": ("ragged", 8, 512, 512, 39, 1.0, "fused", "normal", {}),
    "float16": ("half", 4, 512, 512, 128, 1.0, "fused", "normal", {"half_type": "float16"}),
    "bfloat16": ("half", 8, 256, 256, 64, 0.1, "unfused", "normal", {"half_type": "bfloat16"}),
    "normalized": ("normalized", 8, 256, 256, 128, 0.1, "fused", "normal", {}),
    "barycenter": ("grad", 8, 512, 512, 32, 1.0, "fused", "warped", {}),
}

# name: what errors() gave, (value, gradients, gradients of the median pair): on the GPU with float64 tables / the largest
# of four draws of the oracle on perturbed costs
MEASURED = {
    "tiny": ((1.3e-08, 3.4e-07, 3.2e-07), (3.1e-08, 8.3e-07, 6.0e-07)),
    "l256": ((1.4e-08, 4.5e-06, 4.2e-08), (1.6e-08, 2.7e-05, 2.8e-08)),
    "l256_unfused": ((1.4e-08, 4.7e-08, 4.2e-08), (1.4e-08, 4.2e-08, 2.8e-08)),
    "l512_d128": ((1.5e-08, 2.1e-06, 1.8e-06), (1.5e-08, 1.0e-06, 8.7e-07)),
    "l512_d32": ((2.2e-08, 2.2e-06, 2.4e-06), (2.2e-08, 5.0e-06, 2.4e-06)),
    "walk_l1024": ((2.1e-08, 4.3e-08, 4.2e-08), (2.1e-08, 3.2e-08, 3.0e-08)),
    "walk_l1024_unfused": ((2.4e-08, 4.2e-08, 4.2e-08), (2.4e-08, 2.9e-08, 2.8e-08)),
    "odd_unfused": ((2.0e-08, 4.1e-06, 8.9e-07), (2.1e-08, 6.8e-06, 1.9e-06)),
    "walk_rectangular": ((1.9e-08, 2.5e-07, 1.5e-07), (1.9e-08, 7.4e-07, 5.8e-07)),
    "wide": ((5.7e-09, 5.4e-07, 7.2e-08), (5.7e-09, 1.4e-06, 1.1e-07)),
    "dense": ((3.2e-08, 6.4e-07, 6.5e-07), (3.1e-08, 8.8e-07, 7.1e-07)),
    "banded": ((1.0e-08, 2.1e-05, 7.5e-07), (1.0e-08, 7.9e-05, 3.3e-06)),
    "long_compact": ((1.2e-08, 2.0e-07, 1.6e-07), (1.2e-08, 2.9e-06, 2.1e-06)),
    "ragged": ((3.1e-08, 9.6e-07, 7.6e-07), (3.2e-08, 2.6e-06, 1.5e-06)),
    "float16": ((1.9e-08, 3.6e-06, 1.2e-06), (1.6e-08, 4.8e-05, 1.6e-06)),
    "bfloat16": ((3.0e-08, 1.7e-06, 4.0e-09), (1.8e-08, 1.2e-05, 3.8e-09)),
    "normalized": ((9.7e-08, 7.7e-08, 5.2e-08), (3.9e-08, 1.4e-06, 3.3e-08)),
    "barycenter": ((6.1e-07, 7.0e-06, 7.0e-06), (1.9e-07, 7.0e-06, 6.9e-06)),
}
STORED = 2.0 ** -25  # about what storing the results in float32 costs


def bars(name):
    return [4 * max(gpu, model, STORED) for gpu, model in zip(*MEASURED[name])]


def inputs(name):
    """x, y (float32, as the library gets them; rounded to the half type where the entry point takes one), lengths."""
    entry, B, N, M, D, gamma, _, data, options = PROBLEMS[name]
    seed = 9000 + sorted(PROBLEMS).index(name)
    if data == "warped":  # one averaged sequence against the noisy copies of it
        w = workloads.barycenter_workload(K=B, L=N, D=D, seed=seed, gamma=gamma)
        return w.z0, w.X, None, None
    x, y = (workloads.normal_pairs if data == "normal" else workloads.walk_pairs)(seed, B, N, M, D)
    if entry == "half":
        import torch

        t = getattr(torch, options["half_type"])
        x, y = (torch.from_numpy(a).to(t).float().numpy() for a in (x, y))
    if entry == "ragged":
        return x, y, workloads.ragged_lengths(seed, B, N, N // 4), workloads.ragged_lengths(seed + 1, B, M, M // 4)
    return x, y, None, None


def reference(name, x, y, xl, yl):
    entry, gamma, options = PROBLEMS[name][0], PROBLEMS[name][5], PROBLEMS[name][8]
    if entry == "ragged":
        return oracle.ragged_batch(x, y, xl, yl, gamma)
    if entry == "normalized":
        return oracle.normalized(x, y, gamma)
    return oracle.batch(x, y, gamma, bandwidth=options.get("bandwidth"))


def run_gpu(name, x, y, xl, yl):
    import torch

    import paper_2602_17206_amd as pkg
    from paper_2602_17206_amd import binding

    entry, _, _, _, _, gamma, mode, _, options = PROBLEMS[name]
    mode = {"unfused": pkg.UNFUSED, "fused": pkg.FUSED}[mode]
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    if entry == "half":
        t = getattr(torch, options["half_type"])
        value, desc, ws = pkg.sdtw_forward_half(xd.to(t), yd.to(t), gamma, mode)
        dx, dy, _ = pkg.sdtw_backward_half(desc, ws)
    elif entry == "ragged":
        xld, yld = torch.from_numpy(xl).cuda(), torch.from_numpy(yl).cuda()
        value, desc, ws = pkg.sdtw_forward_ragged(xd, yd, xld, yld, gamma, mode)
        dx, dy, _ = pkg.sdtw_backward_ragged(desc, xd, yd, xld, yld, ws)
    elif entry == "normalized":
        value, desc, ws = pkg.sdtw_normalized_forward(xd, yd, gamma, mode)
        dx, dy = pkg.sdtw_normalized_backward(desc, xd, yd, ws)
    else:
        value, desc, ws = pkg.sdtw_forward(xd, yd, gamma, mode, **options)
        dx, dy, _ = pkg.sdtw_backward(desc, xd, yd, ws)
    torch.cuda.synchronize()
    assert binding.workspace_status(ws) == 0
    return {k: v.cpu().numpy().astype(np.float64) for k, v in (("value", value), ("dx", dx), ("dy", dy))}


def errors(got, ref):
    """Relative 2-norm of the values' error; of the gradients' (the larger of dx and dy) over the whole batch; and the
    median over the batch of the gradients' per pair, which a pair with two nearly equal alignments does not move."""
    def rel(a, b):
        return float(np.linalg.norm(a - b) / np.linalg.norm(b))

    pairs = [max(rel(got[k][b], ref[k][b]) for k in ("dx", "dy")) for b in range(ref["value"].shape[0])]
    return rel(got["value"], ref["value"]), max(rel(got[k], ref[k]) for k in ("dx", "dy")), float(np.median(pairs))


# ------------------------------------------------------------------------------- models of the arithmetic, on the CPU
def exact_cost(x, y):
    x, y = x.astype(np.float64), y.astype(np.float64)
    return ((x[:, None] - y[None]) ** 2).sum(-1)


def perturbed_cost(draw, x, y):
    # seeded by the sequences, so that a draw does not depend on the order in which the pairs' threads run
    rng = np.random.default_rng([draw] + [int(a.view(np.uint32).sum(dtype=np.uint64)) for a in (x, y)])
    norms = (x.astype(np.float64) ** 2).sum(-1)[:, None] + (y.astype(np.float64) ** 2).sum(-1)[None]
    return np.maximum(exact_cost(x, y) + COST_ERROR * norms * rng.standard_normal(norms.shape), 0.0)


def alignment_64(d, gamma, bandwidth=None):
    r = oracle.from_cost(d, gamma, bandwidth=bandwidth)
    return r["value"], r["E"]


def sweep_24(d32, gamma):
    """Table of sums over alignments, m 2^-r: float32 mantissas, int64 scales (the cost's share kept apart)."""
    N, M = d32.shape
    t = d32 * np.float32(np.log2(np.e) / gamma)
    k = np.trunc(t)
    w, k = np.exp2(-(t - k)).astype(np.float32), k.astype(np.int64)
    mant = np.zeros((N + 1, M + 1), np.float32)
    scale = np.full((N + 1, M + 1), 1 << 40, np.int64)
    mant[0, 0], scale[0, 0] = 1, 0
    for s in range(2, N + M + 1):
        i = np.arange(max(1, s - M), min(N, s - 1) + 1)
        j = s - i
        near = [(i - 1, j - 1), (i, j - 1), (i - 1, j)]
        r = np.minimum.reduce([scale[a] for a in near])
        total = np.zeros(i.shape, np.float32)
        for a in near:
            total += np.ldexp(mant[a], np.maximum(r - scale[a], -200).astype(np.int32))
        mant[i, j], e = np.frexp(total * w[i - 1, j - 1])
        scale[i, j] = r + k[i - 1, j - 1] - e
    return mant[1:, 1:], scale[1:, 1:], w, k


def alignment_24(d, gamma, bandwidth=None):
    d32 = d.astype(np.float32)
    rm, rs, w, k = sweep_24(d32, gamma)
    tm, ts = (a[::-1, ::-1] for a in sweep_24(np.ascontiguousarray(d32[::-1, ::-1]), gamma)[:2])
    qm = tm / w  # the reverse table without the cell's own cost
    shift = np.clip(rs[-1, -1] - rs - (ts - k), -300, 300).astype(np.int32)
    E = np.ldexp(rm * (qm / rm[-1, -1]), shift)
    return (rs[-1, -1] - np.log2(float(rm[-1, -1]))) * gamma * np.log(2), E.astype(np.float64)


def model(name, x, y, xl, yl, alignment, cost):
    """The problem's results from ``alignment(cost(x_b, y_b), gamma)`` and gradients in float64."""
    entry, B, gamma, options = PROBLEMS[name][0], PROBLEMS[name][1], PROBLEMS[name][5], PROBLEMS[name][8]

    def one(a, b):
        value, E = alignment(cost(a, b), gamma, bandwidth=options.get("bandwidth"))
        a, b = a.astype(np.float64), b.astype(np.float64)
        return value, 2 * (E.sum(1)[:, None] * a - E @ b), 2 * (E.sum(0)[:, None] * b - E.T @ a)

    def pair(b):
        a, c = (x if x.ndim == 2 else x[b]), y[b]
        if xl is not None:
            a, c = a[:xl[b]], c[:yl[b]]
        value, dx, dy = one(a, c)
        if entry == "normalized":
            (vx, gx, hx), (vy, gy, hy) = one(a, a), one(c, c)
            value, dx, dy = value - 0.5 * (vx + vy), dx - 0.5 * (gx + hx), dy - 0.5 * (gy + hy)
        return value, dx, dy

    with ThreadPoolExecutor(4) as pool:
        results = list(pool.map(pair, range(B)))
    out = {"value": np.array([r[0] for r in results])}
    for n, key, like in ((1, "dx", x), (2, "dy", y)):
        out[key] = np.zeros((B,) + like.shape[-2:])
        for b, r in enumerate(results):
            out[key][b, :r[n].shape[0]] = r[n]
    return {k: v.astype(np.float32).astype(np.float64) for k, v in out.items()}


def assert_within(name, got, ref):
    for what, err, bar in zip(("value", "gradients", "gradients of the median pair"), errors(got, ref), bars(name)):
        assert err <= bar, "%s, %s: relative error %.2e, bar %.2e" % (name, what, err, bar)


@pytest.mark.gpu
@pytest.mark.parametrize("name", PROBLEMS)
def test_precision(name):
    print("precision", name, flush=True)
    args = inputs(name)
    assert_within(name, run_gpu(name, *args), reference(name, *args))


@pytest.mark.parametrize("name", PROBLEMS)
def test_bars_leave_room_for_float32_costs(name):
    args = inputs(name)
    got = model(name, *args, alignment_64, lambda x, y: perturbed_cost(4, x, y))  # draws 0 to 3 are in MEASURED
    assert_within(name, got, reference(name, *args))


@pytest.mark.parametrize("name", ["l256_unfused", "bfloat16"])
def test_a_24_bit_table_entry_misses_the_bar(name):
    """The mistake is planted in a model of the recurrence, with exact costs: gradients of the median pair."""
    args = inputs(name)
    err = errors(model(name, *args, alignment_24, exact_cost), reference(name, *args))[2]
    assert err > bars(name)[2], "%s: %.2e" % (name, err)

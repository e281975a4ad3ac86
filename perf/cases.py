"""The work that a user of this library has it do, as cases that can be timed.

Every case goes through the public entry points of the Python binding, the way a training loop, a scoring
service or a barycenter loop calls them: descriptors' sizes stay the same from call to call, so the
workspace, the output buffers and the optimiser state are made once and kept.

``entry`` of a case:
  grad          sdtw_forward + sdtw_backward: a loss and its gradients, one training step
  score         sdtw_forward with value_only: distances alone
  score_static  sdtw_forward_static_scratch: distances of small batches without a workspace of the caller's
  ragged        sdtw_forward_ragged + sdtw_backward_ragged: a padded batch with one length per sequence
  half          sdtw_forward_half + sdtw_backward_half: float16 / bfloat16 sequences
  normalized    sdtw_normalized_forward + sdtw_normalized_backward
  barycenter    sdtw_barycenter_step: one Adam step of an averaging loop
"""
import ctypes
import math

import torch

from paper_2602_17206_amd import binding as sdtw
from paper_2602_17206_amd.workloads import barycenter_workload

MODES = {"unfused": sdtw.UNFUSED, "fused": sdtw.FUSED}
HALF_TYPES = {"f16": torch.float16, "bf16": torch.bfloat16}
WALK_STEP = 0.1  # standard deviation of a random walk's step


def _case(entry, B, N, M, D, gamma, mode="fused", data="normal", **more):
    c = {"entry": entry, "B": B, "N": N, "M": M, "D": D, "gamma": gamma, "mode": mode, "data": data, "bandwidth": 0,
         "min_memory": False, "half_type": ""}
    c.update(more)
    return c


def listed():
    return [
        # a handful of short, narrow sequences: a unit-sized training step, where latency and launches count
        dict(_case("grad", 4, 64, 64, 8, 1.0, "unfused"), name="grad_tiny_unfused"),
        # nearest-neighbour classification: one query against the references of a class, inside a serving loop
        dict(_case("score_static", 64, 128, 128, 32, 1.0), name="score_query_vs_refs"),
        # the ordinary training step: B = 32 embedding sequences of length 256
        dict(_case("grad", 32, 256, 256, 128, 0.1), name="grad_b32_l256"),
        # the same for mixed-precision training, on longer clips
        dict(_case("half", 32, 512, 512, 128, 1.0, half_type="f16"), name="half_b32_l512"),
        # smooth trajectories of length 1024
        dict(_case("grad", 32, 1024, 1024, 128, 0.1, data="walk"), name="grad_b32_l1024_walk"),
        # speech frames (13 coefficients and two derivatives): utterances of different lengths, padded
        dict(_case("ragged", 32, 1024, 1024, 39, 1.0), name="ragged_b32_l1024_d39"),
        # features wider than the split operand copies take
        dict(_case("grad", 16, 512, 512, 200, 1.0), name="grad_wide_d200"),
        # a large batch of unequal, odd lengths with the cost tensor stored
        dict(_case("grad", 100, 1100, 937, 50, 0.1, "unfused"), name="grad_b100_odd_unfused"),
        # a normalised loss (three terms) at the ordinary size
        dict(_case("normalized", 32, 256, 256, 128, 0.1), name="normalized_b32_l256"),
        # long recordings known to be roughly synchronous: a Sakoe-Chiba band
        dict(_case("grad", 16, 4096, 4096, 64, 0.1, bandwidth=128), name="grad_banded_l4096"),
        # averaging 64 sequences: one optimiser step
        dict(_case("barycenter", 64, 512, 512, 32, 1.0, data="warped"), name="barycenter_k64_l512"),
        # the largest: long sequences at small gamma
        dict(_case("grad", 32, 8192, 8192, 128, 0.01), name="grad_b32_l8192"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    entry = rng.choice(["grad"] * 6 + ["score"] * 2 + ["score_static", "ragged", "half", "normalized"] + ["barycenter"] * 2)
    mode = rng.choice(["fused", "unfused"])
    data = rng.choice(["normal", "walk"])
    D = _log_int(rng, 2, 128)
    gamma = float("%.2g" % math.exp(rng.uniform(math.log(0.05), math.log(2.0))))
    B = _log_int(rng, 1, 128)
    N = _log_int(rng, 16, 2048)
    M = max(8, min(2048, int(N * rng.uniform(0.6, 1.5))))
    cells = 1 << 27  # most cells of a batch
    more = {}
    if entry == "grad":
        kind = rng.random()
        if kind < 0.15:  # wide features
            D, cells = rng.randint(129, 256), 1 << 24
        elif kind < 0.35:  # long sequences, which are run with small gamma
            N = _log_int(rng, 2048, 8192)
            M = int(N * rng.uniform(0.8, 1.0))
            B, cells = _log_int(rng, 1, 32), 1 << 30
            D, data = rng.randint(32, 128), "normal"
            gamma, mode = float("%.2g" % rng.uniform(0.01, 0.05)), "fused"
        elif kind < 0.5:
            more["bandwidth"] = max(abs(N - M), int(max(N, M) * rng.uniform(0.03, 0.3)), 1)
        elif kind < 0.6:
            more["min_memory"] = True
    elif entry == "score_static":
        B, N, M = _log_int(rng, 1, 64), rng.randint(16, 200), rng.randint(16, 200)
    elif entry == "half":
        more["half_type"] = rng.choice(sorted(HALF_TYPES))
    elif entry == "normalized":
        cells = 1 << 25
        if rng.random() < 0.6:
            M = N
    elif entry == "barycenter":
        B, N, data = _log_int(rng, 4, 128), _log_int(rng, 32, 1024), "warped"
        M, D, cells = N, _log_int(rng, 2, 64), 1 << 26
        gamma = float("%.2g" % rng.uniform(0.3, 2.0))
    B = max(1, min(B, cells // (N * M)))
    return _case(entry, B, N, M, D, gamma, mode, data, **more)


def _sequences(gen, case, B, L):
    x = torch.randn((B, L, case["D"]), generator=gen, device="cuda", dtype=torch.float32)
    if case["data"] == "walk":
        x = torch.cumsum(WALK_STEP * x.double(), dim=1).float()
    return x


def prepare(case, seed):
    B, N, M, D, gamma, entry = (case[k] for k in ("B", "N", "M", "D", "gamma", "entry"))
    mode = MODES[case["mode"]]
    s = {"case": case, "gamma": gamma, "mode": mode}

    def empty(*shape):
        return torch.empty(shape, dtype=torch.float32, device="cuda")

    if entry == "barycenter":
        # an averaging loop under way: the moments are those of gradients of the size met in it
        w = barycenter_workload(K=B, L=N, D=D, seed=seed, gamma=gamma)
        gen = torch.Generator(device="cuda").manual_seed(seed)
        s["X"] = torch.from_numpy(w.X).cuda()
        s["z"] = torch.from_numpy(w.z0).cuda()
        s["m"] = torch.randn((N, D), generator=gen, device="cuda") * (0.1 * B)
        s["v"] = (torch.rand((N, D), generator=gen, device="cuda") + 0.5) * (0.01 * B) ** 2
        s["step"], s["lr"] = 10, w.lr
        bdesc = sdtw.make_bary_desc(B, N, M, D, gamma, mode, w.lr, 0.9, 0.999, 1e-8, 1)
        s["workspace"] = sdtw.Workspace(sdtw.sdtw_barycenter_workspace_bytes(bdesc))
        s["loss"], s["dz"] = empty(1), empty(N, D)
        return s

    gen = torch.Generator(device="cuda").manual_seed(seed)
    s["x"] = _sequences(gen, case, B, N)
    s["y"] = _sequences(gen, case, B, M)
    if entry == "score_static":
        s["x"] = s["x"][0].contiguous()  # one query
    s["value"] = empty(B)
    desc = sdtw.make_desc(B, N, M, D, gamma, mode, x_shared=entry == "score_static", bandwidth=case["bandwidth"],
                          flags=sdtw.FLAG_MIN_MEMORY if case["min_memory"] else 0)
    s["desc"] = desc
    if entry == "score_static":
        return s
    if entry == "score":
        desc.flags |= sdtw.FLAG_VALUE_ONLY
    else:
        # the gradient that arrives from the mean over the batch, with a weight per pair
        s["grad_value"] = (torch.rand(B, generator=gen, device="cuda") + 0.5) / B
        s["dx"], s["dy"] = empty(B, N, D), empty(B, M, D)
    if entry == "ragged":
        for name, full in (("x_len", N), ("y_len", M)):
            low = max(1, full // 4)
            s[name] = torch.randint(low, full + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)
    if entry == "half":
        s["x"], s["y"] = (s[k].to(HALF_TYPES[case["half_type"]]) for k in ("x", "y"))
        s["workspace"] = sdtw.Workspace(sdtw.load_library().sdtw_half_workspace_bytes(ctypes.byref(desc)))
    elif entry == "normalized":
        s["workspace"] = sdtw.Workspace(sdtw.sdtw_normalized_workspace_bytes(desc))
    else:
        s["workspace"] = sdtw.Workspace(sdtw.sdtw_workspace_bytes(desc))
    return s


def run(s):
    case, gamma, mode = s["case"], s["gamma"], s["mode"]
    entry, ws = case["entry"], s.get("workspace")
    if entry == "barycenter":
        s["step"] += 1
        sdtw.sdtw_barycenter_step(s["z"], s["X"], s["m"], s["v"], gamma, s["step"], lr=s["lr"], mode=mode, workspace=ws,
                                  loss=s["loss"], dz=s["dz"])
        return {k: s[k] for k in ("loss", "dz", "z", "m", "v")}
    x, y, value = s["x"], s["y"], s["value"]
    if entry == "score_static":
        rc = sdtw.sdtw_forward_static_scratch(s["desc"], x, y, value)
        if rc != sdtw.STATUS_OK:
            raise sdtw.SdtwError(rc, "sdtw_forward_static_scratch")
        return {"value": value}
    if entry == "score":
        sdtw.sdtw_forward(x, y, gamma, mode, workspace=ws, value=value, value_only=True)
        return {"value": value}
    g, dx, dy = s["grad_value"], s["dx"], s["dy"]
    if entry == "grad":
        _, desc, _ = sdtw.sdtw_forward(x, y, gamma, mode, workspace=ws, value=value, bandwidth=case["bandwidth"],
                                       min_memory=case["min_memory"])
        sdtw.sdtw_backward(desc, x, y, ws, grad_value=g, dx=dx, dy=dy)
    elif entry == "ragged":
        _, desc, _ = sdtw.sdtw_forward_ragged(x, y, s["x_len"], s["y_len"], gamma, mode, workspace=ws, value=value)
        sdtw.sdtw_backward_ragged(desc, x, y, s["x_len"], s["y_len"], ws, grad_value=g, dx=dx, dy=dy)
    elif entry == "half":
        _, desc, _ = sdtw.sdtw_forward_half(x, y, gamma, mode, workspace=ws, value=value)
        dx, dy, _ = sdtw.sdtw_backward_half(desc, ws, grad_value=g)
    else:
        _, desc, _ = sdtw.sdtw_normalized_forward(x, y, gamma, mode, workspace=ws, value=value)
        sdtw.sdtw_normalized_backward(desc, x, y, ws, grad_value=g, dx=dx, dy=dy)
    return {"value": value, "dx": dx, "dy": dy}


def work(case):
    """Every sequence read and every result written once; per cell the inner product of the cost (2 D operations), the
    soft-minimum of the forward recurrence and, with gradients, that of the reverse one (12 operations each: minimum,
    three differences, two exponentials, two sums, logarithm, scaling, two additions).  The contraction of the
    alignment matrix is not counted: where it is zero, which it mostly is, there is nothing to contract."""
    B, N, M, D, entry = (case[k] for k in ("B", "N", "M", "D", "entry"))
    cells = float(B) * N * M
    if case["bandwidth"] and case["bandwidth"] < max(N, M):
        w = case["bandwidth"]
        cells = float(B) * sum(max(0, min(M - 1, i + w) - max(0, i - w) + 1) for i in range(N))
    if entry == "ragged":  # lengths uniform in [1/4, 1] of the padded ones
        cells *= 0.625 ** 2
    if entry == "normalized":
        cells = float(B) * (N * M + N * N + M * M)
    elem = 2 if entry == "half" else 4
    if entry == "barycenter":
        return {"bytes": 4.0 * (B * M * D + 7 * N * D), "flops": cells * (2 * D + 24)}
    seq = float(1 if entry == "score_static" else B) * N * D + float(B) * M * D
    if entry in ("score", "score_static"):
        return {"bytes": 4.0 * (seq + B), "flops": cells * (2 * D + 12)}
    return {"bytes": elem * seq + 4.0 * (seq + 2 * B), "flops": cells * (2 * D + 24)}


def tolerance(case):
    """The cost of a cell in float32 is off by about eps (||x||^2 + ||y||^2), eps = 6e-8 (the rounding of its terms);
    over gamma that is the relative error of the weights of two alignments that differ in the cell, and so, where they
    compete, of a gradient; with random signs it adds up to a few times that over the cells in which they differ.
    Not less than 32-bit sums show (1e-5); at most 1e-4, since at small gamma few alignments compete."""
    norms = 2.0 * case["D"]
    if case["data"] == "walk":
        norms = case["D"] * WALK_STEP ** 2 * 0.5 * (case["N"] + case["M"])
    return {"rel": min(1e-4, max(1e-5, 3 * 6e-8 * norms / case["gamma"]))}

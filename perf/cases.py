"""The work that this library is measured on: cases over its public entry points.

`listed()` names the cases, `draw(rng)` gives more of the same ranges,
`prepare` makes what a program has in hand before the call (networks loaded,
images, the tuning table read), `run` makes one call and returns its results,
`work` is what the call cannot do without, and `exact` gives the float results
in double precision (integer results are exact by definition and have none).

Networks and images follow the seeded recipes of paper_1907_12933_amd/inputs.py;
the sizes are those of the benchmark and of the tests.
"""
import math
import os

import numpy as np
import torch

from paper_1907_12933_amd import ibmc, inputs

TUNE_TABLE = os.path.join(os.path.dirname(os.path.abspath(ibmc.__file__)), "tune_gfx950.json")
RECORD_BYTES = ibmc.CEX_DTYPE.itemsize
DEVICE_RECORDS, HOST_RECORDS = 1 << 26, 1 << 25

# the benchmark's delta sets and two of the tests' (pixels to 0 / 255; wide steps)
DELTAS = {
    "8": [-8, 8], "16": [-16, 16], "8_16": [-16, -8, 8, 16], "8_16_32": [-32, -16, -8, 8, 16, 32],
    "all16": list(range(-16, 17)), "255": [-255, 255], "20_60_120": [-120, -60, -20, 20, 60, 120],
}


def listed():
    return [
        # one small property of a small network, first level only: what a
        # caller pays for a call as such (set-up, launches, read-back)
        dict(name="check_tiny", kind="check", act="q8", dims="35-16-5", images=1, deltas="8", k=1),
        # the glyph benchmark: ten small properties of one small network in one call
        dict(name="check_glyphs", kind="check", act="q8", dims="35-16-5", images=10, deltas="all16", k=2),
        # one image of the benchmark network, checked by itself from host memory
        dict(name="check_blob", kind="check", act="q8", dims="784-256-256-10", images=1, deltas="8_16_32", k=2),
        # the benchmark step: 64 images and all their records in device memory
        dict(name="check_blobs", kind="check_dev", act="q8", dims="784-256-256-10", images=64, deltas="8_16_32", k=2),
        # many uneven properties over all eight networks of the batched benchmark
        dict(name="check_batch", kind="batch", act="q8", plan=3, per_net=32, budget=2e12),
        # the same with the float (sigmoid) networks, near ties reported
        dict(name="check_batch_f32", kind="batch", act="f32", plan=33, per_net=8, budget=2e11),
        # the L2 ball of the paper's smallest proximity around ten glyphs
        dict(name="check_ball", kind="ball", dims="35-16-5", images=10, gamma=0.3, k=2),
        # the search ordered by the proposal network, one image
        dict(name="check_ordered", kind="ordered", dims="784-256-256-10", deltas="8_16_32", k=2),
        # neuron-pair coverage of a large test set on a wide network, all four criteria
        dict(name="coverage_sweep", kind="coverage", dims="784-1024-1024-1024-10", pairs=65536),
        # tests generated for one criterion from one image
        dict(name="coverage_search", kind="search", dims="30-40-30-6", criterion="DS", deltas="20_60_120", k=2, tests=64),
        # plain forward pass of a set of images, all potentials returned
        dict(name="forward", kind="forward", act="q8", dims="784-1024-1024-1024-10", images=4096),
        # retraining a float network (one epoch of mini-batch Adam)
        dict(name="fit", kind="fit", dims="35-256-128-10", images=20000, batch=256, epochs=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# later-layer multiply-adds of one drawn call at most
_MACS = 2.4e13


def _fits(dims, points):
    macs = sum(dims[l] * dims[l + 1] for l in range(1, len(dims) - 1))
    return points * max(macs, 16000) <= _MACS


def _random_dims(rng, wide):
    pixels = rng.choice([20, 30, 35, 48, 64, 100, 196, 784, _log(rng, 16, 784)])
    hidden = [_log(rng, 10, wide) for _ in range(rng.choice([1, 2, 2]))]
    if rng.random() < 0.5:  # powers of two as often as ragged widths
        hidden = [1 << max(3, min(int(math.log2(wide)), h.bit_length() - 1)) for h in hidden]
    return [pixels] + hidden + [rng.choice([5, 6, 10, 10, rng.randint(2, 16)])]


def draw(rng):
    kind = rng.choice(["check", "check", "check", "check_dev", "check_dev", "check_dev", "batch", "batch", "ball",
                       "ordered", "coverage", "search", "forward", "fit"])
    while True:
        if kind in ("check", "check_dev"):
            act = rng.choice(["q8", "q8", "q8", "f32"]) if kind == "check" else "q8"
            dims = _random_dims(rng, 512 if act == "q8" else 128)
            deltas, k = rng.choice(sorted(DELTAS)), rng.choice([1, 2, 2, 3])
            images = rng.choice([1, 1, _log(rng, 2, 64)]) if kind == "check" else _log(rng, 2, 64)
            points = images * sum(inputs.point_count(dims[0], len(DELTAS[deltas]), j) for j in range(1, k + 1))
            if _fits(dims, points if act == "q8" else 8 * points) and points <= 1.5e9:
                return dict(kind=kind, act=act, dims="-".join(map(str, dims)), images=images, deltas=deltas, k=k)
        elif kind == "batch":
            act = rng.choice(["q8", "q8", "f32"])
            return dict(kind=kind, act=act, plan=rng.randint(100, 10**6), per_net=_log(rng, 2, 24) if act == "q8" else
                        _log(rng, 2, 8), budget=float("%.2g" % (math.exp(rng.uniform(math.log(1e10), math.log(4e11)))
                                                                 * (1.0 if act == "q8" else 0.25))))
        elif kind == "ball":
            dims = [rng.choice([16, 20, 25, 30, 35]), _log(rng, 8, 48), rng.randint(3, 10)]
            case = dict(kind=kind, dims="-".join(map(str, dims)), images=_log(rng, 1, 10),
                        gamma=round(rng.uniform(0.05, 0.3), 2), k=rng.choice([1, 2, 2]))
            return case
        elif kind == "ordered":
            side = rng.choice([8, 10, 14, 28])
            dims = [side * side, rng.choice([64, 100, 128, 256]), rng.choice([32, 64, 128, 256]), 10]
            return dict(kind=kind, dims="-".join(map(str, dims)), deltas=rng.choice(["8", "8_16", "8_16_32", "20_60_120"]),
                        k=rng.choice([1, 2, 2]))
        elif kind == "coverage":
            dims = [rng.choice([35, 100, 196, 784]), _log(rng, 16, 1024), _log(rng, 16, 1024), _log(rng, 16, 1024), 10]
            if rng.random() < 0.4:
                del dims[2]
            return dict(kind=kind, dims="-".join(map(str, dims)), pairs=_log(rng, 100, 65536))
        elif kind == "search":
            dims = [rng.randint(16, 48), rng.randint(12, 48), rng.randint(12, 40), rng.randint(4, 10)]
            return dict(kind=kind, dims="-".join(map(str, dims)), criterion=rng.choice(["SS", "DS", "SV", "DV"]),
                        deltas=rng.choice(["8_16_32", "20_60_120", "8_16"]), k=rng.choice([1, 2, 2]),
                        tests=rng.choice([8, 32, 64]))
        elif kind == "forward":
            dims = [rng.choice([35, 64, 100, 196, 784])] + [_log(rng, 16, 1024) for _ in range(rng.choice([1, 2, 3]))] + [10]
            act = rng.choice(["q8", "q8", "f32"])
            if act == "f32":
                dims = [min(d, 512) if l else d for l, d in enumerate(dims)]
            return dict(kind=kind, act=act, dims="-".join(map(str, dims)), images=_log(rng, 1, 4096))
        else:
            dims = [35, _log(rng, 16, 256)] + ([_log(rng, 16, 128)] if rng.random() < 0.6 else []) + [10]
            return dict(kind=kind, dims="-".join(map(str, dims)), images=_log(rng, 400, 20000),
                        batch=rng.choice([32, 64, 100, 256]), epochs=1)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

_CTX = None


def _context():
    """The context of this process, with the shipped kernel choices: a
    program makes one and keeps it."""
    global _CTX
    if _CTX is None:
        _CTX = ibmc.Context(0, torch.cuda.current_stream())
        ibmc.ibmc_tune_load(_CTX, TUNE_TABLE)
    return _CTX


def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _images(g, count, n):
    """Binary glyphs up to 100 pixels, blobs above (cut to n pixels where n is no square)."""
    if n <= 100:
        return inputs.glyph_images(g, count, 1, n)
    side = math.isqrt(n - 1) + 1
    return np.ascontiguousarray(inputs.blob_images(g, count, side)[:, :n])


def _qnet(g, dims):
    return inputs.random_qnet(g, dims, shift=7)


def _blobs_dev(seed, count, n):
    """Blob images as inputs.blob_images draws them, many at once on the GPU
    (n pixels of the smallest square that holds them), uint8 [count][n]."""
    t = torch.Generator(device="cuda").manual_seed(seed)
    u = lambda *s: torch.rand(*s, generator=t, device="cuda")  # noqa: E731
    side = math.isqrt(n - 1) + 1
    out = torch.empty(count, n, dtype=torch.uint8, device="cuda")
    at = torch.arange(side, device="cuda", dtype=torch.float32)
    for lo in range(0, count, 8192):
        c = min(8192, count - lo)
        lo_px = min(4.0, (side - 1) / 2.0)
        mid = lo_px + u(c, 3, 2) * (side - 1 - 2 * lo_px)
        sig, amp = 1.5 + 2.5 * u(c, 3), 128.0 + 127.0 * u(c, 3)
        amp = amp * (torch.arange(3, device="cuda") < 1 + (u(c, 1) * 3).long())
        f = lambda m: torch.exp(-((at - m[..., None]) ** 2) / (2.0 * sig[..., None] ** 2))  # noqa: E731
        ys, xs = f(mid[..., 0]) * amp[..., None], f(mid[..., 1])
        img = (ys[..., :, None] * xs[..., None, :]).sum(1).reshape(c, -1)[:, :n]
        noise = (u(c, n) * 2.0 - 1.0) * (20.0 * math.sqrt(3.0))
        out[lo:lo + c] = (img + noise).round().clamp(0, 255).to(torch.uint8)
    return out


def _pairs_dev(seed, count, n):
    """Image pairs of a coverage run: the second differs from the first in
    1-8 pixels by +-1..32, clamped."""
    x1 = _blobs_dev(seed, count, n)
    t = torch.Generator(device="cuda").manual_seed(seed + 1)
    x2 = torch.empty_like(x1)
    for lo in range(0, count, 8192):
        c = min(8192, count - lo)
        at = torch.rand(c, n, generator=t, device="cuda").topk(8, dim=1).indices
        step = torch.randint(1, 33, (c, 8), generator=t, device="cuda")
        step = step * (1 - 2 * torch.randint(0, 2, (c, 8), generator=t, device="cuda"))
        used = torch.arange(8, device="cuda") < torch.randint(1, 9, (c, 1), generator=t, device="cuda")
        a = x1[lo:lo + c].long()
        a.scatter_add_(1, at, step * used)
        x2[lo:lo + c] = a.clamp(0, 255).to(torch.uint8)
    return x1, x2


def _points(case):
    n, m = _dims(case)[0], len(DELTAS[case["deltas"]])
    return case.get("images", 1) * sum(inputs.point_count(n, m, j) for j in range(1, case["k"] + 1))


def _capacity(case):
    return min(_points(case), DEVICE_RECORDS if case["kind"] == "check_dev" else HOST_RECORDS)


def _batch_plan(case):
    """Networks and (network, deltas, k) of the batched workload of this plan number."""
    nets, props = inputs.batch_workload(seed=int(case["plan"]), per_net=int(case["per_net"]), mac_budget=float(case["budget"]))
    return [n.dims for n in nets], [(p.net_index, p.deltas, p.k) for p in props]


def _fit_inputs(case, seed):
    g = inputs.rng(seed)
    net = inputs.random_fnet(g, _dims(case))
    _, X, Y = inputs.labelled_glyphs(g, 10, case["images"], p_flip=0.03, proto_flip=0.15)
    order = np.stack([g.permutation(case["images"]) for _ in range(case["epochs"])]).astype(np.int64)
    return net, X, Y, order


def _forward_inputs(case, seed):
    g = inputs.rng(seed)
    net = _qnet(g, _dims(case))
    if case["act"] == "f32":
        net = inputs.fnet_from_qnet(net)
    return net, _blobs_dev(seed, case["images"], _dims(case)[0]).cpu().numpy()


def prepare(case, seed):
    ctx, kind = _context(), case["kind"]
    s = dict(case=case, ctx=ctx, kind=kind)
    g = inputs.rng(seed)
    if kind in ("check", "check_dev"):
        net = _qnet(g, _dims(case))
        if case["act"] == "f32":
            net = inputs.fnet_from_qnet(net)
        s["net"] = net = ibmc.Mlp(ctx, net)
        s["deltas"] = D = np.array(DELTAS[case["deltas"]], np.int16)
        x = _images(g, case["images"], _dims(case)[0])
        s["cap"] = _capacity(case)
        s["tie_cap"] = min(_points(case), 1 << 16) if case["act"] == "f32" else 0
        if kind == "check_dev":
            x = torch.from_numpy(x).cuda()
            s["records"] = torch.zeros(s["cap"] * RECORD_BYTES, dtype=torch.uint8, device="cuda")
        s["image"] = x[0]
        s["props"] = [(net, x[i], D, 1, case["k"]) for i in range(case["images"])]
    elif kind == "batch":
        dims, props = _batch_plan(case)
        nets = [_qnet(g, d) for d in dims]
        if case["act"] == "f32":
            nets = [inputs.fnet_from_qnet(q) for q in nets]
        nets = [ibmc.Mlp(ctx, q) for q in nets]
        s["props"] = [(nets[i], _images(g, 1, dims[i][0])[0], D, 1, k) for i, D, k in props]
        s["cap"], s["tie_cap"] = HOST_RECORDS, 1 << 16 if case["act"] == "f32" else 0
    elif kind == "ball":
        dims = _dims(case)
        net = ibmc.Mlp(ctx, _qnet(g, dims))
        r2 = int((case["gamma"] * 255) ** 2)
        s["props"] = [(net, x, r2, 1, case["k"]) for x in _images(g, case["images"], dims[0])]
        s["cap"] = min(HOST_RECORDS, int(work(case)["flops"] / _point_flops(dims)))
    elif kind == "ordered":
        dims = _dims(case)
        s["net"] = ibmc.Mlp(ctx, _qnet(g, dims))
        s["image"], s["side"] = _images(g, 1, dims[0])[0], math.isqrt(dims[0])
        s["deltas"] = np.array(DELTAS[case["deltas"]], np.int16)
        s["proposer"] = ibmc.Proposer(ctx, seed=seed)
        s["cap"] = _capacity(case)
    elif kind == "coverage":
        s["net"] = ibmc.Mlp(ctx, _qnet(g, _dims(case)))
        s["x1"], s["x2"] = _pairs_dev(seed, case["pairs"], _dims(case)[0])
    elif kind == "search":
        dims = _dims(case)
        s["net"] = ibmc.Mlp(ctx, inputs.random_qnet(g, dims, shift=[5, 4], wmax=40, bmax=300))
        s["image"] = g.integers(0, 255, size=dims[0], endpoint=True).astype(np.uint8)
        s["deltas"] = np.array(DELTAS[case["deltas"]], np.int16)
        s["records"], s["gains"] = np.zeros(case["tests"], ibmc.CEX_DTYPE), np.zeros(case["tests"], np.int64)
    elif kind == "forward":
        net, s["images"] = _forward_inputs(case, seed)
        s["net"] = ibmc.Mlp(ctx, net)
    elif kind == "fit":
        net, s["images"], s["labels"], s["order"] = _fit_inputs(case, seed)
        s["net"] = ibmc.Mlp(ctx, net)
    else:
        raise ValueError(kind)
    # the program's own record lists, allocated once
    if "cap" in s and "records" not in s:
        s["records"] = np.zeros(s["cap"], ibmc.CEX_DTYPE)
    if "tie_cap" in s:
        s["ties"] = np.zeros(s["tie_cap"], ibmc.CEX_DTYPE)
    if "props" in s:
        s["none"] = s["records"] * 0 if kind == "check_dev" else np.zeros(s["cap"], ibmc.CEX_DTYPE)
    return s


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------

def _verdicts(sums):
    """One row per property: clean label, first unsafe and largest safe k,
    totals, then points, counterexamples and ties per level (three levels' room)."""
    rows = []
    for q in sums:
        pad = [0] * (3 - len(q["levels"]))
        rows.append([q["clean_label"], q["first_unsafe_k"], q["safe_up_to_k"], q["points_total"], q["cex_total"],
                     q["near_ties_total"], *q["points"], *pad, *q["cex"], *pad, *q["ties"], *pad])
    return np.array(rows, np.int64)


def _kept(into, recs):
    """Copies records that a call returns into the program's own list (zeros
    after the last), whose length does not depend on how many there are."""
    into[:len(recs)] = recs
    return into.view(np.int32).reshape(len(into), RECORD_BYTES // 4)


def _all_records(state, status):
    """The records where the buffers held them all; a truncated list is any
    subset of them, and an empty one stands for it."""
    r = state["records"] if status == ibmc.IBMC_OK else state["none"]
    return r if isinstance(r, torch.Tensor) else r.view(np.int32).reshape(len(r), RECORD_BYTES // 4)


def run(state):
    s, case, ctx = state, state["case"], state["ctx"]
    kind = s["kind"]
    if kind == "check" and case["images"] == 1 and case["k"] == 1:
        q, recs, ties = ibmc.ibmc_check_property(ctx, s["net"], s["image"], s["deltas"], 1, 1, cex_capacity=s["cap"],
                                                 near_tie_capacity=s["tie_cap"])
        return dict(verdicts=_verdicts([q]), records=_kept(s["records"], recs), ties=_kept(s["ties"], ties))
    if kind in ("check", "batch"):
        sums, _, ties, status = ibmc.ibmc_check_batch(ctx, s["props"], cex_capacity=s["cap"], cex_buf=s["records"],
                                                      near_tie_capacity=s["tie_cap"])
        return dict(verdicts=_verdicts(sums), records=_all_records(s, status), ties=_kept(s["ties"], ties if status == ibmc.IBMC_OK else ties[:0]))
    if kind == "check_dev":
        sums, _, _, status = ibmc.ibmc_check_batch_dev(ctx, s["props"], cex_capacity=s["cap"], cex_buf=s["records"],
                                                       records_on_device=True)
        return dict(verdicts=_verdicts(sums), records=_all_records(s, status))
    if kind == "ball":
        sums, recs = ibmc.ibmc_check_ball_batch(ctx, s["props"], cex_capacity=s["cap"])
        return dict(verdicts=_verdicts(sums), records=_kept(s["records"], recs))
    if kind == "ordered":
        q, recs = ibmc.ibmc_check_property_ranked(ctx, s["net"], s["proposer"], s["image"], s["side"], s["side"], s["deltas"],
                                                  1, case["k"], cex_capacity=s["cap"])
        return dict(verdicts=_verdicts([q]), before_first=q["points_before_first"], records=_kept(s["records"], recs))
    if kind == "coverage":
        outs = ibmc.ibmc_coverage_all_dev(ctx, s["net"], s["x1"], s["x2"])
        return [dict(covered_pairs=o["covered_pairs"], covered_neurons=o["covered_neurons"], literal=o["literal"],
                     bits=o["bits"].view(np.int64)) for o in outs]
    if kind == "search":
        tests, gains, cov = ibmc.ibmc_coverage_search(ctx, s["net"], s["image"], s["deltas"], case["k"], case["criterion"],
                                                      max_tests=case["tests"])
        s["gains"][:len(gains)] = gains
        return dict(tests=_kept(s["records"], tests), gains=s["gains"], covered=cov["covered_pairs"],
                    bits=cov["bits"].view(np.int64))
    if kind == "forward":
        potentials, labels = ibmc.ibmc_forward(ctx, s["net"], s["images"])
        return dict(potentials=potentials, labels=labels)
    trained, losses = ibmc.ibmc_fit_mlp(ctx, s["net"], s["images"], s["labels"], epochs=case["epochs"], batch=case["batch"],
                                        lr=1e-3, order=s["order"])
    W, b = trained.params
    return dict(W=W, b=b, losses=losses)


# ---------------------------------------------------------------------------
# what a call cannot do without
# ---------------------------------------------------------------------------

def _later(dims):
    return sum(dims[l] * dims[l + 1] for l in range(1, len(dims) - 1))


def _point_flops(dims):
    """One point: its last pixel's first-layer update and the later layers."""
    return 2.0 * (dims[1] + _later(dims))


def _net_bytes(dims, size=1):
    return sum(dims[l + 1] * (dims[l] * size + 4) for l in range(len(dims) - 1))


def _ball_points(n, r2, k):
    """Points of levels 1..k <= 2 around a binary image: every pixel moves one way only."""
    rd = min(math.isqrt(r2), 255)
    one = n * rd
    two = sum(min(math.isqrt(r2 - a * a), 255) for a in range(1, rd + 1) if a * a <= r2)
    return one + (math.comb(n, 2) * two if k > 1 else 0)


def work(case):
    kind = case["kind"]
    if kind == "batch":
        dims, props = _batch_plan(case)
        flops = sum(_point_flops(dims[i]) * sum(inputs.point_count(dims[i][0], len(D), j) for j in range(1, k + 1))
                    for i, D, k in props)
        return dict(bytes=sum(_net_bytes(d, 1 if case["act"] == "q8" else 4) for d in dims) + sum(dims[i][0] for i, _, _ in props),
                    flops=flops)
    dims = _dims(case)
    if kind in ("check", "check_dev", "ordered"):
        size = 4 if case.get("act") == "f32" else 1
        return dict(bytes=_net_bytes(dims, size) + case.get("images", 1) * dims[0], flops=_points(case) * _point_flops(dims))
    if kind == "ball":
        pts = case["images"] * _ball_points(dims[0], int((case["gamma"] * 255) ** 2), case["k"])
        return dict(bytes=_net_bytes(dims) + case["images"] * dims[0], flops=pts * _point_flops(dims))
    if kind == "coverage":
        full = sum(dims[l] * dims[l + 1] for l in range(len(dims) - 1))
        pairs = sum(dims[l] * dims[l + 1] for l in range(1, len(dims) - 1))
        # both images' later layers, the first layer of one and about 4.5 changed pixels of the other
        return dict(bytes=2 * case["pairs"] * dims[0] + _net_bytes(dims) + pairs // 2,
                    flops=2.0 * case["pairs"] * (full + _later(dims) + 4.5 * dims[1]))
    if kind == "search":
        return dict(bytes=_net_bytes(dims) + dims[0], flops=_points(case) * 2.0 * (case["k"] * dims[1] + _later(dims)))
    if kind == "forward":
        full = sum(dims[l] * dims[l + 1] for l in range(len(dims) - 1))
        size = 4 if case["act"] == "f32" else 1
        return dict(bytes=case["images"] * (dims[0] + 4 * sum(dims[1:]) + 4) + _net_bytes(dims, size),
                    flops=2.0 * case["images"] * full)
    full = sum(dims[l] * dims[l + 1] for l in range(len(dims) - 1))
    steps = case["epochs"] * -(-case["images"] // case["batch"])
    # forward, weight gradient and the deltas of every layer but the first; weights and moments once a step
    return dict(bytes=case["epochs"] * case["images"] * (dims[0] + 4) + steps * 24 * full,
                flops=2.0 * case["epochs"] * case["images"] * (2 * full + _later(dims)))


# ---------------------------------------------------------------------------
# the float results in double precision
# ---------------------------------------------------------------------------

def _sigmoid(u):
    return 1.0 / (1.0 + np.exp(-u))


def _exact_forward(net, X):
    a, pots = X.astype(np.float64) / 256.0, []
    for l, (W, b) in enumerate(zip(net.W, net.b)):
        u = a @ W.astype(np.float64).T + b.astype(np.float64)
        pots.append(u)
        a = _sigmoid(u)
    return np.concatenate(pots, 1)


def _exact_fit(case, seed):
    net, X, Y, order = _fit_inputs(case, seed)
    P = [p.astype(np.float64) for pair in zip(net.W, net.b) for p in pair]
    M, V = [np.zeros_like(p) for p in P], [np.zeros_like(p) for p in P]
    t, losses, L = 0, [], len(net.W)
    for at in order:
        total = 0.0
        for lo in range(0, len(at), case["batch"]):
            idx = at[lo:lo + case["batch"]]
            acts = [X[idx].astype(np.float64) / 256.0]
            for l in range(L):
                u = acts[-1] @ P[2 * l].T + P[2 * l + 1]
                acts.append(_sigmoid(u) if l < L - 1 else u)
            z = acts[-1] - acts[-1].max(1, keepdims=True)
            logp = z - np.log(np.exp(z).sum(1, keepdims=True))
            rows = np.arange(len(idx))
            total -= logp[rows, Y[idx]].sum()
            d = np.exp(logp)
            d[rows, Y[idx]] -= 1.0
            d /= len(idx)
            G = [None] * (2 * L)
            for l in range(L - 1, -1, -1):
                G[2 * l], G[2 * l + 1] = d.T @ acts[l], d.sum(0)
                if l:
                    d = (d @ P[2 * l]) * acts[l] * (1.0 - acts[l])
            t += 1
            # the options as the library holds them: float32 values
            lr, b1, b2, eps = (float(np.float32(v)) for v in (1e-3, 0.9, 0.999, 1e-8))
            for i, gr in enumerate(G):
                M[i] = b1 * M[i] + (1 - b1) * gr
                V[i] = b2 * V[i] + (1 - b2) * gr * gr
                P[i] = P[i] - lr * (M[i] / (1 - b1 ** t)) / (np.sqrt(V[i] / (1 - b2 ** t)) + eps)
        losses.append(total / len(at))
    return dict(W=P[0::2], b=P[1::2], losses=np.array(losses))


def exact(case, seed):
    if case["kind"] == "fit":
        return _exact_fit(case, seed)
    if case["kind"] == "forward" and case["act"] == "f32":
        net, X = _forward_inputs(case, seed)
        return dict(potentials=_exact_forward(net, X), labels=None)
    return None

"""The calls whose speed matters to a user of this framework, over the range they are made in.

A case is a dict of plain values.  ``listed()`` names twelve of them, ``draw(rng)`` gives more of the
same ranges.  Inputs are the framework's usual synthetic stand-in for video-latent attention (tokens on a
T x Y x X grid, Q and K sharing one positional projection per head, similar requests 0.3 noise apart),
drawn on the GPU from the seed alone.  Masks that a call only reads are cut here with plain torch from
the same rule the mask builder follows, so the inputs of such a call do not depend on the framework.

Fields: ``kind`` (which call), ``T, Y, X`` (grid, S = T Y X tokens), ``H`` heads of 128, ``B`` requests,
``dtype`` (bf16, f16, or fp8: e4m3 codes with block scales), ``density`` (share of the kv blocks that a
mask keeps: top_p is set for it, with a floor of a quarter of it), ``kv_block`` (64 or 128), ``shared``
(one mask, of request 0, for all requests), ``first`` (tokens of an enhanced first frame, 0: none), ``lse``.
"""

from __future__ import annotations

import math

import torch

from paper_2606_25040_amd import ops

D = 128
BLOCK = 64
BETA = 1.3            # first-frame key enhancement
SM = 1.0 / math.sqrt(D)


def _case(kind, grid, H, B=1, dtype="bf16", density=0.15, kv_block=64, shared=False, first=0, lse=False, **name):
    T, Y, X = grid
    return dict(name, kind=kind, T=T, Y=Y, X=X, H=H, B=B, dtype=dtype, density=density, kv_block=kv_block,
                shared=shared, first=first, lse=lse)


def listed():
    return [
        # the smallest call: one attention over 4,096 tokens of two heads with a fixed mask (latency)
        _case("attend", (4, 32, 32), 2, dtype="f16", density=0.25, name="tiny_f16"),
        # a short clip in one go: build the mask, plan, attend (launches and host time count)
        _case("step", (3, 30, 52), 12, density=0.25, name="short_clip_step_bf16"),
        # one layer's attention, 720p 5B, 20 % mask of the request itself
        _case("attend", (31, 22, 40), 24, density=0.20, name="wan5b_720p_bf16"),
        # the benchmark's: four 480p 14B requests under one cached mask
        _case("attend", (21, 30, 52), 40, B=4, shared=True, name="wan14b_480p_batch4_bf16"),
        # two requests with a mask each, f16, kv blocks of 128, enhanced first frame, ragged length
        _case("attend", (9, 33, 59), 16, B=2, dtype="f16", density=0.20, kv_block=128, first=33 * 59, lse=True,
              name="clip_f16_kv128_first_frame"),
        # one layer's attention on fp8 codes, 720p 14B, 10 % mask
        _case("attend", (21, 45, 80), 40, dtype="fp8", density=0.10, name="wan14b_720p_fp8"),
        # a middle-sized fp8 layer in one go: quantise, build from the block sums, plan, attend
        _case("step", (13, 30, 52), 24, dtype="fp8", density=0.12, kv_block=128, first=30 * 52,
              name="clip_step_fp8_kv128"),
        # mask acquisition of a 480p 14B layer from bf16 Q and K
        _case("build", (21, 30, 52), 40, name="wan14b_480p_build_bf16"),
        # what precedes the attention of a 720p 14B fp8 layer: quantise Q, K, V; build; plan
        _case("build", (21, 45, 80), 40, dtype="fp8", density=0.10, name="wan14b_720p_route_fp8"),
        # a historical request's dense pass (no mask yet), whose LSE the block masses need
        _case("dense", (21, 30, 52), 40, lse=True, name="wan14b_480p_dense_bf16"),
        # the historical request's true block masses
        _case("mass", (21, 30, 52), 40, name="wan14b_480p_mass_bf16"),
        # a mask cached from block masses: cut, plan, coverage on a new request, visit map and refresh
        _case("cache", (21, 30, 52), 40, name="wan14b_480p_cache"),
    ]


def draw(rng):
    kind = rng.choice(["attend"] * 5 + ["step", "step", "dense", "build", "build", "mass", "cache"])
    S = math.exp(rng.uniform(math.log(900), math.log(60000)))
    T = rng.randint(1, 24)
    side = math.sqrt(max(S / T, 16.0))
    Y = max(3, round(side * rng.uniform(0.6, 0.95)))
    X = max(3, round(S / (T * Y)))
    S = T * Y * X
    H = rng.choice([1, 2, 3, 5, 8, 12, 16, 24, 40])
    B = rng.choice([1, 1, 1, 2, 3, 4])
    dtype = rng.choice(["bf16", "bf16", "f16", "fp8", "fp8"])
    if kind in ("mass", "cache") and dtype == "fp8":
        dtype = "bf16"
    density = round(rng.uniform(0.08, 0.4), 3)
    c = _case(kind, (T, Y, X), H, B, dtype, density, rng.choice([64, 64, 128]), rng.random() < 0.4,
              rng.choice([0, 0, Y * X]), rng.random() < 0.3 or kind == "dense")
    while work(c)["flops"] > 1.2e13 or c["B"] * c["H"] * _blocks(S) ** 2 * 64 > 4e9:
        if c["B"] > 1:
            c["B"] -= 1
        elif c["H"] > 1:
            c["H"] = c["H"] * 2 // 3
        else:
            break
    return c


def _blocks(S, block=BLOCK):
    return -(-S // block)


def _tokens(case):
    return case["T"] * case["Y"] * case["X"]


def work(case):
    """Each input read once, each output written once; two products per kept block pair (block masses: one)."""
    S, H, B = _tokens(case), case["H"], case["B"]
    n, nk = _blocks(S), _blocks(S, case["kv_block"])
    Bm = 1 if case["shared"] else B
    rows = Bm * H * n
    el, elem = B * S * H * D, 1 if case["dtype"] == "fp8" else 2
    mask = 4 * (rows * nk * case["density"] + rows + 1)
    attend = {"bytes": 3 * el * elem + 2 * el + mask, "flops": 4.0 * B * H * S * S * D * case["density"]}
    # the builder: Q and K of the mask's requests, the block scores, the mask
    build = {"bytes": 2 * 2 * Bm * S * H * D + mask + 4 * B * H, "flops": 2.0 * rows * nk * D + 2.0 * Bm * S * H * D}
    if case["dtype"] == "fp8":   # quantising reads two bytes and writes one per element; the builder then reads block sums
        build["bytes"] = 3 * 3 * el + 2 * 8 * B * H * n * D + mask + 4 * B * H
    kind = case["kind"]
    if kind == "attend":
        w = attend
    elif kind == "dense":
        w = {"bytes": 3 * el * elem + 2 * el, "flops": 4.0 * B * H * S * S * D}
    elif kind == "build":
        w = build
    elif kind == "step":
        w = {"bytes": attend["bytes"] + build["bytes"], "flops": attend["flops"] + build["flops"]}
    elif kind == "mass":
        w = {"bytes": 2 * el * 2 + 4 * B * H * S + 4 * B * H * n * nk, "flops": 2.0 * B * H * S * S * D}
    else:   # cache: masses read by the cut, kept ones by the coverage; the refreshed mask keeps what was not visited
        kept = rows * nk * case["density"]
        w = {"bytes": 4 * rows * nk + 4 * kept * 3 + 4 * (rows * nk - kept), "flops": 2.0 * rows * nk}
    if case["lse"] and kind in ("attend", "dense", "step"):
        w["bytes"] += 4 * B * H * S
    return {"bytes": int(w["bytes"]), "flops": int(w["flops"])}


def tolerance(case):
    kind, dtype = case["kind"], case["dtype"]
    if kind == "build":
        return "exact"                       # codes, scales, exact block sums, mask
    if kind == "cache":
        return {"rel": 1e-9, "max": 1e-8}    # masks and maps are whole numbers; coverage is float64
    if kind == "mass":
        return {"rel": 4e-6, "max": 1e-4}    # fp32 logits and exponentials
    if dtype == "fp8":
        return {"rel": 0.03, "max": 0.9}     # probabilities are rounded to e4m3
    return {"rel": 1e-2, "max": 0.2} if dtype == "bf16" else {"rel": 1.2e-3, "max": 0.04}


# --------------------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------------------

def _features(case):
    """[S, 16] position features of the grid."""
    T, Y, X = case["T"], case["Y"], case["X"]
    i = torch.arange(T * Y * X, device="cuda", dtype=torch.float64)
    t, y, x = torch.floor(i / (Y * X)), torch.floor(i / X) % Y, i % X
    cols = []
    for c, P in ((t, 2 * T), (t, T), (y, 2 * Y), (y, Y), (y, Y / 2), (x, 2 * X), (x, X), (x, X / 2)):
        cols += [torch.sin(2 * math.pi * c / P), torch.cos(2 * math.pi * c / P)]
    return torch.stack(cols, 1).float()


def _inputs(case, seed):
    """(q, k, v), each [B, S, H, 128] 16-bit; requests after the draw of one base are 0.3 noise from it."""
    S, H, B = _tokens(case), case["H"], case["B"]
    g = torch.Generator("cuda").manual_seed(seed)
    dt = torch.float16 if case["dtype"] == "f16" else torch.bfloat16
    f = _features(case)
    gamma = 0.6 + 0.4 * torch.arange(H, device="cuda") / max(1, H - 1)
    w = torch.randn(16, H, D, device="cuda", generator=g) * (gamma / 4)[None, :, None]
    where = (f @ w.reshape(16, H * D)).reshape(S, H, D)
    base = [where + 0.5 * torch.randn(S, H, D, device="cuda", generator=g) for _ in range(2)]
    out = [torch.empty(B, S, H, D, dtype=dt, device="cuda") for _ in range(3)]
    for b in range(B):
        for t, x in zip(out, base):
            t[b] = x if B == 1 else x + 0.3 * torch.randn(S, H, D, device="cuda", generator=g)
        out[2][b] = torch.randn(S, H, D, device="cuda", generator=g)
    return out


def _quantised(x):
    """(codes, scales) of the framework's fp8 format: e4m3fn, one fp32 scale per (request, head, 64 tokens)."""
    B, S, H, _ = x.shape
    n = _blocks(S)
    codes = torch.empty(B, S, H, D, dtype=torch.uint8, device="cuda")
    scales = torch.empty(B, H, n, device="cuda")
    for b in range(B):
        y = torch.zeros(n * BLOCK, H, D, device="cuda")
        y[:S] = x[b]
        y = y.reshape(n, BLOCK, H, D)
        amax = y.abs().amax((1, 3))                                     # [n, H]
        c = (y * (448.0 / amax)[:, None, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn)
        codes[b] = c.view(torch.uint8).reshape(n * BLOCK, H, D)[:S]
        scales[b] = (amax / 448.0).t()
    return codes, scales


def _means(x, block, first):
    """[H, ceil(S / block), 128] float64 block means of one request [S, H, 128] (its first tokens times BETA)."""
    S, H, _ = x.shape
    n = _blocks(S, block)
    y = torch.zeros(n * block, H, D, dtype=torch.float64, device="cuda")
    y[:S] = x
    y[:first] *= float(torch.tensor(BETA, dtype=torch.float32))
    cnt = torch.full((n,), float(block), dtype=torch.float64, device="cuda")
    cnt[-1] = S - (n - 1) * block
    return (y.reshape(n, block, H, D).sum(1) / cnt[:, None, None]).permute(1, 0, 2).contiguous()


def _scores(case, q, k):
    """[Bm * H * n, nk] float64 block scores of the requests the mask is built from."""
    rows = []
    for b in range(1 if case["shared"] else case["B"]):
        qm, km = _means(q[b], BLOCK, 0), _means(k[b], case["kv_block"], case["first"])
        rows.append(torch.cat([(qm[h] @ km[h].t())[None] for h in range(case["H"])]) * SM)
    s = torch.cat(rows)
    return s.reshape(-1, s.shape[-1])


def _cut(rank, share, density, top_p=None):
    """(keep [rows, nk], top_p): the framework's top-p / top-k rule over rows ranked by `rank` with masses
    `share`; without a top_p, the one that gives the density is taken (to three digits)."""
    nk = rank.shape[1]
    order = torch.sort(rank, dim=1, descending=True, stable=True).indices
    mass = torch.cumsum(torch.gather(share, 1, order), 1)
    floor = max(1, math.ceil(density / 4 * nk - 1e-9))

    def counts(p):
        return ((mass < p).sum(1) + 1).clamp(floor, nk)

    if top_p is None:
        lo, hi = 0.0, 1.0
        for _ in range(11):
            top_p = (lo + hi) / 2
            if float(counts(top_p).double().mean()) / nk < density:
                lo = top_p
            else:
                hi = top_p
    kept = torch.arange(nk, device="cuda")[None, :] < counts(top_p)[:, None]
    return torch.zeros_like(kept).scatter_(1, order, kept), top_p


def _keep(case, q, k):
    s = _scores(case, q, k)
    return _cut(s, torch.softmax(s, 1), case["density"])


def _csr(case, keep):
    ptr = torch.zeros(keep.shape[0] + 1, dtype=torch.int32, device="cuda")
    ptr[1:] = torch.cumsum(keep.sum(1), 0)
    return ops.BlockMask(ptr, keep.nonzero()[:, 1].to(torch.int32), 1 if case["shared"] else case["B"], case["H"],
                         _blocks(_tokens(case)), case["kv_block"])


def _mask_buffers(case):
    """Empty buffers for a mask, as a serving loop keeps them."""
    S, H = _tokens(case), case["H"]
    Bm, n = 1 if case["shared"] else case["B"], _blocks(_tokens(case))
    rows = Bm * H * n
    return ops.BlockMask(torch.zeros(rows + 1, dtype=torch.int32, device="cuda"),
                         torch.zeros(rows * _blocks(S, case["kv_block"]), dtype=torch.int32, device="cuda"), Bm, H, n,
                         case["kv_block"])


def _first(case):
    return (case["first"], BETA) if case["first"] else None


def _masses(case, seed):
    """Row-normalised block masses [B, H, n, nk] (fp32) with the spread that pooled scores have."""
    q, k, _ = _inputs(case, seed)
    s = torch.softmax(_scores(dict(case, shared=False), q, k), 1).float()
    return s.reshape(case["B"], case["H"], _blocks(_tokens(case)), -1)


def prepare(case, seed):
    kind, S, B = case["kind"], _tokens(case), case["B"]
    state = {"case": case, "S": S, "first": _first(case)}
    if kind == "cache":
        # the masses of the historical requests and of new ones; the mask of the group's last layer
        case = dict(case, shared=False)
        state["case"] = case
        state["mass"], state["new_mass"] = _masses(case, seed), _masses(case, seed + 500)
        last = _masses(case, seed + 1000).reshape(-1, state["mass"].shape[-1]).double()
        state["last"] = _csr(case, _cut(last, last / last.sum(1, keepdim=True), case["density"])[0])
        m = state["mass"].reshape(-1, state["mass"].shape[-1]).double()
        state["top_p"] = _cut(m, m / m.sum(1, keepdim=True), case["density"])[1]
        state["mask"], state["refreshed"] = _mask_buffers(case), _mask_buffers(case)
        state["visits"] = ops.VisitMap(B, case["H"], _blocks(S), block=case["kv_block"])
        return state
    q, k, v = _inputs(case, seed)
    if kind in ("step", "build"):
        state["top_p"] = _keep(case, q, k)[1]
        state["mask"] = _mask_buffers(case)
        state["qkv"] = (q, k, v)
    elif kind == "mass":
        state["qkv"] = (q, k)
        state["lse"] = ops.block_sparse_attn_fwd(q, k, v, None, return_lse=True, key_scale=state["first"])[1]
    else:
        state["mask"] = state["plan"] = state["scales"] = None
        if kind == "attend":
            state["mask"] = _csr(case, _keep(case, q, k)[0])
            state["plan"] = ops.plan_block_mask(state["mask"], B, S)
        state["qkv"] = (q, k, v)
        if case["dtype"] == "fp8":
            codes = [_quantised(x) for x in (q, k, v)]
            state["qkv"], state["scales"] = tuple(c for c, _ in codes), tuple(s for _, s in codes)
    return state


# --------------------------------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------------------------------

def _build(state):
    """Mask and plan of a layer from its 16-bit Q and K; for an fp8 layer quantised on the way."""
    case, (q, k, v) = state["case"], state["qkv"]
    floor, kvb, mask = case["density"] / 4, case["kv_block"], state["mask"]
    if case["dtype"] != "fp8":
        Bm = mask.mask_batch
        mask = ops.build_block_mask(q[:Bm], k[:Bm], state["top_p"], floor, out=mask, key_scale=state["first"],
                                    kv_block=kvb)
        return mask, ops.plan_block_mask(mask, case["B"], state["S"]), None
    qc, qs, q_sums = ops.quantize_fp8_blockwise_sums(q)
    kc, ks, k_sums = ops.quantize_fp8_blockwise_sums(k, key_scale=state["first"])
    vc, vs = ops.quantize_fp8_blockwise(v)
    Bm = mask.mask_batch
    mask = ops.build_block_mask_from_sums(q_sums[:Bm], k_sums[:Bm], state["S"], state["top_p"], floor, out=mask,
                                          kv_block=kvb)
    return mask, ops.plan_block_mask(mask, case["B"], state["S"]), (qc, kc, vc, qs, ks, vs, q_sums, k_sums)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("attend", "dense"):
        return ops.block_sparse_attn_fwd(*state["qkv"], state["mask"], scales=state["scales"], schedule=state["plan"],
                                         return_lse=case["lse"], key_scale=state["first"])
    if kind == "build":
        mask, plan, quant = _build(state)
        return [mask.row_ptr, mask.col_idx, plan] + list(quant or ())
    if kind == "step":
        mask, plan, quant = _build(state)
        qkv, scales = (state["qkv"], None) if quant is None else (quant[:3], quant[3:6])
        out = ops.block_sparse_attn_fwd(*qkv, mask, scales=scales, schedule=plan, return_lse=case["lse"],
                                        key_scale=state["first"])
        return [mask.row_ptr, mask.col_idx, out]
    if kind == "mass":
        return ops.attn_block_mass(*state["qkv"], state["lse"], key_scale=state["first"], kv_block=case["kv_block"])
    mask = ops.select_block_mask(state["mass"], state["S"], state["top_p"], case["density"] / 4, out=state["mask"],
                                 kv_block=case["kv_block"])
    plan = ops.plan_block_mask(mask, case["B"], state["S"])
    coverage = ops.mask_coverage(mask, state["new_mass"], state["S"])
    visits = state["visits"]
    visits.reset(mask)
    visits.update(mask)
    refreshed = visits.refresh(state["last"], out=state["refreshed"])
    return [mask.row_ptr, mask.col_idx, plan, coverage, visits.bits, refreshed.row_ptr, refreshed.col_idx]


# --------------------------------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------------------------------

def _attention(case, q, k, v, keep):
    """(O [B, S, H, 128], lse [B, H, S]) in float64; keep [Bm, H, n, nk] or None (every block)."""
    B, S, H = case["B"], _tokens(case), case["H"]
    n, kvb = _blocks(S), case["kv_block"]
    out = torch.empty(B, S, H, D, dtype=torch.float64, device="cuda")
    lse = torch.empty(B, H, S, dtype=torch.float64, device="cuda")
    step = max(1, min(n, int(4e8) // (8 * BLOCK * S)))
    beta = float(torch.tensor(BETA, dtype=torch.float32))
    for b in range(B):
        for h in range(H):
            qh, kh, vh = (x(b, h) for x in (q, k, v))
            kh[:case["first"]] *= beta
            for i0 in range(0, n, step):
                t0, t1 = i0 * BLOCK, min(S, (i0 + step) * BLOCK)
                if keep is None:
                    kk, vv, no = kh, vh, None
                else:
                    rows = keep[b % keep.shape[0], h, i0:i0 + step]
                    used = rows.any(0).repeat_interleave(kvb)[:S].nonzero()[:, 0]
                    kk, vv = kh[used], vh[used]
                    no = ~rows[:, used // kvb].repeat_interleave(BLOCK, 0)[:t1 - t0]
                z = (qh[t0:t1] @ kk.t()).mul_(SM)
                if no is not None:
                    z.masked_fill_(no, -math.inf)
                m = z.amax(1, keepdim=True)
                z.sub_(m).exp_()
                l = z.sum(1, keepdim=True)
                out[b, t0:t1, h] = (z @ vv) / l
                lse[b, h, t0:t1] = (m + l.log())[:, 0]
    return out, lse


def _block_masses(case, q, k):
    """[B, H, n, nk] float64: mean over a q-block's queries of their probabilities summed over a kv block."""
    B, S, H, kvb = case["B"], _tokens(case), case["H"], case["kv_block"]
    n, nk = _blocks(S), _blocks(S, case["kv_block"])
    out = torch.empty(B, H, n, nk, dtype=torch.float64, device="cuda")
    step = max(1, min(n, int(4e8) // (8 * BLOCK * S)))
    beta = float(torch.tensor(BETA, dtype=torch.float32))
    for b in range(B):
        for h in range(H):
            qh, kh = q[b, :, h].double(), k[b, :, h].double()
            kh[:case["first"]] *= beta
            for i0 in range(0, n, step):
                t0, t1 = i0 * BLOCK, min(S, (i0 + step) * BLOCK)
                p = torch.softmax((qh[t0:t1] @ kh.t()).mul_(SM), 1)
                p = torch.nn.functional.pad(p, (0, nk * kvb - S)).reshape(t1 - t0, nk, kvb).sum(2)
                for i in range(i0, min(n, i0 + step)):
                    out[b, h, i] = p[(i - i0) * BLOCK:(i - i0 + 1) * BLOCK].mean(0)
    return out


def exact(case, seed):
    kind, S, H = case["kind"], _tokens(case), case["H"]
    if kind == "cache":
        case = dict(case, shared=False)
        mass, new = _masses(case, seed), _masses(case, seed + 500)
        m = mass.reshape(-1, mass.shape[-1]).double()
        keep = _cut(m, m / m.sum(1, keepdim=True), case["density"])[0].reshape(mass.shape)
        cnt = torch.full((mass.shape[2],), float(BLOCK), dtype=torch.float64, device="cuda")
        cnt[-1] = S - (mass.shape[2] - 1) * BLOCK
        coverage = ((new.double() * keep).sum(3) * cnt).sum(2) / S
        return [None, None, None, coverage, None, None, None]
    q, k, v = _inputs(case, seed)
    if kind == "mass":
        return _block_masses(case, q, k)
    if kind == "build":
        if case["dtype"] != "fp8":
            return None   # whole numbers only
        sums = []
        for x, first in ((q, 0), (k, case["first"])):
            n = _blocks(S)
            cnt = torch.full((n,), float(BLOCK), dtype=torch.float64, device="cuda")
            cnt[-1] = S - (n - 1) * BLOCK
            sums.append(torch.stack([_means(x[b], BLOCK, first) * cnt[None, :, None] for b in range(case["B"])]))
        scales = [_quantised(x)[1].double() for x in (q, k, v)]
        return [None] * 6 + scales + sums
    keep = None
    if kind != "dense":
        keep = _keep(case, q, k)[0].reshape(1 if case["shared"] else case["B"], H, _blocks(S), -1)
    if case["dtype"] == "fp8":
        codes = [_quantised(x) for x in (q, k, v)]
        read = [lambda b, h, c=c, s=s: (c[b, :, h].contiguous().view(torch.float8_e4m3fn).double()
                                        * s[b, h].double().repeat_interleave(BLOCK)[:S, None]) for c, s in codes]
    else:
        read = [lambda b, h, x=x: x[b, :, h].double() for x in (q, k, v)]
    out, lse = _attention(case, *read, keep)
    out = (out, lse) if case["lse"] else out
    return [None, None, out] if kind == "step" else out

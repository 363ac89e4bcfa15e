"""GPU parity: the HIP path (through the C ABI) against the CPU oracle.

Small cases compare every output; the full-size workloads compare sampled
rows and work items the oracle computes one by one.  Tolerances: masks
bit-exact apart from excused near-ties (tests/compare.py); outputs max-abs
2e-3 for f16/bf16 and 3e-2 for fp8; fp8 codes and scales bit-exact.
"""

import math

import numpy as np
import pytest
import torch

from oracle import attention as oa
from oracle import fp8 as of
from oracle import guidance as og
from oracle import mask as om
from paper_2606_25040_amd import ops
import workloads as wk
from tests.compare import compare_masks, max_abs_err

pytestmark = pytest.mark.gpu

TOL16 = 2e-3
TOL8 = 3e-2


@pytest.fixture(scope="module", autouse=True)
def device():
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    ops.load_library()
    torch.cuda.set_device(0)
    yield


def np64(t: torch.Tensor) -> np.ndarray:
    return t.float().cpu().numpy()


def rand_qkv(gen, B, S, H, dtype, scale=0.5):
    """Random Q, K (logit std ~ scale^2) and V ~ N(0, 1).  The default keeps
    attention diffuse like the workloads (|O| < 0.5), where the 16-bit output
    rounding stays inside the absolute tolerance; peaked cases use
    ``within_rounding`` instead."""
    q = (torch.randn(B, S, H, 128, generator=gen) * scale).to(dtype)
    k = (torch.randn(B, S, H, 128, generator=gen) * scale).to(dtype)
    v = torch.randn(B, S, H, 128, generator=gen).to(dtype)
    return q, k, v


def positional_qk(B, S, H, dtype, seed):
    """Block-structured Q/K (shared positional projection) for builder tests."""
    g = np.random.Generator(np.random.PCG64(seed))
    f = np.stack([np.sin(2 * np.pi * np.arange(S) / P) for P in (37.0, 200.0, 911.0, 3000.0)] +
                 [np.cos(2 * np.pi * np.arange(S) / P) for P in (37.0, 200.0, 911.0, 3000.0)], 1)
    q = np.empty((B, S, H, 128), np.float32)
    k = np.empty((B, S, H, 128), np.float32)
    for h in range(H):
        W = g.standard_normal((8, 128)) * 0.5
        for b in range(B):
            q[b, :, h] = f @ W + 0.5 * g.standard_normal((S, 128))
            k[b, :, h] = f @ W + 0.5 * g.standard_normal((S, 128))
    return torch.from_numpy(q).to(dtype), torch.from_numpy(k).to(dtype)


def within_rounding(got, ref, dtype, atol=TOL16, ref_abs=None):
    """Error bound for cases far from the workloads' diffuse regime: the
    absolute tolerance plus one unit of the 16-bit type's relative rounding
    on the output (|O|) and on the probabilities (sum_c p_c |v_c|, passed as
    ``ref_abs`` = attention applied to |V|)."""
    rel = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -10
    bound = atol + rel * np.abs(ref)
    if ref_abs is not None:
        bound = bound + rel * ref_abs
    return bool(np.all(np.abs(got - ref) <= bound))


# --------------------------------------------------------------------------- quantiser
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_quantizer_bit_exact(dtype):
    gen = torch.Generator().manual_seed(11)
    B, S, H = 2, 1000, 3
    x = torch.randn(B, S, H, 128, generator=gen) * torch.tensor([0.01, 1.0, 30.0]).view(1, 1, 3, 1)
    x[0, 64:128, 1] = 0.0                                  # amax == 0 block
    x[1, 128:192, 0] = -0.0
    x[1, 192:256, 2] *= 1e-3                               # values deep in the subnormal range
    x[0, 960:, 2] = 1e4 if dtype == torch.bfloat16 else 6e4
    if dtype == torch.bfloat16:
        # amax below 448 / FLT_MAX (the reciprocal is taken after a 2^64
        # pre-scale), with fp32-subnormal inputs and a subnormal scale
        x[1, 320:384, 1] *= 2.0 ** -123
    x = x.to(dtype)
    codes, scales = ops.quantize_fp8_blockwise(x.cuda())
    torch.cuda.synchronize()
    oc, os_ = of.quantize_blockwise(np64(x))
    assert np.array_equal(codes.cpu().numpy(), oc)
    assert np.array_equal(scales.cpu().numpy(), os_)


# --------------------------------------------------------------------------- builder
BUILD_CASES = [(0.5, 0.05), (0.9, 0.0), (0.0, 0.3), (1.0, 0.0), (0.3, 1.0), (0.75, 0.1)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_builder_small_all_rows(dtype):
    B, S, H = 2, 1000, 3                                    # 16 blocks, last one 40 tokens
    q, k = positional_qk(B, S, H, dtype, 5)
    qd, kd = q.cuda(), k.cuda()
    sm = 1.0 / math.sqrt(128)
    for top_p, mk in BUILD_CASES:
        m = ops.build_block_mask(qd, kd, top_p, mk, sm_scale=sm, return_scores=True)
        rp, ci = m.to_host()
        o = om.build_block_mask(np64(q), np64(k), sm, top_p, mk)
        rep = compare_masks(rp, ci, o, range(m.rows), top_p, mk)
        assert rep.ok, rep.failing[:5]
        assert ops.validate_block_mask(m) == 0
        s32 = m.block_scores.cpu().numpy()
        assert np.array_equal(s32, o.scores.astype(np.float32)) or \
            np.max(np.abs(s32 - o.scores) / (np.abs(o.scores) + 1e-30)) < 1.2e-7


def test_builder_single_block_and_tiny_sequences():
    sm = 1.0 / math.sqrt(128)
    for S in (1, 63, 64, 65, 130):
        q, k = positional_qk(1, S, 2, torch.bfloat16, S)
        m = ops.build_block_mask(q.cuda(), k.cuda(), 0.6, 0.0, sm_scale=sm)
        rp, ci = m.to_host()
        o = om.build_block_mask(np64(q), np64(k), sm, 0.6, 0.0)
        rep = compare_masks(rp, ci, o, range(m.rows), 0.6, 0.0)
        assert rep.ok, (S, rep.failing[:3])


@pytest.mark.parametrize("top_p,mk", [(0.5, 0.0), (0.3, 0.4), (0.0, 0.25), (0.97, 0.0)])
def test_builder_exact_ties(top_p, mk):
    """Bit-identical block scores: constant Q/K (every score of a row equal)
    and K whose blocks repeat with period 4 (four-way ties per row).  Equal
    scores are kept lowest index first."""
    sm = 1.0 / math.sqrt(128)
    S, H = 64 * 20, 2
    const = torch.full((1, S, H, 128), 0.25, dtype=torch.bfloat16)
    gen = torch.Generator().manual_seed(3)
    q = (torch.randn(1, S, H, 128, generator=gen) * 0.5).to(torch.bfloat16)
    base = (torch.randn(1, 4 * 64, H, 128, generator=gen) * 0.5).to(torch.bfloat16)
    k_rep = base.repeat(1, S // (4 * 64), 1, 1).contiguous()
    for qq, kk in ((const, const), (q, k_rep)):
        m = ops.build_block_mask(qq.cuda(), kk.cuda(), top_p, mk, sm_scale=sm)
        rp, ci = m.to_host()
        o = om.build_block_mask(np64(qq), np64(kk), sm, top_p, mk)
        rep = compare_masks(rp, ci, o, range(m.rows), top_p, mk)
        assert rep.ok, rep.failing[:3]
    # constant rows keep a prefix of indices: k = 10 of 20 in exact arithmetic
    # (the float64 running sum of ten 1/20 lands one ulp below 0.5, hence 11
    # is accepted too; the comparator above excuses that boundary)
    m = ops.build_block_mask(const.cuda(), const.cuda(), 0.5, 0.0, sm_scale=sm)
    rp, ci = m.to_host()
    for r in range(m.rows):
        row = ci[rp[r]:rp[r + 1]]
        assert len(row) in (10, 11) and np.array_equal(row, np.arange(len(row)))


@pytest.mark.parametrize("n_blocks", [511, 700, 1500, 2000])
def test_builder_row_lengths_every_selection_path(n_blocks):
    """Rows of 511, 700, 1500 and 2000 blocks (each register budget of the
    one-wave-per-row selection), every row against the oracle."""
    sm = 1.0 / math.sqrt(128)
    S = 64 * n_blocks - 13
    q, k = positional_qk(1, S, 1, torch.bfloat16, n_blocks)
    for top_p, mk in ((0.45, 0.02), (0.0, 0.07), (0.9, 0.0)):
        m = ops.build_block_mask(q.cuda(), k.cuda(), top_p, mk, sm_scale=sm)
        rp, ci = m.to_host()
        o = om.build_block_mask(np64(q), np64(k), sm, top_p, mk)
        rep = compare_masks(rp, ci, o, range(m.rows), top_p, mk)
        assert rep.ok, (n_blocks, top_p, mk, rep.failing[:3])


def test_builder_largest_supported_row():
    """n = 4096 blocks (the largest row): every row against the oracle."""
    sm = 1.0 / math.sqrt(128)
    S = 64 * 4096 - 7
    q, k = positional_qk(1, S, 1, torch.bfloat16, 21)
    for top_p, mk in ((0.4, 0.01), (0.0, 0.1)):
        m = ops.build_block_mask(q.cuda(), k.cuda(), top_p, mk, sm_scale=sm)
        rp, ci = m.to_host()
        o = om.build_block_mask(np64(q), np64(k), sm, top_p, mk)
        rep = compare_masks(rp, ci, o, range(m.rows), top_p, mk)
        assert rep.ok, rep.failing[:3]


# --------------------------------------------------------------------------- attention
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_attention_peaked_logits(dtype):
    gen = torch.Generator().manual_seed(77)
    B, S, H = 1, 700, 2
    q, k, v = rand_qkv(gen, B, S, H, dtype, scale=1.6)      # logit std ~ 2.6
    n = (S + 63) // 64
    rng = np.random.Generator(np.random.PCG64(77))
    rp, ci = wk.random_csr(rng, H * n, n, 0.5)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n)
    out = ops.block_sparse_attn_fwd(q.cuda(), k.cuda(), v.cuda(), mask)
    O, _ = oa.attention(np64(q), np64(k), np64(v), rp, ci, 1.0 / math.sqrt(128), 1)
    Oabs, _ = oa.attention(np64(q), np64(k), np.abs(np64(v)), rp, ci, 1.0 / math.sqrt(128), 1)
    assert within_rounding(np64(out), O, dtype, ref_abs=Oabs)


def attn_ref_full(q, k, v, rp, ci, mask_batch, sm):
    return oa.attention(np64(q), np64(k), np64(v), rp, ci, sm, mask_batch)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("S,B,H,mask_batch", [(64, 1, 1, 1), (100, 2, 2, 1), (1000, 2, 3, 2),
                                              (1000, 2, 3, 1), (2048, 1, 2, 1)])
def test_attention_small_full(dtype, S, B, H, mask_batch):
    gen = torch.Generator().manual_seed(S + 7 * B + H)
    q, k, v = rand_qkv(gen, B, S, H, dtype)
    n = (S + 63) // 64
    rng = np.random.Generator(np.random.PCG64(S))
    rp, ci = wk.random_csr(rng, mask_batch * H * n, n, 0.4, empty_frac=0.1 if n > 1 else 0.0)
    mask = ops.BlockMask.from_host(rp, ci, mask_batch, H, n)
    sm = 1.0 / math.sqrt(128)
    out, lse = ops.block_sparse_attn_fwd(q.cuda(), k.cuda(), v.cuda(), mask, sm_scale=sm,
                                         return_lse=True)
    torch.cuda.synchronize()
    O, L = attn_ref_full(q, k, v, rp, ci, mask_batch, sm)
    # few keys per row here, so |O| reaches ~0.7: allow the output rounding on top
    assert within_rounding(np64(out), O, dtype)
    lg = lse.cpu().numpy()
    fin = np.isfinite(L)
    assert np.array_equal(np.isfinite(lg), fin)
    if fin.any():
        assert np.max(np.abs(lg[fin] - L[fin])) <= 1e-3
    # empty rows are exactly zero
    counts = np.diff(rp)
    for b in range(B):
        for h in range(H):
            for i in range(n):
                r = oa.mask_row_index(b, h, i, H, n, mask_batch)
                if counts[r] == 0:
                    assert torch.all(out[b, i * 64:(i + 1) * 64, h] == 0)


def test_attention_full_density_equals_dense_sdpa():
    gen = torch.Generator().manual_seed(3)
    B, S, H = 1, 777, 2
    q, k, v = rand_qkv(gen, B, S, H, torch.bfloat16)
    n = (S + 63) // 64
    rp = np.arange(H * n + 1) * n
    ci = np.tile(np.arange(n), H * n)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n)
    out = ops.block_sparse_attn_fwd(q.cuda(), k.cuda(), v.cuda(), mask)
    ref = torch.nn.functional.scaled_dot_product_attention(
        q.double().permute(0, 2, 1, 3), k.double().permute(0, 2, 1, 3),
        v.double().permute(0, 2, 1, 3)).permute(0, 2, 1, 3)
    assert within_rounding(np64(out), ref.numpy(), torch.bfloat16)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "fp8"])
@pytest.mark.parametrize("key_scale", [None, (400, 1.5)])
def test_attention_without_mask_is_the_full_density_mask(dtype, key_scale):
    """mask = NULL (every kv block, the dense instantiations) gives bitwise the
    output of an explicit full-density mask, and that matches the oracle."""
    gen = torch.Generator().manual_seed(5)
    B, S, H = 2, 700, 2
    tdt = torch.float16 if dtype == "f16" else torch.bfloat16
    q, k, v = rand_qkv(gen, B, S, H, tdt)
    n = (S + 63) // 64
    rp = np.arange(H * n + 1) * n
    ci = np.tile(np.arange(n), H * n)
    full = ops.BlockMask.from_host(rp, ci, 1, H, n)
    if dtype == "fp8":
        cs = [ops.quantize_fp8_blockwise(x.cuda()) for x in (q, k, v)]
        args, kw = [c for c, _ in cs], {"scales": tuple(s_ for _, s_ in cs)}
        ins = [of.dequantize_blockwise(c.cpu().numpy(), s_.cpu().numpy()) for c, s_ in cs]
        tol = TOL8
    else:
        args, kw = [x.cuda() for x in (q, k, v)], {}
        ins = [np64(x) for x in (q, k, v)]
        tol = TOL16
    dense = ops.block_sparse_attn_fwd(*args, None, key_scale=key_scale, **kw)
    listed = ops.block_sparse_attn_fwd(*args, full, key_scale=key_scale, **kw)
    torch.cuda.synchronize()
    assert torch.equal(dense.view(torch.int16), listed.view(torch.int16))
    kk = ins[1] if key_scale is None else og.enhance_first_frame_keys(ins[1], *key_scale)
    O, _ = oa.attention(ins[0], kk, ins[2], rp, ci, 1.0 / math.sqrt(128), 1)
    assert within_rounding(np64(dense), O, tdt, atol=tol), float(np.max(np.abs(np64(dense) - O)))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,S,H", [(1, 1, 1), (1, 64, 3), (2, 129, 2), (1, 511, 8), (3, 193, 90), (2, 320, 64), (1, 850, 17),
                                   (16, 260, 64), (8, 383, 90), (8, 850, 40)])
def test_dense_kernel_variants_are_bitwise_the_full_mask(dtype, B, S, H):
    """The dense kernel runs with four or eight waves per workgroup by the
    amount of work, in pipelined and single steps by the number of full kv
    blocks: every variant, with sequence ends inside and at the edge of a
    workgroup's rows, gives the bits and the LSE of the masked kernel under an
    explicit full mask."""
    gen = torch.Generator(device="cuda").manual_seed(S)
    q, k, v = (torch.randn(B, S, H, 128, generator=gen, device="cuda").to(dtype) for _ in range(3))
    n = (S + 63) // 64
    # up to 14 kv blocks every masked walk starts at block 0, as the dense one does
    full = ops.BlockMask.from_host(np.arange(H * n + 1) * n, np.tile(np.arange(n), H * n), 1, H, n)
    for key_scale in (None, (min(S, 100), 1.5)):
        out, lse = ops.block_sparse_attn_fwd(q, k, v, None, return_lse=True, key_scale=key_scale)
        ref, ref_lse = ops.block_sparse_attn_fwd(q, k, v, full, return_lse=True, key_scale=key_scale)
        assert torch.equal(lse, ref_lse) and torch.equal(out.view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("kv_block", [64, 128])
@pytest.mark.parametrize("key_scale", [None, (700, 1.5)])
@pytest.mark.parametrize("H,S", [(16, 1000), (17, 960), (32, 1000), (33, 960), (40, 970)])
def test_attention_in_list_parts_matches_oracle(dtype, kv_block, key_scale, H, S):
    """Launches whose rows split into four, two or no parts: rows
    shorter than the number of parts, empty rows, ids outside [0, n_kv) and a
    missing second half at the end, first and last head against the oracle."""
    gen = torch.Generator().manual_seed(H)
    q, k, v = rand_qkv(gen, 1, S, H, dtype)
    n, nk = (S + 63) // 64, (S + kv_block - 1) // kv_block
    rng = np.random.Generator(np.random.PCG64(H + S))
    rp, ci = wk.random_csr(rng, H * n, nk, 0.4, empty_frac=0.15)
    rows = [np.concatenate([[-1], ci[rp[r]:rp[r + 1]], [nk]]) if r % 4 == 3 else ci[rp[r]:rp[r + 1]]
            for r in range(H * n)]
    mask = ops.BlockMask.from_host(np.concatenate([[0], np.cumsum([len(x) for x in rows])]), np.concatenate(rows), 1, H,
                                   n, block=kv_block)
    out, lse = ops.block_sparse_attn_fwd(q.cuda(), k.cuda(), v.cuda(), mask, return_lse=True, key_scale=key_scale)
    for h in (0, H - 1):
        kk = np64(k[:, :, h:h + 1])
        kk = kk if key_scale is None else og.enhance_first_frame_keys(kk, *key_scale)
        a, b = rp[h * n], rp[(h + 1) * n]
        O, L = oa.attention(np64(q[:, :, h:h + 1]), kk, np64(v[:, :, h:h + 1]), rp[h * n:(h + 1) * n + 1] - a, ci[a:b],
                            1.0 / math.sqrt(128), 1, kv_block=kv_block)
        assert within_rounding(np64(out[:, :, h:h + 1]), O, dtype, atol=TOL16)
        got = lse[:, h:h + 1].cpu().numpy()
        assert np.array_equal(np.isfinite(got), np.isfinite(L))
        fin = np.isfinite(L)
        assert np.max(np.abs(got[fin] - L[fin])) <= 1e-3


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("kv_block", [64, 128])
@pytest.mark.parametrize("key_scale", [None, (200, 1.25)])
@pytest.mark.parametrize("B,H,S,mask_batch", [(3, 30, 443, 3), (3, 30, 960, 1), (2, 40, 1025, 2), (1, 16, 2049, 1)])
def test_unsplit_rows_at_the_edges(dtype, kv_block, key_scale, B, H, S, mask_batch):
    """More than 64 rows on the fullest XCD, so no list is split (the kernel of
    every large call): odd numbers of q-blocks (a missing second half with kv
    blocks of 128), a mask per request or one for all, slices of one packed QKV
    tensor, row maxima that rise by 2^40 along the sequence, empty rows, ids
    outside [0, n_kv).  First, middle and last (request, head) against the
    oracle; P rounds to the type, so the bound carries one rounding of
    sum(p |v|)."""
    n, nk = (S + 63) // 64, -(-S // kv_block)
    assert -(-B * H // 8) * n > 64
    gen = torch.Generator(device="cuda").manual_seed(S + kv_block)
    qkv = torch.randn(B, S, 3, H, 128, generator=gen, device="cuda") * 0.5
    qkv[:, :, 0, :, 0] = 4.0
    qkv[:, :, 1, :, 0] += (80 * torch.arange(S, device="cuda") / S)[None, :, None]
    qkv = qkv.to(dtype)
    q, k, v = qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2]
    rng = np.random.Generator(np.random.PCG64(S))
    rp, ci = wk.random_csr(rng, mask_batch * H * n, nk, 0.5, empty_frac=0.1)
    rows = [ci[rp[r]:rp[r + 1]] for r in range(mask_batch * H * n)]
    rows2 = [np.concatenate([[-1], x, [nk, nk + 5]]) if r % 4 == 3 else x for r, x in enumerate(rows)]
    mask = ops.BlockMask.from_host(np.concatenate([[0], np.cumsum([len(x) for x in rows2])]), np.concatenate(rows2),
                                   mask_batch, H, n, block=kv_block)
    out, lse = ops.block_sparse_attn_fwd(q, k, v, mask, return_lse=True, key_scale=key_scale)
    if kv_block == 128:   # bitwise the mask of 64-token blocks that lists both halves
        half = [np.array([c for j in x for c in (2 * j, 2 * j + 1) if c < n], dtype=np.int64) for x in rows]
        split = ops.BlockMask.from_host(np.concatenate([[0], np.cumsum([len(x) for x in half])]), np.concatenate(half),
                                        mask_batch, H, n)
        out2, lse2 = ops.block_sparse_attn_fwd(q, k, v, split, return_lse=True, key_scale=key_scale)
        assert torch.equal(out.view(torch.int16), out2.view(torch.int16)) and torch.equal(lse, lse2)
    for b, h in ((0, 0), (B - 1, H // 2), (B - 1, H - 1)):
        qq, kk, vv = (np64(x[b:b + 1, :, h:h + 1]).astype(np.float64) for x in (q, k, v))
        if key_scale is not None:
            kk = og.enhance_first_frame_keys(kk, *key_scale)
        r0 = ((b if mask_batch > 1 else 0) * H + h) * n
        args = (rp[r0:r0 + n + 1] - rp[r0], ci[rp[r0]:rp[r0 + n]], 1.0 / math.sqrt(128), 1)
        O, L = oa.attention(qq, kk, vv, *args, kv_block=kv_block)
        A, _ = oa.attention(qq, kk, np.abs(vv), *args, kv_block=kv_block)
        assert within_rounding(np64(out[b:b + 1, :, h:h + 1]), O, dtype, ref_abs=A)
        got = lse[b:b + 1, h:h + 1].cpu().numpy()
        fin = np.isfinite(L)
        assert np.array_equal(np.isfinite(got), fin)
        assert np.max(np.abs(got[fin] - L[fin])) <= 1e-3


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("H,n", [(40, 14), (40, 8), (8, 40)])
def test_a_request_alone_and_in_a_batch(dtype, H, n):
    """As the header says: a launch that splits no list gives a request the same
    bits alone and in a batch of three (40 heads x 14 blocks, 70 and 210 rows on
    the fullest XCD); where the launch alone splits them (40 and 40 rows) the two
    differ by rounding only."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn(3, 64 * n, H, 128, generator=gen, device="cuda").to(dtype) for _ in range(3))
    rp, ci = wk.random_csr(np.random.Generator(np.random.PCG64(n)), H * n, n, 0.6)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n)
    batch = ops.block_sparse_attn_fwd(q, k, v, mask)
    alone = ops.block_sparse_attn_fwd(q[1:2], k[1:2], v[1:2], mask)
    if H // 8 * n > 64:
        assert torch.equal(batch[1:2].view(torch.int16), alone.view(torch.int16))
    else:
        # both round P and O once: within two roundings of sum(p |v|) and of O
        bound = ops.block_sparse_attn_fwd(q, k, v.abs(), mask)[1:2].float() + batch[1:2].float().abs()
        rel = 2.0 ** (-8 if dtype == torch.bfloat16 else -11)
        assert bool(((batch[1:2].float() - alone.float()).abs() <= 2 * rel * bound).all())


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,S,H", [(1, 189, 600), (1, 250, 200), (2, 850, 20), (1, 1950, 40), (1, 4150, 8), (2, 4150, 32)])
def test_dense_over_growing_logits_matches_oracle(dtype, B, S, H):
    """No mask, with rows not split: the masked kernel's workgroups (3, 4 and 14
    kv blocks), four waves (31 and 65) and eight (65, 64 heads), on slices of one
    packed QKV tensor.  The row maxima rise by 2^80 over the first 60 % of the
    walk and fall after it, so O and l are rescaled along the way.  First and
    last (request, head) against the oracle; P rounds to the type, so the bound
    carries one rounding of sum(p |v|)."""
    gen = torch.Generator(device="cuda").manual_seed(S)
    qkv = torch.randn(B, S, 3, H, 128, generator=gen, device="cuda") * 0.5
    qkv[:, :, 0, :, 0] = 4.0
    t = torch.arange(S, device="cuda") / S
    qkv[:, :, 1, :, 0] += (160 * torch.minimum(t / 0.6, 1 - (t - 0.6)))[None, :, None]
    qkv = qkv.to(dtype)
    q, k, v = qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2]
    n = (S + 63) // 64
    for key_scale in (None, (S // 3, 1.25)):
        out, lse = ops.block_sparse_attn_fwd(q, k, v, None, return_lse=True, key_scale=key_scale)
        for b, h in ((0, 0), (B - 1, H - 1)):
            qq, kk, vv = (np64(x[b:b + 1, :, h:h + 1]).astype(np.float64) for x in (q, k, v))
            if key_scale is not None:
                kk = og.enhance_first_frame_keys(kk, *key_scale)
            rp, ci = np.arange(n + 1) * n, np.tile(np.arange(n), n)
            O, L = oa.attention(qq, kk, vv, rp, ci, 1.0 / math.sqrt(128), 1)
            A, _ = oa.attention(qq, kk, np.abs(vv), rp, ci, 1.0 / math.sqrt(128), 1)
            assert within_rounding(np64(out[b:b + 1, :, h:h + 1]), O, dtype, ref_abs=A)
            assert np.max(np.abs(lse[b:b + 1, h:h + 1].cpu().numpy() - L)) <= 1e-3


@pytest.mark.parametrize("kv_block", [64, 128])
@pytest.mark.parametrize("H,n", [(1, 3), (2, 22), (8, 32), (9, 16), (9, 17), (17, 21), (17, 22)])
def test_rows_of_every_length_in_list_parts(kv_block, H, n):
    """The most parts follow the fullest XCD's rows (up to 32: four, up to 64:
    two, whole heads to an XCD: 9 heads x 16 and 17, 17 x 21 and 22 blocks lie on
    both sides), a row's parts its length: 0 to all blocks, so lists of 3, 4, 15
    and 16 steps and a missing second half at the end, against the oracle."""
    gen = torch.Generator().manual_seed(n)
    S = 64 * n - 17
    q, k, v = rand_qkv(gen, 1, S, H, torch.bfloat16)
    nk = -(-S // kv_block)
    rng = np.random.Generator(np.random.PCG64(H))
    rows = [np.sort(rng.choice(nk, (r + r // n) % (nk + 1), replace=False)) for r in range(H * n)]
    rp, ci = np.concatenate([[0], np.cumsum([len(x) for x in rows])]), np.concatenate(rows)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n, block=kv_block)
    out, lse = ops.block_sparse_attn_fwd(q.cuda(), k.cuda(), v.cuda(), mask, return_lse=True)
    for h in sorted({0, H // 2, H - 1}):
        a, b = rp[h * n], rp[(h + 1) * n]
        O, L = oa.attention(*(np64(x[:, :, h:h + 1]) for x in (q, k, v)), rp[h * n:(h + 1) * n + 1] - a, ci[a:b],
                            1.0 / math.sqrt(128), 1, kv_block=kv_block)
        assert within_rounding(np64(out[:, :, h:h + 1]), O, torch.bfloat16, atol=TOL16)
        got = lse[:, h:h + 1].cpu().numpy()
        assert np.array_equal(np.isfinite(got), np.isfinite(L))
        fin = np.isfinite(L)
        assert np.max(np.abs(got[fin] - L[fin])) <= 1e-3


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("kv_block", [64, 128])
@pytest.mark.parametrize("masked", [True, False])
@pytest.mark.parametrize("H,n", [(2, 30), (20, 14), (40, 14)])
def test_keys_masked_through_k_weigh_nothing(dtype, kv_block, masked, H, n):
    """Keys whose logits are -inf for every query (one element of K at -inf, of
    Q at 1) weigh nothing wherever their blocks lie in a row's list, as long as
    the walk does not begin with them: whole blocks in the middle and at the
    end, so that the parts of a split list (two heads: four, 20: two) begin with
    them and the unsplit walk (40) passes over them.  Reference: float64 softmax
    with those keys left out."""
    gen = torch.Generator().manual_seed(H)
    S = 64 * n - 9
    q, k, v = (x.cuda() for x in rand_qkv(gen, 1, S, H, dtype))
    nk = -(-S // kv_block)
    dead = torch.zeros(S, dtype=torch.bool, device="cuda")
    for a, b in ((2, 4), (5, 7)) if n == 14 else ((5, 8), (11, 15)):   # no row's walk starts there
        dead[128 * a:128 * b] = True
    q[..., 0] = 1.0
    k[:, dead, :, 0] = -math.inf
    keep = torch.ones(n, nk, dtype=torch.bool)
    if masked:
        keep[:, 1::2] = torch.rand(n, nk // 2, generator=gen) < 0.7
    mask = None
    if masked or kv_block == 128:
        rows = keep.repeat(H, 1)
        mask = ops.BlockMask.from_host(np.concatenate([[0], np.cumsum(rows.sum(1).numpy())]), rows.nonzero()[:, 1].numpy(),
                                       1, H, n, block=kv_block)
    out, lse = ops.block_sparse_attn_fwd(q, k, v, mask, return_lse=True)
    live = keep.cuda().repeat_interleave(64, 0)[:S].repeat_interleave(kv_block, 1)[:, :S] & ~dead
    for h in (0, H - 1):
        kk = k[0, :, h].double().masked_fill(dead[:, None], 0.0)
        s = (q[0, :, h].double() @ kk.t() / math.sqrt(128)).masked_fill(~live, -math.inf)
        O = torch.softmax(s, 1) @ v[0, :, h].double()
        assert within_rounding(np64(out[0, :, h]), O.cpu().numpy(), dtype)
        assert float((lse[0, h].double() - torch.logsumexp(s, 1)).abs().max()) <= 1e-3


def test_attention_strided_views_and_determinism():
    gen = torch.Generator().manual_seed(9)
    B, S, H = 2, 500, 2
    qkv = torch.randn(B, S, 3, H, 128, generator=gen).to(torch.bfloat16).cuda()
    q, k, v = qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2]
    n = (S + 63) // 64
    rng = np.random.Generator(np.random.PCG64(1))
    rp, ci = wk.random_csr(rng, H * n, n, 0.5)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n)
    o1 = ops.block_sparse_attn_fwd(q, k, v, mask)
    o2 = ops.block_sparse_attn_fwd(q, k, v, mask)
    order = ops.plan_block_mask(mask, B, S)
    o3 = ops.block_sparse_attn_fwd(q, k, v, mask, schedule=order)
    torch.cuda.synchronize()
    assert torch.equal(o1.view(torch.int16), o2.view(torch.int16))
    assert torch.equal(o1.view(torch.int16), o3.view(torch.int16))
    assert sorted(order.cpu().tolist()) == list(range(B * H))
    O, _ = oa.attention(np64(q.cpu()), np64(k.cpu()), np64(v.cpu()), rp, ci,
                        1.0 / math.sqrt(128), 1)
    assert within_rounding(np64(o1), O, torch.bfloat16)


def greedy_plan(rp, B, H, n, mask_batch, xcds=8):
    """The plan rule restated in plain Python: unit cost = listed blocks +
    q-blocks; heaviest first (ties by id) to the least-loaded XCD with room
    (lowest XCD id on equal load); units listed XCD by XCD, ascending id."""
    U = B * H
    cost = []
    for u in range(U):
        b, h = divmod(u, H)
        r0 = ((b if mask_batch > 1 else 0) * H + h) * n
        cost.append(int(rp[r0 + n] - rp[r0]) + n)
    cap = [U // xcds + (1 if x < U % xcds else 0) for x in range(xcds)]
    load, used, where = [0] * xcds, [0] * xcds, [0] * U
    for u in sorted(range(U), key=lambda u: (-cost[u], u)):
        best = min((x for x in range(xcds) if used[x] < cap[x]), key=lambda x: (load[x], x))
        load[best] += cost[u]
        used[best] += 1
        where[u] = best
    return [u for x in range(xcds) for u in range(U) if where[u] == x]


@pytest.mark.parametrize("B,H,mask_batch", [(1, 24, 1), (4, 40, 1), (3, 7, 3), (1, 1, 1), (2, 600, 2)])
def test_plan_follows_greedy_rule(B, H, mask_batch):
    n = 9
    rng = np.random.Generator(np.random.PCG64(B * 1000 + H))
    rows = mask_batch * H * n
    counts = rng.integers(1, n + 1, size=rows)
    rp = np.zeros(rows + 1, np.int64)
    np.cumsum(counts, out=rp[1:])
    ci = np.concatenate([np.sort(rng.choice(n, c, replace=False)) for c in counts])
    mask = ops.BlockMask.from_host(rp, ci, mask_batch, H, n)
    order = ops.plan_block_mask(mask, B, 64 * n).cpu().tolist()
    assert order == greedy_plan(rp, B, H, n, mask_batch)


@pytest.mark.parametrize("B,H", [(1, 24), (2, 13), (1, 5)])
def test_plan_equal_costs_follow_the_tie_rules(B, H):
    # every unit lists every block: all costs equal, so only the tie rules
    # (units by id, XCDs by id on equal load) decide the order
    n = 6
    rows = H * n
    rp = np.arange(0, rows * n + 1, n, dtype=np.int64)
    ci = np.tile(np.arange(n), rows)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n)
    order = ops.plan_block_mask(mask, B, 64 * n).cpu().tolist()
    assert order == greedy_plan(rp, B, H, n, 1)
    assert sorted(order) == list(range(B * H))


def test_attention_fp8_small_full():
    gen = torch.Generator().manual_seed(21)
    B, S, H = 2, 1000, 3
    q, k, v = rand_qkv(gen, B, S, H, torch.bfloat16)
    n = (S + 63) // 64
    rng = np.random.Generator(np.random.PCG64(2))
    rp, ci = wk.random_csr(rng, H * n, n, 0.5, empty_frac=0.05)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n)
    qc, qs = ops.quantize_fp8_blockwise(q.cuda())
    kc, ks = ops.quantize_fp8_blockwise(k.cuda())
    vc, vs = ops.quantize_fp8_blockwise(v.cuda())
    out, lse = ops.block_sparse_attn_fwd(qc, kc, vc, mask, scales=(qs, ks, vs), return_lse=True)
    torch.cuda.synchronize()
    dq = of.dequantize_blockwise(qc.cpu().numpy(), qs.cpu().numpy())
    dk = of.dequantize_blockwise(kc.cpu().numpy(), ks.cpu().numpy())
    dv = of.dequantize_blockwise(vc.cpu().numpy(), vs.cpu().numpy())
    O, L = oa.attention(dq, dk, dv, rp, ci, 1.0 / math.sqrt(128), 1)
    assert within_rounding(np64(out), O, torch.bfloat16, atol=TOL8)
    lg = lse.cpu().numpy()
    fin = np.isfinite(L)
    assert np.array_equal(np.isfinite(lg), fin)
    if fin.any():
        assert np.max(np.abs(lg[fin] - L[fin])) <= 1e-3


@pytest.mark.parametrize("kind", ["bf16", "f16", "fp8"])
def test_attention_skips_out_of_range_ids(kind):
    """Ids outside [0, n) in a mask row are skipped (the contract in
    include/chorus.h): rows with -1 ahead of their ids, or n and n + 5 after
    them, give the output of the same rows without those ids, also where a
    row holds nothing else.  Each q-block's kv walk starts at a rotated
    position of its row, which has to land on the valid ids of such rows."""
    gen = torch.Generator().manual_seed(5)
    B, S, H = 1, 1000, 3
    q, k, v = rand_qkv(gen, B, S, H, torch.float16 if kind == "f16" else torch.bfloat16)
    n = (S + 63) // 64
    rng = np.random.Generator(np.random.PCG64(11))
    rp, ci = wk.random_csr(rng, H * n, n, 0.4, empty_frac=0.1)
    rows = []
    for r in range(H * n):
        ids = [int(j) for j in ci[rp[r]:rp[r + 1]]]
        if r % 3 == 0:
            ids = [-1] + ids
        elif r % 3 == 1:
            ids = ids + [n, n + 5]
        rows.append(ids)
    assert any(len(x) == 1 and x[0] == -1 for x in rows)   # a row of invalid ids only
    rp2 = np.concatenate([[0], np.cumsum([len(x) for x in rows])])
    ci2 = np.array([j for x in rows for j in x], dtype=np.int64)
    mask = ops.BlockMask.from_host(rp2, ci2, 1, H, n)
    sm = 1.0 / math.sqrt(128)
    if kind == "fp8":
        (qc, qs), (kc, ks), (vc, vs) = (ops.quantize_fp8_blockwise(x.cuda()) for x in (q, k, v))
        out, lse = ops.block_sparse_attn_fwd(qc, kc, vc, mask, scales=(qs, ks, vs), sm_scale=sm,
                                             return_lse=True)
        deq = [of.dequantize_blockwise(c.cpu().numpy(), s_.cpu().numpy())
               for c, s_ in ((qc, qs), (kc, ks), (vc, vs))]
        O, L = oa.attention(*deq, rp, ci, sm, 1)
        atol = TOL8
    else:
        out, lse = ops.block_sparse_attn_fwd(q.cuda(), k.cuda(), v.cuda(), mask, sm_scale=sm,
                                             return_lse=True)
        O, L = attn_ref_full(q, k, v, rp, ci, 1, sm)
        atol = TOL16
    torch.cuda.synchronize()
    assert within_rounding(np64(out), O, torch.float16 if kind == "f16" else torch.bfloat16, atol=atol)
    lg = lse.cpu().numpy()
    fin = np.isfinite(L)
    assert np.array_equal(np.isfinite(lg), fin)
    assert np.max(np.abs(lg[fin] - L[fin])) <= 1e-3


def test_attention_fp8_extreme_value_block_scales():
    """V blocks whose fp8 scale is zero-input (scale 1), denormal (values of
    order 1e-37) or large sit next to ordinary blocks in the same rows: the
    per-block V scale folded into the exponent stays finite and the output
    matches the oracle on the dequantised inputs."""
    gen = torch.Generator().manual_seed(33)
    B, S, H = 1, 640, 2
    q, k, v = rand_qkv(gen, B, S, H, torch.bfloat16)
    n = S // 64
    v = v.float()
    v[:, 64:128] = 0.0                      # all-zero block: scale 1, codes 0
    v[:, 192:256] *= 1e-36                  # subnormal block scale (amax / 448 < FLT_MIN)
    v[:, 448:512] *= 2.0 ** -123            # amax below 448 / FLT_MAX
    v[:, 320:384] *= 3e3                    # large block next to unit ones
    v = v.to(torch.bfloat16)
    rp = np.arange(0, H * n * n + 1, n)
    ci = np.tile(np.arange(n), H * n)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n)
    (qc, qs), (kc, ks), (vc, vs) = (ops.quantize_fp8_blockwise(x.cuda()) for x in (q, k, v))
    assert float(vs[0, 0, 3].item()) < 1.17549435e-38   # the denormal case is present
    out = ops.block_sparse_attn_fwd(qc, kc, vc, mask, scales=(qs, ks, vs))
    torch.cuda.synchronize()
    got = np64(out)
    assert np.all(np.isfinite(got))
    deq = [of.dequantize_blockwise(c.cpu().numpy(), s_.cpu().numpy()) for c, s_ in ((qc, qs), (kc, ks), (vc, vs))]
    O, _ = oa.attention(*deq, rp, ci, 1.0 / math.sqrt(128), 1)
    # fp8 P~ (relative 2^-4 per weight) on values up to 3e3 in magnitude
    Oabs, _ = oa.attention(deq[0], deq[1], np.abs(deq[2]), rp, ci, 1.0 / math.sqrt(128), 1)
    bound = np.maximum(TOL8, 1e-3 + 2.0 ** -4 * Oabs) + 2.0 ** -8 * np.abs(O)
    assert np.all(np.abs(got - O) <= bound), float(np.max(np.abs(got - O) - bound))


# --------------------------------------------------------------------------- mask checker
def test_validate_flags():
    H, n = 2, 5
    good_rp = np.array([0, 2, 3, 3, 5, 6, 8, 9, 9, 10, 12])
    good_ci = np.array([0, 3, 1, 2, 4, 0, 1, 2, 3, 0, 1, 4])
    assert ops.validate_block_mask(ops.BlockMask.from_host(good_rp, good_ci, 1, H, n)) == 0
    bad = good_ci.copy()
    bad[1] = 0                                              # not ascending
    assert ops.validate_block_mask(ops.BlockMask.from_host(good_rp, bad, 1, H, n)) & 8
    bad = good_ci.copy()
    bad[4] = 5                                              # out of range
    assert ops.validate_block_mask(ops.BlockMask.from_host(good_rp, bad, 1, H, n)) & 4
    rp = good_rp.copy()
    rp[3] = 1                                               # decreasing
    assert ops.validate_block_mask(ops.BlockMask.from_host(rp, good_ci, 1, H, n)) & 2


def test_abi_rejects_bad_arguments_on_device():
    q = torch.zeros(2, 100, 2, 128, dtype=torch.bfloat16, device="cuda")
    n = 2
    mask = ops.BlockMask.from_host(np.arange(3 * 2 * n + 1), np.zeros(3 * 2 * n), 3, 2, n)
    with pytest.raises(RuntimeError, match="INVALID_ARG"):
        ops.block_sparse_attn_fwd(q, q, q, mask)
    with pytest.raises(RuntimeError, match="INVALID_ARG"):
        ops.build_block_mask(q, q, 1.5, 0.0)


# --------------------------------------------------------------------------- full-size workloads
_cache = {}


def workload_state(key):
    if key in _cache:
        return _cache[key]
    _cache.clear()
    torch.cuda.empty_cache()
    wl = wk.WORKLOADS[key]
    inp = wk.make_inputs(wl)
    st = {"wl": wl, "inp": inp}
    q, k, v = inp.q.cuda(), inp.k.cuda(), inp.v.cuda()
    mq, mk = inp.mask_q.cuda(), inp.mask_k.cuda()
    mask = ops.build_block_mask(mq, mk, wl.top_p, wl.min_top_k, sm_scale=wl.sm_scale)
    st.update(q=q, k=k, v=v, mask=mask)
    if wl.dtype == "fp8":
        st["q8"] = ops.quantize_fp8_blockwise(q)
        st["k8"] = ops.quantize_fp8_blockwise(k)
        st["v8"] = ops.quantize_fp8_blockwise(v)
    torch.cuda.synchronize()
    _cache[key] = st
    return st


FULL = ["wan5b_720p_bf16", "wan14b_480p_reuse_bf16", "wan14b_720p_fp8", "wan14b_480p_batch4_bf16"]


@pytest.mark.parametrize("key", FULL)
def test_full_size_mask_sampled_heads(key):
    st = workload_state(key)
    wl, inp, mask = st["wl"], st["inp"], st["mask"]
    rp, ci = mask.to_host()
    heads = sorted({0, wl.H // 2, wl.H - 1})
    o = om.build_block_mask(inp.mask_q.float().numpy(), inp.mask_k.float().numpy(), wl.sm_scale,
                            wl.top_p, wl.min_top_k, heads=heads)
    n = wl.n_blocks
    rows = [h * n + i for h in heads for i in range(n)]
    rep = compare_masks(rp, ci, o, rows, wl.top_p, wl.min_top_k)
    assert rep.ok, rep.failing[:5]
    assert abs(mask.density - wl.density) < 0.01
    assert ops.validate_block_mask(mask) == 0


def _check_heads(wl, out, lse, rp, ci, ins, heads, tol):
    """Every q-block (the partial last one included) of the listed heads of
    every request against the oracle, outputs and LSE.  ``ins(b, h)`` gives
    the float64 [S, D] q, k, v of (b, h) exactly as the kernel read them."""
    n = wl.n_blocks
    worst = worst_lse = 0.0
    for b in range(wl.B):
        for h in heads:
            qh, kh, vh = ins(b, h)
            oh = np64(out[b, :, h].cpu())
            lh = lse[b, h].cpu().numpy().astype(np.float64)
            for i in range(n):
                r = oa.mask_row_index(b, h, i, wl.H, n, 1)
                o_ref, l_ref = oa.attention_block(qh, kh, vh, oa.row_blocks(rp, ci, r), i, wl.sm_scale)
                rows = slice(i * 64, i * 64 + o_ref.shape[0])
                worst = max(worst, max_abs_err(oh[rows], o_ref))
                worst_lse = max(worst_lse, max_abs_err(lh[rows], l_ref))
    assert worst <= tol, worst
    assert worst_lse <= 1e-3, worst_lse
    return worst


@pytest.mark.parametrize("key", FULL)
def test_full_size_attention_every_q_block_of_two_heads(key):
    """Full-size launch (planned XCD order, as the benchmark runs it): every
    q-block of the sharpest and the most diffuse head of every request
    against the oracle; the unplanned order gives bitwise the same output."""
    st = workload_state(key)
    wl, mask = st["wl"], st["mask"]
    rp, ci = mask.to_host()
    order = ops.plan_block_mask(mask, wl.B, wl.S)
    if wl.dtype == "fp8":
        (qc, qs), (kc, ks), (vc, vs) = st["q8"], st["k8"], st["v8"]
        out, lse = ops.block_sparse_attn_fwd(qc, kc, vc, mask, scales=(qs, ks, vs), schedule=order,
                                             return_lse=True)
        out2 = ops.block_sparse_attn_fwd(qc, kc, vc, mask, scales=(qs, ks, vs))
        tol = TOL8

        def ins(b, h):
            sl = lambda c, s: of.dequantize_blockwise(c[b:b + 1, :, h:h + 1].cpu().numpy(),
                                                      s[b:b + 1, h:h + 1].cpu().numpy())[0, :, 0]
            return sl(qc, qs), sl(kc, ks), sl(vc, vs)
    else:
        out, lse = ops.block_sparse_attn_fwd(st["q"], st["k"], st["v"], mask, schedule=order,
                                             return_lse=True)
        out2 = ops.block_sparse_attn_fwd(st["q"], st["k"], st["v"], mask)
        tol = TOL16

        def ins(b, h):
            return tuple(np64(x[b, :, h].cpu()).astype(np.float64) for x in (st["q"], st["k"], st["v"]))
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
    _check_heads(wl, out, lse, rp, ci, ins, (0, wl.H - 1), tol)


def test_plan_beyond_4096_units_keeps_natural_order_and_results():
    """B * H > 4096 units: the plan keeps the natural order; any order gives
    bitwise the same attention output."""
    B, H, S = 65, 64, 64
    n = 1
    rng = np.random.Generator(np.random.PCG64(4097))
    rp = np.arange(B * H * n + 1, dtype=np.int64)
    ci = np.zeros(B * H * n, dtype=np.int64)
    mask = ops.BlockMask.from_host(rp, ci, B, H, n)
    order = ops.plan_block_mask(mask, B, S)
    assert order.cpu().tolist() == list(range(B * H))
    gen = torch.Generator().manual_seed(2)
    q, k, v = rand_qkv(gen, B, S, H, torch.bfloat16)
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    ref = ops.block_sparse_attn_fwd(q, k, v, mask)
    perm = torch.from_numpy(rng.permutation(B * H).astype(np.int32)).cuda()
    out = ops.block_sparse_attn_fwd(q, k, v, mask, schedule=perm)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))


def test_tiny_f16_workload_every_element():
    """The tiny f16 check (B 1, H 2, S 4096 on a 4 x 32 x 32 grid, fixed
    random 25 % mask with the diagonal kept) through the C ABI: every output
    element and every LSE against the oracle's literal form (64 x S logits per
    q-block, unlisted blocks at -inf), plain and planned launch order."""
    wl = wk.WORKLOADS["tiny_f16"]
    inp = wk.make_inputs(wl)
    rp, ci = inp.random_mask
    mask = ops.BlockMask.from_host(rp, ci, 1, wl.H, wl.n_blocks)
    q, k, v = inp.q.cuda(), inp.k.cuda(), inp.v.cuda()
    out, lse = ops.block_sparse_attn_fwd(q, k, v, mask, sm_scale=wl.sm_scale, return_lse=True)
    order = ops.plan_block_mask(mask, wl.B, wl.S)
    out2 = ops.block_sparse_attn_fwd(q, k, v, mask, sm_scale=wl.sm_scale, schedule=order)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))
    O, L = oa.attention(np64(inp.q), np64(inp.k), np64(inp.v), rp, ci, wl.sm_scale, 1, form="literal")
    assert max_abs_err(np64(out), O) <= TOL16
    assert max_abs_err(lse.cpu().numpy(), L) <= 1e-3


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("B,H", [(1, 13), (3, 3), (1, 1)])
def test_planned_order_with_units_not_a_multiple_of_eight(dtype, B, H):
    """B * H (request, head) units not a multiple of the 8 XCDs: each XCD
    walks exactly the units the plan gave it; any order gives bitwise the
    same output, and it matches the oracle."""
    gen = torch.Generator().manual_seed(B * 100 + H)
    S = 700
    q, k, v = rand_qkv(gen, B, S, H, torch.bfloat16)
    n = (S + 63) // 64
    rng = np.random.Generator(np.random.PCG64(B * 7 + H))
    rp, ci = wk.random_csr(rng, H * n, n, 0.4)
    mask = ops.BlockMask.from_host(rp, ci, 1, H, n)
    order = ops.plan_block_mask(mask, B, S)
    assert sorted(order.cpu().tolist()) == list(range(B * H))
    if dtype == "fp8":
        cs = [ops.quantize_fp8_blockwise(x.cuda()) for x in (q, k, v)]
        args, kw = [c for c, _ in cs], {"scales": tuple(s_ for _, s_ in cs)}
        ins = [of.dequantize_blockwise(c.cpu().numpy(), s_.cpu().numpy()) for c, s_ in cs]
        tol = TOL8
    else:
        args, kw = [x.cuda() for x in (q, k, v)], {}
        ins = [np64(x) for x in (q, k, v)]
        tol = TOL16
    natural = ops.block_sparse_attn_fwd(*args, mask, **kw)
    planned = ops.block_sparse_attn_fwd(*args, mask, schedule=order, **kw)
    perm = torch.from_numpy(rng.permutation(B * H).astype(np.int32)).cuda()
    shuffled = ops.block_sparse_attn_fwd(*args, mask, schedule=perm, **kw)
    torch.cuda.synchronize()
    assert torch.equal(natural.view(torch.int16), planned.view(torch.int16))
    assert torch.equal(natural.view(torch.int16), shuffled.view(torch.int16))
    O, _ = oa.attention(*ins, rp, ci, 1.0 / math.sqrt(128), 1)
    assert within_rounding(np64(natural), O, torch.bfloat16, atol=tol)

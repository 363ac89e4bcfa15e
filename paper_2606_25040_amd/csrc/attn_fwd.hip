// Block-sparse attention forward, fp16 / bf16 (Chorus II Sec. 3.2 "Efficient
// block-sparse kernel": only the listed block pairs enter QK^T, softmax, PV).
//
// One workgroup = one work item (request b, head h, 64-query block i), two
// waves of 32 queries, 32 KB of LDS, so four workgroups (two waves per SIMD)
// share a CU.  The listed kv blocks are walked from a rotated start
// (walk_target), so the q-blocks in flight on an XCD read about the same kv
// blocks at the same time.  For each listed block j the wave works in two
// steps, one per 32-key half of the block:
//   * S^T = K Q^T of that half of the NEXT listed block, with
//     v_mfma_f32_32x32x16 (A = K rows from LDS, B = Q fragments kept in
//     registers): each lane holds scores of ONE query (lanes l and l ^ 32
//     split the keys), so the row max and row sum are lane-local plus one
//     half-wave exchange;
//   * beside those products, which need nothing of block j, the probabilities
//     of this half of block j: online softmax in the log2 domain; the running
//     max is only moved (and O, l rescaled) when some row's max grew by more
//     than kRescaleLog2, so P <= 2^kRescaleLog2 and most blocks skip the
//     64-register rescale;
//   * O^T += V^T P^T of the half with the same MFMA; V^T fragments come from
//     the row-major tile through ds_read_b64_tr_b16; P is the score
//     accumulator converted to 16-bit in registers.
// K and V halves (8 KB) go global -> LDS with global_load_lds_dwordx4 (no
// register staging) into two buffers each, so a half is requested a whole step
// before it is read; one barrier per step.  After the last listed block the
// products for a next one run on stale tiles and are not used, which costs
// less than a second copy of the loop body (whose registers spill); rows of one
// block pay 0.2 us for it (6.5 against 6.3 us in the version below).
// What bounds it: the tile feed (L2 misses, and the clock under that load)
// and the vector instructions beside the MFMAs.  Same bits as the version that
// ran QK^T, softmax and PV of a 64-key block one after the other on single
// buffers, and faster: batch-4 480p 14B (bf16, 15 %) 13.93 against 14.76 ms,
// 720p 5B (bf16, 20 %) 1.99 against 2.09 ms, f16 with kv blocks of 128 and a
// key scale (2 x 16 heads, S = 17,523) 1.16 against 1.21 ms.  Measured beside
// it: two q-blocks per workgroup walking the union of their lists 15.8 ms
// (every fifth step has work for one of them only), separate waits for K and V
// 15.60 against 15.17 ms, raised wave priority during QK^T 15.39.
// LDS tiles are XOR-swizzled in 16-byte chunks (the direct loads permute the
// global addresses instead of the LDS ones) so that the b128 K reads and the
// transposed b64 V reads are bank-conflict free.
// Epilogue: O = O^T / l written as 16-bit, lse = ln(sum exp) in fp32.
// With P > 1 a workgroup of P wave pairs splits the row's walk into up to P runs,
// each with tiles of its own, and part 0 merges the (m, l, O) of the others at the
// end: for launches with too few rows to fill the chip (list_parts).
// Template flags: DENSE walks every kv block; KSCALE multiplies the logits of
// keys below n_first by beta (first-frame key enhancement, Eq. 1); KV2 reads a mask of 128-token kv blocks
// and walks each as its two 64-token halves.  Each flag is its own
// instantiation, so the plain path carries none of the others' work.
// Without a mask attn_dense_16_kernel below runs, except on small launches
// (launch_dense).
#include <cfloat>

#include "attn_common.h"

namespace chorus {
namespace {

constexpr float kRescaleLog2 = 8.f;
constexpr int kTileBytes = kBlock * kHeadDim * 2;   // 16 KB per 16-bit tile

// 16-byte chunk position of chunk c in row r.
__device__ inline int k_swz(int r, int c) { return c ^ (r & 15); }
__device__ inline int v_swz_bits(int r) { return (0xE4A0 >> (4 * (r & 3))) & 15; }   // {0, 10, 4, 14}
__device__ inline int v_swz(int r, int c) { return c ^ v_swz_bits(r); }

template <bool BF16>
struct Elt;
// The transposed LDS reads go through the typed builtin (or a whole-vector
// bitcast) and are joined with __builtin_shufflevector: assembling the
// operand element by element from the i16 variant was miscompiled.
template <>
struct Elt<true> {
  using vec8 = bf16x8;
  using scalar = __bf16;
  static __device__ inline f32x16 mfma(vec8 a, vec8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ inline vec8 tr_pair(const char* lo, const char* hi) {
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)lo);
    const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)hi);
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};
template <>
struct Elt<false> {
  using vec8 = f16x8;
  using scalar = _Float16;
  static __device__ inline f32x16 mfma(vec8 a, vec8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
  static __device__ inline vec8 tr_pair(const char* lo, const char* hi) {
    const f16x4 a = __builtin_bit_cast(f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)lo));
    const f16x4 b = __builtin_bit_cast(f16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)hi));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

constexpr int kHalfBytes = kTileBytes / 2;   // 32 keys

// This wave's share (one of two) of a 32 x 128 half tile: load u fills LDS rows
// 8u + 4 wave .. + 3 (1 KB, lane-linear), each lane fetching the global chunk
// that the swizzle places at its slot.  Full blocks add a per-lane offset
// fixed for the whole kernel to the half's first row.
struct HalfLoader {
  const char* base;
  uint32_t ss;
  uint32_t off[4];
  int r0, p;
  template <bool IS_K>
  __device__ void init(const uint16_t* b, int64_t stride, int wave, int lane) {
    base = reinterpret_cast<const char*>(b);
    ss = (uint32_t)(stride * 2);
    r0 = 4 * wave + (lane >> 4);
    p = lane & 15;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 8 * u + r0;
      off[u] = (uint32_t)r * ss + (uint32_t)(IS_K ? k_swz(r, p) : v_swz(r, p)) * 16;
    }
  }
  template <bool IS_K>
  __device__ void load(uint32_t lds, int j, int t, int S, int wave) const {
    const int tok0 = j * kBlock + 32 * t;
    uint32_t o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = off[u];
    const char* from = base + (int64_t)tok0 * ss;
    if (j * kBlock + kBlock > S) {
      // partial last block: rows past the end re-read row S - 1 (offsets from
      // token 0: the half may start past the end)
      from = base;
      int pp = p, rr = r0;
      asm volatile("" : "+v"(pp), "+v"(rr));   // computed here: kept across the loop it would cost registers
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 8 * u + rr;
        o[u] = (uint32_t)min(tok0 + r, S - 1) * ss + (uint32_t)(IS_K ? k_swz(r, pp) : v_swz(r, pp)) * 16;
      }
    }
    dma16x4(lds + wave * 1024, from, o);
  }
};

// Listed blocks from which a row is split in two and in four parts.  The merge
// costs about 1 us of a row's latency, a block 0.75 us unsplit: a list of 3
// takes 9.0 us unsplit and 9.2 in two parts, one of 5 11.2 and 10.4; one of 12
// 14.2 in two and 14.8 in four, one of 20 19.4 and 18.8.
constexpr int kSplit2 = 4, kSplit4 = 16;

template <bool BF16, bool DENSE, bool KSCALE, bool KV2, int P>
__global__ __launch_bounds__(128 * P) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_fwd_16_kernel(AttnArgs a) {
  using E = Elt<BF16>;
  using vec8 = typename E::vec8;
  using scalar = typename E::scalar;
  __shared__ __attribute__((aligned(1024))) char kv_s[P][4][kHalfBytes];   // per part: two K halves, two V halves

  const int item = work_item(a.order, a.B * a.H, a.n);
  if (item < 0) return;
  const int n = a.n, H = a.H, S = a.S;
  const int i = item % n;
  const int bh = item / n;
  const int h = bh % H, b = bh / H;
  // The CSR row of (b, h, i) (DENSE: every kv block).  KV2: it lists kv blocks
  // of 128 tokens and the walk visits both 64-token halves of each (positions
  // 2 p and 2 p + 1 of the doubled list, without a missing second half at its
  // end).
  int kb0 = 0, kb1 = n;
  ConstI32* cidx = as_constant(a.col_idx);   // scalar loads
  auto kv_at = [&](int p) { return DENSE ? p : KV2 ? 2 * cidx[p >> 1] + (p & 1) : cidx[p]; };
  if (!DENSE) {
    const int64_t mrow = ((int64_t)(a.mask_batch > 1 ? b : 0) * H + h) * n + i;
    kb0 = a.row_ptr[mrow];
    kb1 = a.row_ptr[mrow + 1];
    if (KV2) {
      kb0 *= 2;
      kb1 *= 2;
      if (kb1 > kb0 && kv_at(kb1 - 1) == n) --kb1;
    }
  }
  const int tid = threadIdx.x;
  const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = wave_id & 1, part = wave_id >> 1;   // query half, share of the list
  const int L = kb1 - kb0;
  // Short lists use fewer parts than the launch brings; the waves of the others
  // leave here, ahead of every barrier.
  const int parts = P == 1 ? 1 : L < kSplit2 ? 1 : P == 2 || L < kSplit4 ? 2 : 4;
  if (P > 1 && part >= parts) return;
  int left = L, pos = kb0;
  if (!DENSE && L > 0) pos += walk_rotation_wave<KV2>(a.col_idx, kb0, kb1, walk_target(i, n));
  if (P > 1) {   // this part's run of the walk
    const int lp = parts >> 1;   // log2(parts)
    const int w0 = (int)((int64_t)part * L >> lp);
    left = (int)((int64_t)(part + 1) * L >> lp) - w0;
    pos += w0;
    if (pos >= kb1) pos -= L;
  }
  // next listed block (-1 when done), the id after it read ahead; ids outside
  // [0, n) are skipped (the builder never emits them)
  int ahead = left > 0 ? kv_at(pos) : 0;
  auto next = [&]() {
    for (;;) {
      if (left <= 0) return -1;
      const int j = ahead;
      --left;
      ++pos;
      if (pos == kb1) pos = kb0;
      if (left > 0) ahead = kv_at(pos);
      if ((unsigned)j < (unsigned)n) return j;
    }
  };

  const int lane = tid & 63;
  const int l32 = lane & 31, hl = lane >> 5;
  const int g = lane >> 4, j16 = lane & 15;

  const uint16_t* kbase = static_cast<const uint16_t*>(a.k.data) + (int64_t)b * a.k.sb + (int64_t)h * a.k.sh;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.v.data) + (int64_t)b * a.v.sb + (int64_t)h * a.v.sh;
  HalfLoader kl, vl;
  kl.init<true>(kbase, a.k.ss, wave, lane);
  vl.init<false>(vbase, a.v.ss, wave, lane);
  char(*k_s)[kHalfBytes] = &kv_s[P > 1 ? part : 0][0];
  char(*v_s)[kHalfBytes] = &kv_s[P > 1 ? part : 0][2];
  const uint32_t klds = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)k_s;
  const uint32_t vlds = klds + 2 * kHalfBytes;
  int jc = next();
  if (jc >= 0) {
    kl.load<true>(klds, jc, 0, S, wave);
    kl.load<true>(klds + kHalfBytes, jc, 1, S, wave);
  }
  int jn = next();

  const int qrow = i * kBlock + wave * 32 + l32;
  vec8 qf[8];
  {
    const uint16_t* qp = static_cast<const uint16_t*>(a.q.data) + (int64_t)b * a.q.sb + (int64_t)qrow * a.q.ss +
                         (int64_t)h * a.q.sh + 8 * hl;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (qrow < S) {
        qf[s] = *reinterpret_cast<const vec8*>(qp + 16 * s);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[s][e] = (scalar)0.f;
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0)
  __syncthreads();

  const int k_row_off = l32 * 256;
  const int k_swzl = l32 & 15;
  const int v_lane_off = (j16 >> 2) * 256 + 8 * (j16 & 1) + 4 * (g >> 1) * 256;
  const int v_c0 = 2 * (g & 1) + ((j16 & 3) >> 1);
  const int v_sl = v_swz_bits(j16 >> 2);

  const float cl2 = a.sm_scale * kLog2e;
  // The running max of parts 1 .. P - 1 starts at the lowest finite value: a
  // part may begin with a block whose logits are all -inf (keys masked through
  // K), and -inf - (-inf) is NaN.  Part 0 begins where the unsplit walk does.
  float m_run = P > 1 && part > 0 ? -FLT_MAX : -INFINITY, l_run = 0.f, rs = 0.f;
  f32x16 o[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[u][r] = 0.f;

  auto qk = [&](f32x16& s, const char* kt) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int d = 0; d < 8; ++d)
      s = E::mfma(*reinterpret_cast<const vec8*>(kt + k_row_off + (((2 * d + hl) ^ k_swzl) << 4)), qf[d], s);
  };
  auto fix = [&](f32x16 (&s)[2], int j) {   // key scale (Eq. 1) and the end of the sequence
    int hl4 = 4 * hl;
    asm volatile("" : "+v"(hl4));   // the key indices are computed here each time
    if (KSCALE && j * kBlock < a.ks.n_first) {
      const int lim = a.ks.n_first - j * kBlock;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (32 * t + 8 * (r >> 2) + hl4 + (r & 3) < lim) s[t][r] *= a.ks.beta;
    }
    if (j * kBlock + kBlock > S) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (j * kBlock + 32 * t + 8 * (r >> 2) + hl4 + (r & 3) >= S) s[t][r] = -INFINITY;
    }
  };
  auto row_max = [&](const f32x16 (&s)[2]) {
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[t][r]);
    return pair_max(mx);
  };
  auto rescale = [&](float mx) {
    const float m_new = fmaxf(m_run, mx * cl2);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run + kRescaleLog2) != 0) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[u][r] *= alpha;
    }
  };
  auto probs = [&](const f32x16& s, vec8 (&pf)[2]) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = __builtin_amdgcn_exp2f(s[r] * cl2 - m_run);
      rs += p;
      pf[r >> 3][r & 7] = (scalar)p;
    }
  };
  auto pv = [&](const vec8 (&pf)[2], const char* vt) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int cu = (4 * u + v_c0) ^ v_sl;
        const char* lo = vt + 16 * hh * 256 + v_lane_off + (cu << 4);
        const vec8 vf = E::tr_pair(lo, lo + 8 * 256);
        o[u] = E::mfma(vf, pf[hh], o[u]);
      }
  };

  f32x16 s0[2], s1[2];
  float mx = -INFINITY;
  if (jc >= 0) {
    qk(s0[0], k_s[0]);
    qk(s0[1], k_s[1]);
    fix(s0, jc);
    mx = row_max(s0);
  }
  CHORUS_WAIT_LDS_TILES();
  __syncthreads();
  if (jc >= 0) {
    vl.load<false>(vlds, jc, 0, S, wave);
    if (jn >= 0) kl.load<true>(klds, jn, 0, S, wave);
  }
  // block jc: probabilities and PV, half by half, beside QK^T of the same half
  // of block jn.  With P > 1 a part that is done only keeps the barriers.
  auto step = [&](f32x16 (&sc)[2], f32x16 (&sn)[2]) {
    const int j2 = next();
    CHORUS_WAIT_LDS_TILES();
    __syncthreads();
    if (P == 1 || jc >= 0) {
      if (jn >= 0) kl.load<true>(klds + kHalfBytes, jn, 1, S, wave);
      vl.load<false>(vlds + kHalfBytes, jc, 1, S, wave);
      rescale(mx);
      rs = 0.f;
      vec8 pf[2];
      qk(sn[0], k_s[0]);
      probs(sc[0], pf);
      pv(pf, v_s[0]);
    }
    CHORUS_WAIT_LDS_TILES();
    __syncthreads();
    if (P == 1 || jc >= 0) {
      if (j2 >= 0) kl.load<true>(klds, j2, 0, S, wave);
      if (jn >= 0) vl.load<false>(vlds, jn, 0, S, wave);
      vec8 pf[2];
      qk(sn[1], k_s[1]);
      probs(sc[1], pf);
      pv(pf, v_s[1]);
      l_run += rs;
      mx = row_max(sn);
      if (jn >= 0 && ((KSCALE && jn * kBlock < a.ks.n_first) || jn * kBlock + kBlock > S)) {
        fix(sn, jn);   // rare: first-frame blocks and a partial last one take the maximum again
        mx = row_max(sn);
      }
    }
    jc = jn;
    jn = j2;
  };
  if (P == 1) {
    while (jc >= 0) {
      step(s0, s1);
      if (jc < 0) break;
      step(s1, s0);
    }
  } else {
    const int steps = (L + parts - 1) >> (parts >> 1);   // of the longest part
    for (int x = 0; x < steps; ++x) {
      step(s0, s1);
      if (++x >= steps) break;
      step(s1, s0);
    }
  }

  float l_tot = pair_sum(l_run);   // lane pair (l, l ^ 32) holds partial sums of the same query
  if (P > 1 && parts > 1) {
    // Parts 1 .. parts - 1 hand their (m, l, O) to part 0 through the tiles.
    float* mine = reinterpret_cast<float*>(&kv_s[part][0][0]);
    __shared__ float ml[P][2][2][32];   // [part][query half][m, l][query]
    CHORUS_WAIT_LDS_TILES();
    __syncthreads();
    if (part > 0) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
          reinterpret_cast<float4*>(mine)[((4 * u + rr) * 2 + wave) * 64 + lane] =
              make_float4(o[u][4 * rr], o[u][4 * rr + 1], o[u][4 * rr + 2], o[u][4 * rr + 3]);
      if (hl == 0) {
        ml[part][wave][0][l32] = m_run;
        ml[part][wave][1][l32] = l_tot;
      }
    }
    CHORUS_WAIT_LDS_TILES();
    __syncthreads();
    if (part > 0) return;
    float m_all = m_run;
#pragma unroll
    for (int x = 1; x < P; ++x)
      if (x < parts) m_all = fmaxf(m_all, ml[x][wave][0][l32]);
    // m_all is finite or +inf: a part that saw no finite logit gets weight 0,
    // or has nothing to add
    auto weight = [&](float m) { return __builtin_amdgcn_exp2f(m - m_all); };
    const float f0 = weight(m_run);
    l_tot *= f0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[u][r] *= f0;
#pragma unroll
    for (int x = 1; x < P; ++x) {
      if (x >= parts) break;
      const float f = weight(ml[x][wave][0][l32]);
      l_tot += f * ml[x][wave][1][l32];
      const float4* their = reinterpret_cast<const float4*>(&kv_s[x][0][0]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const float4 t = their[((4 * u + rr) * 2 + wave) * 64 + lane];
          o[u][4 * rr] += f * t.x;
          o[u][4 * rr + 1] += f * t.y;
          o[u][4 * rr + 2] += f * t.z;
          o[u][4 * rr + 3] += f * t.w;
        }
    }
    m_run = m_all;
  }

  const bool live = kb1 > kb0 && l_tot > 0.f;
  const float inv_l = live ? 1.f / l_tot : 0.f;
  if (qrow < S) {
    uint16_t* op = static_cast<uint16_t*>(const_cast<void*>(a.o.data)) + (int64_t)b * a.o.sb +
                   (int64_t)qrow * a.o.ss + (int64_t)h * a.o.sh;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        scalar v4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v4[e] = (scalar)(o[u][4 * rr + e] * inv_l);
        uint2 packed;
        __builtin_memcpy(&packed, v4, 8);
        *reinterpret_cast<uint2*>(op + 32 * u + 8 * rr + 4 * hl) = packed;
      }
    if (a.lse && hl == 0)
      a.lse[((int64_t)b * H + h) * S + qrow] = live ? (m_run + __builtin_log2f(l_tot)) * kLn2 : -INFINITY;
  }
}

// This wave's share (1 of NW) of a 64 x 128 16-bit tile.
template <int NW>
struct SharedTileLoader {
  static constexpr int kInstr = 16 / NW;   // 1 KB instructions per wave, 4 rows each
  const char* base;
  uint32_t ss;
  uint32_t off;        // lane offset (row r0, swizzled chunk): 4 NW rows on, the swizzle repeats
  int r0, p;
  template <bool IS_K>
  __device__ void init(const uint16_t* b, int64_t stride, int wave, int lane) {
    base = reinterpret_cast<const char*>(b);
    ss = (uint32_t)(stride * 2);
    r0 = 4 * wave + (lane >> 4);
    p = lane & 15;
    static_assert(4 * NW % 16 == 0, "the K swizzle has a period of 16 rows");
    off = (uint32_t)r0 * ss + (uint32_t)(IS_K ? k_swz(r0, p) : v_swz(r0, p)) * 16;
  }
  template <bool IS_K>
  __device__ void load(uint32_t lds, int j, int S, int wave) const {
    if (j * kBlock + kBlock <= S) {
      const char* rowj = base + (int64_t)j * kBlock * ss;
#pragma unroll
      for (int u = 0; u < kInstr; ++u)
        dma16(lds + (NW * u + wave) * 1024, rowj + (int64_t)(4 * NW * u) * ss, off);
    } else {
#pragma unroll
      for (int u = 0; u < kInstr; ++u) {
        const int r = 4 * NW * u + r0;
        const int c = IS_K ? k_swz(r, p) : v_swz(r, p);
        const int tok = min(j * kBlock + r, S - 1);
        dma16(lds + (NW * u + wave) * 1024, base, (uint32_t)tok * ss + (uint32_t)c * 16);
      }
    }
  }
};

// Dense attention (no mask): every q-block visits every kv block, so NW waves
// of 32 queries share each tile and the work inside a wave is pipelined.  At
// step j a wave issues QK^T of block j + 1 (its 16 MFMAs need nothing of block
// j) beside the exponentials of block j, then PV of block j beside the row max
// of block j + 1, so the matrix cores have work during the softmax; K and V
// are double-buffered (64 KB), refilled a whole step ahead, one barrier per kv
// block.  Each output row takes the same operations as in the masked kernel, in
// the natural order of the kv blocks: an explicit full mask gives the same bits
// up to 14 kv blocks, beyond which some rows' masked walks start rotated.
// Measured at 480p 14B (S = 32,760, 40 heads, bf16): 17.8-18.6 ms, 1,180-1,230
// TFLOP/s, matrix cores busy 62 % of the cycles, against 22.8-23.2 ms for the
// masked kernel's two-wave workgroup (46 %); four waves 19.0 ms.  What is left
// is the clock (1.8 GHz under this load) and the issue of the softmax's vector
// instructions.
template <bool BF16, bool KSCALE, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_dense_16_kernel(AttnArgs a, int np) {
  using E = Elt<BF16>;
  using vec8 = typename E::vec8;
  using scalar = typename E::scalar;
  __shared__ __attribute__((aligned(1024))) char k_s[2][kTileBytes];
  __shared__ __attribute__((aligned(1024))) char v_s[2][kTileBytes];

  const int item = work_item(a.order, a.B * a.H, np);
  if (item < 0) return;
  const int n = a.n, H = a.H, S = a.S;
  const int ip = item % np;
  const int bh = item / np;
  const int h = bh % H, b = bh / H;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int l32 = lane & 31, hl = lane >> 5;
  const int g = lane >> 4, j16 = lane & 15;

  const uint16_t* kbase = static_cast<const uint16_t*>(a.k.data) + (int64_t)b * a.k.sb + (int64_t)h * a.k.sh;
  const uint16_t* vbase = static_cast<const uint16_t*>(a.v.data) + (int64_t)b * a.v.sb + (int64_t)h * a.v.sh;
  SharedTileLoader<NW> kl, vl;
  kl.template init<true>(kbase, a.k.ss, wave, lane);
  vl.template init<false>(vbase, a.v.ss, wave, lane);
  const uint32_t klds = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)&k_s[0][0];
  const uint32_t vlds = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)&v_s[0][0];
  kl.template load<true>(klds, 0, S, wave);

  const int qrow = (ip * NW + wave) * 32 + l32;
  vec8 qf[8];
  {
    const uint16_t* qp = static_cast<const uint16_t*>(a.q.data) + (int64_t)b * a.q.sb + (int64_t)qrow * a.q.ss +
                         (int64_t)h * a.q.sh + 8 * hl;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (qrow < S) {
        qf[s] = *reinterpret_cast<const vec8*>(qp + 16 * s);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[s][e] = (scalar)0.f;
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0)
  __syncthreads();
  if (n > 1) kl.template load<true>(klds + kTileBytes, 1, S, wave);
  vl.template load<false>(vlds, 0, S, wave);

  const int k_row_off = l32 * 256;
  const int k_swzl = l32 & 15;
  const int v_lane_off = (j16 >> 2) * 256 + 8 * (j16 & 1) + 4 * (g >> 1) * 256;
  const int v_c0 = 2 * (g & 1) + ((j16 & 3) >> 1);
  const int v_sl = v_swz_bits(j16 >> 2);

  const float cl2 = a.sm_scale * kLog2e;
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 o[4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[u][r] = 0.f;

  auto qk = [&](f32x16 (&s)[2], const char* kt) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[t][r] = 0.f;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      const int koff = k_row_off + (((2 * d + hl) ^ k_swzl) << 4);
#pragma unroll
      for (int t = 0; t < 2; ++t)
        s[t] = E::mfma(*reinterpret_cast<const vec8*>(kt + t * 32 * 256 + koff), qf[d], s[t]);
    }
  };
  auto fix = [&](f32x16 (&s)[2], int j) {   // key scale and the end of the sequence
    if (KSCALE && j * kBlock < a.ks.n_first) {
      const int lim = a.ks.n_first - j * kBlock;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (32 * t + 8 * (r >> 2) + 4 * hl + (r & 3) < lim) s[t][r] *= a.ks.beta;
    }
    if (j * kBlock + kBlock > S) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (j * kBlock + 32 * t + 8 * (r >> 2) + 4 * hl + (r & 3) >= S) s[t][r] = -INFINITY;
    }
  };
  auto row_max = [&](const f32x16 (&s)[2]) {
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[t][r]);
    return pair_max(mx);
  };
  auto rescale = [&](float mx) {
    const float m_new = fmaxf(m_run, mx * cl2);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run + kRescaleLog2) != 0) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[u][r] *= alpha;
    }
  };
  auto probs = [&](const f32x16 (&s)[2], vec8 (&pf)[2][2]) {
    float rs = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(s[t][r] * cl2 - m_run);
        rs += p;
        pf[t][r >> 3][r & 7] = (scalar)p;
      }
    l_run += rs;
  };
  auto pv = [&](const vec8 (&pf)[2][2], const char* vt) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int cu = (4 * u + v_c0) ^ v_sl;
          const char* lo = vt + (32 * t + 16 * hh) * 256 + v_lane_off + (cu << 4);
          const vec8 vf = E::tr_pair(lo, lo + 8 * 256);
          o[u] = E::mfma(vf, pf[t][hh], o[u]);
        }
  };

  f32x16 s0[2], s1[2];
  qk(s0, k_s[0]);
  fix(s0, 0);
  float mx = row_max(s0);

  // step j (fused): PV of block j, QK^T of block j + 1 beside its softmax
  auto fused = [&](int j, int par, f32x16 (&sc)[2], f32x16 (&sn)[2]) {
    CHORUS_WAIT_LDS_TILES();
    __syncthreads();
    if (j + 2 < n) kl.template load<true>(klds + par * kTileBytes, j + 2, S, wave);
    vl.template load<false>(vlds + (par ^ 1) * kTileBytes, j + 1, S, wave);
    rescale(mx);
    vec8 pf[2][2];
    qk(sn, k_s[par ^ 1]);
    probs(sc, pf);
    if (KSCALE) fix(sn, j + 1);
    pv(pf, v_s[par]);
    mx = row_max(sn);
  };
  int j = 0;
  const int n_full = S / kBlock;
  for (; j + 2 < n_full; j += 2) {
    fused(j, 0, s0, s1);
    fused(j + 1, 1, s1, s0);
  }
  for (; j < n; ++j) {
    const int par = j & 1;
    CHORUS_WAIT_LDS_TILES();
    __syncthreads();
    if (j + 2 < n) kl.template load<true>(klds + par * kTileBytes, j + 2, S, wave);
    if (j + 1 < n) vl.template load<false>(vlds + (par ^ 1) * kTileBytes, j + 1, S, wave);
    rescale(mx);
    vec8 pf[2][2];
    probs(s0, pf);
    pv(pf, v_s[0] + par * kTileBytes);
    if (j + 1 < n) {
      qk(s0, k_s[0] + (par ^ 1) * kTileBytes);
      fix(s0, j + 1);
      mx = row_max(s0);
    }
  }

  const float l_tot = pair_sum(l_run);
  const bool live = l_tot > 0.f;
  const float inv_l = live ? 1.f / l_tot : 0.f;
  if (qrow < S) {
    uint16_t* op = static_cast<uint16_t*>(const_cast<void*>(a.o.data)) + (int64_t)b * a.o.sb +
                   (int64_t)qrow * a.o.ss + (int64_t)h * a.o.sh;
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        scalar v4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v4[e] = (scalar)(o[u][4 * rr + e] * inv_l);
        uint2 packed;
        __builtin_memcpy(&packed, v4, 8);
        *reinterpret_cast<uint2*>(op + 32 * u + 8 * rr + 4 * hl) = packed;
      }
    if (a.lse && hl == 0)
      a.lse[((int64_t)b * H + h) * S + qrow] = live ? (m_run + __builtin_log2f(l_tot)) * kLn2 : -INFINITY;
  }
}

}  // namespace

namespace {
template <bool BF16, bool DENSE, bool KV2, int P>
void launch_16(const AttnArgs& a, hipStream_t st) {
  const dim3 grid(work_grid(a.B * a.H, a.n)), block(128 * P);
  if (a.ks.n_first > 0)
    hipLaunchKernelGGL((attn_fwd_16_kernel<BF16, DENSE, true, KV2, P>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((attn_fwd_16_kernel<BF16, DENSE, false, KV2, P>), grid, block, 0, st, a);
}

// Parts a row's list is split into, at most (short lists use fewer, kSplit2
// and kSplit4).  A workgroup with P parts takes P times the LDS, so a CU holds
// four (P = 1), two or one of them; a split pays while the rows alone leave
// that room empty.  Rows are dealt to the XCDs by whole (request, head) units,
// so what counts is the fullest XCD's share against its 32 CUs.  One row per CU
// or fewer: four parts (4,096 tokens, 2 heads, all blocks listed: 41 us, two
// parts 48, unsplit 78).  Two per CU or fewer: two parts (12 heads x 20 blocks,
// 40 rows on XCDs 0..3: 27 us, unsplit 37, four parts 35).  Beyond that the rows
// fill the chip (12 heads x 42 blocks, 84 rows: 85 us, unsplit 77).  Dense calls
// of that size run here too, 3,120 tokens x 4 heads: 35 us against 53 with
// attn_dense_16_kernel.  The rule reads sizes only, so a full mask and no mask
// take the same split.
int list_parts(const AttnArgs& a) {
  if (a.n < kSplit2) return 1;
  const unsigned rows = work_grid(a.B * a.H, a.n) / kNumXcd;
  return rows <= 32 ? 4 : rows <= 64 ? 2 : 1;
}

template <bool BF16, int NW>
void launch_dense_nw(const AttnArgs& a, hipStream_t st) {
  const int np = (a.S + 32 * NW - 1) / (32 * NW);
  const dim3 grid(work_grid(a.B * a.H, np)), block(64 * NW);
  if (a.ks.n_first > 0)
    hipLaunchKernelGGL((attn_dense_16_kernel<BF16, true, NW>), grid, block, 0, st, a, np);
  else
    hipLaunchKernelGGL((attn_dense_16_kernel<BF16, false, NW>), grid, block, 0, st, a, np);
}

// Dense calls whose rows are not split.  The masked kernel's workgroups (two
// waves) while the dense kernel's larger ones fill the chip worse than its
// pipeline gains: below 4 kv blocks (1,000 heads x 3 blocks 47-51 us against 54)
// and, for short sequences, up to 96 rows on the fullest XCD (80 heads x 9
// blocks 26.6 against 27.7, 128 x 5 18.0 against 19.1, 24 x 28 56.8 against
// 56.5).  Otherwise the dense kernel: more waves share a tile, fewer leave
// smaller pieces for the CUs (each CU holds eight such waves).  With long
// sequences and four rounds of eight-wave workgroups over the 256 CUs the
// sharing wins (480p 14B: 17.9 against 19.0 ms; 256 heads x 32 blocks 565
// against 597 us); below that the uneven last round costs more (S = 8,215, 3
// heads: 0.204 ms with eight waves, 0.164 with four), and on short sequences the
// waves past the end (1,000 heads x 5 blocks: 154 us against 111, x 13 520
// against 462).  Two waves were slower even there (0.236 ms).
template <bool BF16>
void launch_dense(const AttnArgs& a, hipStream_t st) {
  const unsigned rows = work_grid(a.B * a.H, a.n) / kNumXcd;
  const int64_t rows32 = (int64_t)a.B * a.H * ((a.S + 31) / 32);
  if (a.n < 4 || (a.n < 32 && rows <= 96))
    launch_16<BF16, true, false, 1>(a, st);
  else if (a.n >= 64 && rows32 >= 4 * 256 * 8)
    launch_dense_nw<BF16, 8>(a, st);
  else
    launch_dense_nw<BF16, 4>(a, st);
}

template <bool BF16, bool DENSE, bool KV2>
void launch_parts(const AttnArgs& a, int parts, hipStream_t st) {
  if (parts == 4)
    launch_16<BF16, DENSE, KV2, 4>(a, st);
  else
    launch_16<BF16, DENSE, KV2, 2>(a, st);
}

template <bool BF16>
void launch_16_mask(const AttnArgs& a, hipStream_t st) {
  const int parts = list_parts(a);
  const bool kv2 = a.kv_block == 2 * kBlock;
  if (a.row_ptr == nullptr) {
    if (parts > 1)
      launch_parts<BF16, true, false>(a, parts, st);
    else
      launch_dense<BF16>(a, st);
  } else if (parts > 1) {
    kv2 ? launch_parts<BF16, false, true>(a, parts, st) : launch_parts<BF16, false, false>(a, parts, st);
  } else {
    kv2 ? launch_16<BF16, false, true, 1>(a, st) : launch_16<BF16, false, false, 1>(a, st);
  }
}
}  // namespace

hipError_t launch_attn_fwd_16(chorus_dtype dt, const AttnArgs& a, hipStream_t st) {
  if (dt == CHORUS_BF16)
    launch_16_mask<true>(a, st);
  else
    launch_16_mask<false>(a, st);
  return hipGetLastError();
}

}  // namespace chorus

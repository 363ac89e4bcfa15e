// True block attention mass and mask coverage (Chorus II Sec. 3.2 "Mask
// Caching and Retrieval": a historical request's masks are selected from its
// own attention map; Sec. 3.2 Obs. 1: a mask is judged by the share of a
// request's attention mass that falls inside its blocks).
//
// block_mass_kernel: one workgroup per (request, head, run of four q-blocks),
// eight waves of 32 queries that share every K tile.  For every kv block j it
// recomputes S^T = K_j Q^T with v_mfma_f32_32x32x16 (as the attention kernel
// does: each lane holds 32 scores of one query), turns the scores into the
// dense attention probabilities with the log-sum-exp of the dense forward
// pass, p = 2^(s log2(e) sm_scale - lse log2(e)), and sums them over the
// block's queries and keys: mass[i, j] = sum / |T_i|.  For kv blocks of 128
// tokens the sums of the two 64-key halves are added before the division.
//
// Bound by the exponentials and adds beside the products (96 vector
// instructions, 32 of them half-rate, per 16 MFMAs of a wave), so the kernel
// is laid out for waves in flight: at most 128 registers, four waves per SIMD
// (two workgroups of eight waves per CU), K tiles double-buffered by direct
// global -> LDS loads, one barrier per kv block.  The per-lane sums of four
// kv blocks are reduced over the wave together (ten instructions instead of
// four times six LDS-crossbar steps) and sixteen blocks' masses are written
// together (64-byte runs).  480p 14B (S = 32,760, 40 heads), bf16: 9.8-10.2 ms,
// 1,080-1,125 TFLOP/s of QK^T, matrix cores busy 57 % of the cycles, against
// 18.9 ms for the earlier workgroup of one q-block (two waves, a shuffle
// reduction and a four-byte store per kv block).
// Four waves of the same code: 10.0 ms; three waves per SIMD 10.3 ms; QK^T of
// the next block issued beside this block's exponentials (a second score
// tile, two waves per SIMD) 10.8 ms.
#include <type_traits>

#include "attn_common.h"

namespace chorus {
namespace {

constexpr int kMassTile = kBlock * kHeadDim * 2;   // 16 KB per 16-bit K tile

__device__ inline int km_swz(int r, int c) { return c ^ (r & 15); }

template <bool BF16>
struct MassElt;
template <>
struct MassElt<true> {
  using vec8 = bf16x8;
  using scalar = __bf16;
  static __device__ inline f32x16 mfma(vec8 a, vec8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct MassElt<false> {
  using vec8 = f16x8;
  using scalar = _Float16;
  static __device__ inline f32x16 mfma(vec8 a, vec8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};

constexpr int kMassWaves = 8;            // waves of 32 queries: four q-blocks share each K tile
constexpr int kMassGroup = 16;           // kv blocks whose sums are written together

// This wave's share of a 64 x 128 K tile: instruction u fills LDS rows
// 32u + 4 wave .. + 3 (lane-linear), each lane fetching the global chunk that
// the swizzle places at its slot; rows past the sequence end re-read row S - 1.
__device__ inline void load_k_share(uint32_t lds, const char* base, uint32_t ss, uint32_t off, int j, int S, int wave,
                                    int lane) {
  if (j * kBlock + kBlock <= S) {
    const char* rowj = base + (int64_t)j * kBlock * ss;
#pragma unroll
    for (int u = 0; u < 16 / kMassWaves; ++u)
      dma16(lds + (kMassWaves * u + wave) * 1024, rowj + (int64_t)(4 * kMassWaves * u) * ss, off);
  } else {
    // computed here each time: kept across the loop they would cost registers
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int u = 0; u < 16 / kMassWaves; ++u) {
      const int r = 4 * kMassWaves * u + 4 * wave + (lane >> 4);
      const int tok = min(j * kBlock + r, S - 1);
      dma16(lds + (kMassWaves * u + wave) * 1024, base, (uint32_t)tok * ss + (uint32_t)km_swz(r, lane & 15) * 16);
    }
  }
}

// Sums of four per-lane values over the wave: lane row r (16 lanes) ends with
// the sum of v[2 (r & 1) + (r >> 1)] at each of its lanes.  The two swaps
// halve the number of live values, so four sums cost ten vector instructions.
__device__ inline float wave_sum4(const float (&v)[4]) {
  auto halves = [](float x, float y) {   // lanes 0..31: x over both halves, 32..63: y
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  };
  const float a = halves(v[0], v[1]), b = halves(v[2], v[3]);
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  float s = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  auto dpp = [](float x, auto ctrl) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(x), decltype(ctrl)::value, 0xF, 0xF,
                                                              false));
  };
  s += dpp(s, std::integral_constant<int, 0xB1>{});    // quad_perm [1, 0, 3, 2]
  s += dpp(s, std::integral_constant<int, 0x4E>{});    // quad_perm [2, 3, 0, 1]
  s += dpp(s, std::integral_constant<int, 0x141>{});   // row_half_mirror
  s += dpp(s, std::integral_constant<int, 0x140>{});   // row_mirror
  return s;
}

template <bool BF16>
__global__ __launch_bounds__(64 * kMassWaves) __attribute__((amdgpu_waves_per_eu(4, 4)))
void block_mass_kernel(TensorArg q, TensorArg k, const float* __restrict__ lse, int B, int S, int H, int n, int np,
                       float sm_scale, KeyScale ks, bool kv2, float* __restrict__ mass) {
  using E = MassElt<BF16>;
  using vec8 = typename E::vec8;
  using scalar = typename E::scalar;
  __shared__ __attribute__((aligned(1024))) char k_s[2][kMassTile];
  __shared__ float red[2][kMassWaves][kMassGroup];

  const int item = work_item(nullptr, B * H, np);
  if (item < 0) return;
  const int ip = item % np;
  const int bh = item / np;
  const int h = bh % H, b = bh / H;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int l32 = lane & 31, hl = lane >> 5;

  const char* kbase = static_cast<const char*>(k.data) + ((int64_t)b * k.sb + (int64_t)h * k.sh) * 2;
  const uint32_t kss = (uint32_t)(k.ss * 2);
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)&k_s[0][0];
  const int r0 = 4 * wave + (lane >> 4);
  const uint32_t koff_lane = (uint32_t)r0 * kss + (uint32_t)km_swz(r0, lane & 15) * 16;
  load_k_share(lds0, kbase, kss, koff_lane, 0, S, wave, lane);

  const int qrow = (ip * kMassWaves + wave) * 32 + l32;
  const bool q_valid = qrow < S;
  vec8 qf[8];
  {
    const uint16_t* qp = static_cast<const uint16_t*>(q.data) + (int64_t)b * q.sb + (int64_t)qrow * q.ss +
                         (int64_t)h * q.sh + 8 * hl;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (q_valid) {
        qf[s] = *reinterpret_cast<const vec8*>(qp + 16 * s);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[s][e] = (scalar)0.f;
      }
    }
  }
  const float lse2 = q_valid ? lse[(int64_t)bh * S + qrow] * kLog2e : 0.f;
  const float cl2 = sm_scale * kLog2e;
  __builtin_amdgcn_s_waitcnt(0xF70);   // vmcnt(0): Q and the first K tile

  const int k_row_off = l32 * 256;
  const int k_swzl = l32 & 15;
  // kv2: kv blocks of 128 tokens, each the sum of two 64-token halves
  const int nk = kv2 ? (n + 1) / 2 : n;

  // writes the sums of blocks g kMassGroup .. + 15 (all waves have published)
  auto flush = [&](int g) {
    int t = tid;
    asm volatile("" : "+v"(t));   // as in fix: addresses are not kept across the loop
    const int x = t & (kMassGroup - 1), qb = t / kMassGroup;
    const int i = ip * (kMassWaves / 2) + qb, j = g * kMassGroup + x;
    if (qb >= kMassWaves / 2 || i >= n || j >= n || (kv2 && (x & 1))) return;
    const float(*r)[kMassGroup] = &red[g & 1][2 * qb];
    float v = r[0][x] + r[1][x];
    if (kv2 && j + 1 < n) v += r[0][x + 1] + r[1][x + 1];
    mass[((int64_t)bh * n + i) * nk + (kv2 ? j >> 1 : j)] = v / (float)min(kBlock, S - i * kBlock);
  };

  auto qk = [&](f32x16 (&sacc)[2], const char* kt) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[t][r] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int koff = k_row_off + (((2 * s + hl) ^ k_swzl) << 4);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const vec8 kf = *reinterpret_cast<const vec8*>(kt + t * 32 * 256 + koff);
        sacc[t] = E::mfma(kf, qf[s], sacc[t]);
      }
    }
  };
  auto fix = [&](f32x16 (&sacc)[2], int j) {
    int hl4 = 4 * hl;                     // key indices are computed here each time:
    asm volatile("" : "+v"(hl4));         // kept across the loop they would cost registers
    // first-frame keys (Eq. 1): their logits count beta times
    if (j * kBlock < ks.n_first) {
      const int lim = ks.n_first - j * kBlock;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (32 * t + 8 * (r >> 2) + hl4 + (r & 3) < lim) sacc[t][r] *= ks.beta;
    }
    // keys past the end have probability 2^-inf = 0
    if (j * kBlock + kBlock > S) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (j * kBlock + 32 * t + 8 * (r >> 2) + hl4 + (r & 3) >= S) sacc[t][r] = -INFINITY;
    }
  };
  auto prob_sum = [&](const f32x16 (&sacc)[2]) {
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(sacc[t][r] * cl2 - lse2);
    return sum;
  };
  auto publish = [&](const float (&acc)[4], int j0) {
    const float s = wave_sum4(acc);
    const int row = lane >> 4;
    if ((lane & 15) == 0) red[(j0 / kMassGroup) & 1][wave][j0 % kMassGroup + 2 * (row & 1) + (row >> 1)] = s;
  };

  for (int j0 = 0; j0 < n; j0 += 4) {
    float acc[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      acc[x] = 0.f;
      const int j = j0 + x;
      if (j >= n) continue;
      CHORUS_WAIT_LDS_TILES();   // K_j landed; the sums this wave published are in LDS
      __syncthreads();
      if (j + 1 < n) load_k_share(lds0 + ((x + 1) & 1) * kMassTile, kbase, kss, koff_lane, j + 1, S, wave, lane);
      if (x == 0 && j0 > 0 && j0 % kMassGroup == 0) flush(j0 / kMassGroup - 1);
      f32x16 sacc[2];
      qk(sacc, k_s[x & 1]);
      if (j * kBlock < ks.n_first || j * kBlock + kBlock > S) fix(sacc, j);
      acc[x] = q_valid ? prob_sum(sacc) : 0.f;
    }
    publish(acc, j0);
  }
  CHORUS_WAIT_LDS_TILES();
  __syncthreads();
  flush((n - 1) / kMassGroup);
}

// Coverage of a mask: one workgroup of sixteen waves per (request, head), of
// four where there are no more than sixteen q-blocks.  Sixteen lanes take a row,
// so 64 rows are in flight, the ids are read in runs of sixteen, four of a
// lane's ids (then their masses) at a time, and the next row's bounds ahead;
// each lane adds its kept masses weighted by the row's valid tokens in float64.
// Bound by the latency of the dependent reads (id, then mass) over few
// workgroups: 480p 14B at 15 % (40 heads x 512 rows of 77 ids) takes 35 us,
// against 164 us with one thread per row and 256 threads.  Waves without a row
// would only cost their start (1,000 units of 13 rows: 5.2 us with sixteen,
// 3.7 with four).
template <int kCovThreads>
__global__ __launch_bounds__(kCovThreads) void coverage_kernel(const int32_t* __restrict__ row_ptr,
                                                               const int32_t* __restrict__ col_idx, int mask_batch,
                                                               const float* __restrict__ mass, int S, int H, int n,
                                                               int nk, double* __restrict__ coverage) {
  __shared__ double red[kCovThreads / 64];
  const int h = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, sub = tid & 15;
  const float* mb = mass + ((int64_t)b * H + h) * n * nk;
  double acc = 0.0;
  const int64_t r0 = ((int64_t)(mask_batch > 1 ? b : 0) * H + h) * n;
  constexpr int kStep = kCovThreads / 16;
  int i = tid >> 4;
  int beg = i < n ? row_ptr[r0 + i] : 0, end = i < n ? row_ptr[r0 + i + 1] : 0;
  while (i < n) {
    const int next = i + kStep;   // its bounds are read while this row's ids and masses are
    const int beg_n = next < n ? row_ptr[r0 + next] : 0, end_n = next < n ? row_ptr[r0 + next + 1] : 0;
    const float* mrow = mb + (int64_t)i * nk;
    double row = 0.0;
    for (int e = beg + sub; e < end; e += 64) {
      int j[4];
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) j[u] = e + 16 * u < end ? col_idx[e + 16 * u] : -1;
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = j[u] >= 0 && j[u] < nk ? mrow[j[u]] : 0.f;
#pragma unroll
      for (int u = 0; u < 4; ++u) row += (double)v[u];
    }
    acc += row * (double)min(kBlock, S - i * kBlock);
    i = next;
    beg = beg_n;
    end = end_n;
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < kCovThreads / 64; ++w) t += red[w];
    coverage[(int64_t)b * H + h] = t / (double)S;
  }
}

}  // namespace

hipError_t launch_block_mass(chorus_dtype dt, TensorArg q, TensorArg k, const float* lse, int B, int S, int H,
                             float sm_scale, KeyScale ks, int kvb, float* mass, hipStream_t st) {
  const bool kv2 = kvb == 2 * kBlock;
  const int n = blocks_of(S);
  const int np = (n + kMassWaves / 2 - 1) / (kMassWaves / 2);
  const dim3 grid(work_grid(B * H, np)), block(64 * kMassWaves);
  if (dt == CHORUS_BF16)
    hipLaunchKernelGGL(block_mass_kernel<true>, grid, block, 0, st, q, k, lse, B, S, H, n, np, sm_scale, ks, kv2, mass);
  else
    hipLaunchKernelGGL(block_mass_kernel<false>, grid, block, 0, st, q, k, lse, B, S, H, n, np, sm_scale, ks, kv2,
                       mass);
  return hipGetLastError();
}

hipError_t launch_coverage(const int32_t* row_ptr, const int32_t* col_idx, int mask_batch, const float* mass, int B,
                           int S, int H, int kvb, double* coverage, hipStream_t st) {
  const int n = blocks_of(S), nk = (S + kvb - 1) / kvb;
  auto kernel = n <= 16 ? coverage_kernel<256> : coverage_kernel<1024>;
  hipLaunchKernelGGL(kernel, dim3(H, B), dim3(n <= 16 ? 256 : 1024), 0, st, row_ptr, col_idx, mask_batch, mass, S, H, n,
                     nk, coverage);
  return hipGetLastError();
}

}  // namespace chorus

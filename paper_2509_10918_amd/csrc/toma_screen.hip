// Which merge weights can be nonzero at all: a bound on every logit of the global merge from a 4-bit product.
//
// The merge weights are a softmax over all destinations of a sample, at a small temperature: a source's largest logit
// stands hundreds of units above nearly all others, whose weights are then below e^-110 and exact zeros.  Which tiles of 32 sources x 16 destinations hold anything else is found without the full product:
//   k_fp4_bounds  per token: the row rounded to 4-bit floats (e2m1, one scale per token) with the exact norm of what
//                 the rounding dropped; per source a lower bound on its largest logit, the exact product with the
//                 destinations of its own selection region.
//   k_screen      the product of the rounded rows on the 4-bit matrix cores (four times the bf16 rate, a quarter of the
//                 bytes) and, per tile, one bit: can any logit come within the gap of its source's largest?
//                     <x_s, x_j> <= <q_s, q_j> + |x_s - q_s| |x_j| + |q_s| |x_j - q_j|      (Cauchy-Schwarz, twice)
//                 It also fills A with zeros: its own work leaves the memory idle.
// The weights kernel then computes the marked tiles exactly and writes them over the zeros (toma_merge.hip).  A tile
// left out holds only weights that underflow, so A, Z and all that follows are those of the full product; where the
// softmax is not sharp every tile is marked and everything is computed.
// 128 x 128 grid (two samples, 640 channels, half kept): statistics and write pass of the full product 645 us, these
// kernels and the exact one 65 + 126 + 60 us, of which writing A (537 MB) takes about 110.
#include "toma_gemm.h"
#include "toma_internal.h"
#include "toma_region.h"
#include "toma_weights.h"

namespace toma {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// A logit so far (in units of the logit) below a lower bound of its source's largest gives a zero weight: e^-110 is
// below half of the smallest positive number of either type; the rest covers the fp32 rounding of the logits.
constexpr float kScreenGap = 118.0f;
// Sources with scale |x|^2 below this do not screen: with the bound's errors (about a fifth of |x|^2) even a destination
// at a right angle is within the gap.  Blocks of such sources mark every tile without any product.
constexpr float kScreenSoft = 168.0f;
// The two error terms of the bound as one product E_s F_j: sqrt(r_s^2 + (k n_s)^2) sqrt(n_j^2 + (r_j / k)^2) bounds
// r_s n_j + n_s r_j for any k > 0 and equals it where r / n = k, which is what 4-bit rounding gives (0.09 to 0.14).
// The third pair of terms, n_s n_j / 4096, covers the rounding of the products that the bound stands for.
constexpr float kRoundRatio = 0.12f;

// Eight consecutive channels of a row as fp32.
__device__ __forceinline__ void load8(float (&x)[8], const bf16_t *p) {
  const Pkt q = pkt_load(p);
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const uint32_t u = q.v[i];
    x[2 * i] = __builtin_bit_cast(float, u << 16);
    x[2 * i + 1] = __builtin_bit_cast(float, u & 0xffff0000u);
  }
}
// Does `p` hold in all 512 threads?  One barrier (what __syncthreads_and does takes two); `slot` is used once.
__device__ __forceinline__ bool block_all(bool p, uint32_t (&slot)[8]) {
  const uint32_t all = __all(p);
  if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = all;
  __syncthreads();
  const u32x4 a = *reinterpret_cast<const u32x4 *>(&slot[0]), b = *reinterpret_cast<const u32x4 *>(&slot[4]);
  return __builtin_amdgcn_readfirstlane((int)(a[0] & a[1] & a[2] & a[3] & b[0] & b[1] & b[2] & b[3])) != 0;
}
// operand of a product of 4-bit floats: 32 of them in the first four registers
__device__ __forceinline__ i32x8 four_bit(const u32x4 &q) { return (i32x8){(int)q[0], (int)q[1], (int)q[2], (int)q[3], 0, 0, 0, 0}; }

// One workgroup (8 waves) per 32 sources in region order.  What bounds it is the chain of dependent loads (rows and
// indices, then the rows of the products, three K steps ahead).
// q4: rows of kb bytes (64 per 128 channels, the rest of the last 128 zeros), in grid order of the tokens;
// src, dst: per token (grid order) the two numbers k_screen needs of it as a source and as a destination.
__global__ __launch_bounds__(512) void k_fp4_bounds(const RegionView<bf16_t> v, const int32_t *__restrict__ idx, float scale,
                                                    int n_loc, int d_loc, uint8_t *__restrict__ q4, int kb,
                                                    float2 *__restrict__ src, float2 *__restrict__ dst,
                                                    int2 *__restrict__ order) {
  typedef bf16_t T;
  __shared__ __align__(1024) WeightsLds<T> lds;
  __shared__ float best[8][32], enorm[32], sscale[32];
  __shared__ int ids[2048];
  __shared__ __align__(16) uint32_t all_soft[8];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int blocks = (v.N + 31) / 32;
  const int work = xcd_remap(blockIdx.x, gridDim.x);
  const int b = work / blocks, m0 = (work - b * blocks) * 32, C = v.C;
  const T *Xb = v.X + (size_t)b * v.N * C;

  auto dest = [&](int j) {
    const int t = idx[(size_t)b * v.D + j];
    return t < 0 ? 0 : (t >= v.N ? v.N - 1 : t);
  };
  // ---- the destinations of a region in grid order: every workgroup ranks a share of its region's ----
  // (pick order scatters neighbours over a region's tiles: with tiles of it, twice as many are marked)
  for (int p = m0 / n_loc; p * n_loc < min(m0 + 32, v.N); p++) {
    const int lo = max(m0 - p * n_loc, 0), hi = min(min(m0 + 32, v.N) - p * n_loc, n_loc);
    const int ja = lo * d_loc / n_loc, jb = hi * d_loc / n_loc;
    for (int j = tid; j < d_loc; j += 512) ids[j] = dest(p * d_loc + j);
    __syncthreads();
    for (int j = ja + (tid >> 5); j < jb; j += 16) {  // 32 lanes count the destinations before j
      const int t = ids[j];
      int rank = 0;
      for (int k = tid & 31; k < d_loc; k += 32) rank += ids[k] < t || (ids[k] == t && k < j) ? 1 : 0;
#pragma unroll
      for (int m = 1; m < 32; m <<= 1) rank += __shfl_xor(rank, m, 32);
      if ((tid & 31) == 0) order[(size_t)b * v.D + p * d_loc + rank] = make_int2(t, p * d_loc + j);
    }
    __syncthreads();
  }
  // ---- rows to 4 bits, norms: 16 lanes per row, 128 channels per step (2 kb of them with the padding) ----
  bool soft;
  {
    const int mr = 4 * w + g;  // this lane's row of the block
    const bool live = m0 + mr < v.N;
    const int t = v.token(0, min(m0 + mr, v.N - 1)), steps = kb / 64;
    const T *row = Xb + (size_t)t * C + 8 * c;
    constexpr int NB = 5;  // steps whose loads are in flight together
    float amax = 0.f;
    bool bad = false;  // a NaN, which a maximum would drop
    auto batch = [&](int i0, auto &&use) {
      float x[NB][8];
#pragma unroll
      for (int u = 0; u < NB; u++) load8(x[u], row + min(128 * (i0 + u), C - 8 - 8 * c));  // (a row is at least as long)
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < NB; u++) {
        const int ch = 128 * (i0 + u) + 8 * c;
        if (i0 + u < steps) use(x[u], ch, ch < C);
      }
    };
    for (int i = 0; i < steps; i += NB)
      batch(i, [&](const float (&x)[8], int, bool in) {
        if (!in) return;
#pragma unroll
        for (int u = 0; u < 8; u++) { amax = fmaxf(amax, fabsf(x[u])); bad |= x[u] != x[u]; }
      });
    amax = row16_max_f32(amax);
    bad = row16_max_f32(bad ? 1.f : 0.f) > 0.f || !(amax < 1e18f);
    // (rows too small or too large for the arithmetic below round to zero and are all remainder)
    const bool plain = amax > 1e-18f && !bad;
    const float up = plain ? 6.0f / amax : 0.f, down = plain ? amax / 6.0f : 1.f;
    float n2 = 0.f, r2 = 0.f;
    uint8_t *out = q4 + ((size_t)b * v.N + t) * kb;
    for (int i = 0; i < steps; i += NB)
      batch(i, [&](const float (&x)[8], int ch, bool in) {
        uint32_t q = 0;
        if (in && plain) {
          q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, x[0] * up, x[1] * up, 1.0f, 0);
          q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, x[2] * up, x[3] * up, 1.0f, 1);
          q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, x[4] * up, x[5] * up, 1.0f, 2);
          q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, x[6] * up, x[7] * up, 1.0f, 3);
        }
        if (in) {
          const f32x2 d0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(q, 1.0f, 0), d1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(q, 1.0f, 1);
          const f32x2 d2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(q, 1.0f, 2), d3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(q, 1.0f, 3);
          const float d[8] = {d0[0], d0[1], d1[0], d1[1], d2[0], d2[1], d3[0], d3[1]};
#pragma unroll
          for (int u = 0; u < 8; u++) {
            n2 = fmaf(x[u], x[u], n2);
            const float e = fmaf(-d[u], down, x[u]);
            r2 = fmaf(e, e, r2);
          }
        }
        if (live) *reinterpret_cast<uint32_t *>(out + ch / 2) = q;
      });
    n2 = row16_sum_f32(n2);
    r2 = row16_sum_f32(r2);
    soft = !live || scale * n2 < kScreenSoft;
    if (c == 0 && live) {
      constexpr float k2 = kRoundRatio * kRoundRatio, tiny = 1.0f / 4096;
      const float grow = bad ? __builtin_inff() : 1.0001f / down;  // (also covers the rounding of these few operations)
      // (|q_s| |x_j - q_j| with |q_s| <= |x_s| + r_s; the first factor keeps both)
      const float q = sqrtf(n2) + sqrtf(r2);
      enorm[mr] = sqrtf(r2 + k2 * q * q + tiny * n2) * grow;
      sscale[mr] = bad ? __builtin_nanf("") : 1.0f / down;
      dst[(size_t)b * v.N + t] = make_float2(sqrtf(n2 + r2 / k2 + tiny * n2) * grow, 1.0f / down);
    }
  }

  if (block_all(soft, all_soft)) {
    if (tid < 32 && m0 + tid < v.N) src[(size_t)b * v.N + v.token(0, m0 + tid)] = make_float2(enorm[tid], __builtin_nanf(""));
    return;
  }

  // ---- lower bound of each source's largest product: the destinations of its own region ----
  // (a block that lies in two regions: all of them for every source - any destination's product is a bound)
  const int p0 = m0 / n_loc, p1 = min(m0 + 31, v.N - 1) / n_loc, d0 = p0 * d_loc, nd = (p1 - p0 + 1) * d_loc;
  const int nt = (nd + 15) / 16;
  float mx[2][4];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int r = 0; r < 4; r++) mx[i][r] = -__builtin_inff();
  auto run = [&](auto nj_c) {
    constexpr int NJ = decltype(nj_c)::value;
    for (int e0 = 0; e0 < nt; e0 += 8 * NJ) {
      f32x4 acc[2][NJ];
      weights_products<T, NJ>(acc, lds, v, b, 0, m0, [&](int j, int r) { return dest(d0 + min(16 * (e0 + 8 * j + w) + r, nd - 1)); });
#pragma unroll
      for (int j = 0; j < NJ; j++)  // (a tile past the last repeats a destination)
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int r = 0; r < 4; r++)  // (NaN stays)
            mx[i][r] = __builtin_elementwise_maximum(mx[i][r], acc[i][j][r]);
    }
  };
  if (nt > 16) run(std::integral_constant<int, 4>{});
  else if (nt > 8) run(std::integral_constant<int, 2>{});
  else run(std::integral_constant<int, 1>{});
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      float m = mx[i][r];
#pragma unroll
      for (int k = 1; k < 16; k <<= 1) m = __builtin_elementwise_maximum(m, wave_xor_f32(m, k));
      if (c == 0) best[w][16 * i + 4 * g + r] = m;
    }
  __syncthreads();
  if (tid < 32 && m0 + tid < v.N) {
    float lb = best[0][tid];
#pragma unroll
    for (int q = 1; q < 8; q++) lb = __builtin_elementwise_maximum(lb, best[q][tid]);
    // (a bound that is no finite number screens nothing)
    float t = lb - kScreenGap / scale - 1e-4f * fabsf(lb);
    if (!(fabsf(t) < 1e30f)) t = __builtin_nanf("");
    src[(size_t)b * v.N + v.token(0, m0 + tid)] = make_float2(enorm[tid], t * sscale[tid]);
  }
}

// k_screen: 8 waves, as SG groups of 32 sources (their fragments in registers for the whole kernel) x 8 / SG shares of the
// destination tiles; a chunk of destinations streams through two LDS buffers in stages of SD rows.  With q scaled to integers of the 4-bit grid the bound
//     s_s s_j <q_s, q_j> + E_s F_j < T_s      becomes      <q_s, q_j> + e_s f_j - t_s i_j < 0.
// act: one byte per (sample, block of 32 sources, 128 destinations).
// What bounds it: the zeros of A (128 x 128 grid: 537 MB, about 110 us); its own products take about half of that.
template <int KC, int SD, int SG>
__global__ __launch_bounds__(512) void k_screen(const RegionView<bf16_t> v, const int2 *__restrict__ order,
                                                const uint8_t *__restrict__ q4, int kc, const float2 *__restrict__ src,
                                                const float2 *__restrict__ dst, bf16_t *__restrict__ A, uint8_t *__restrict__ act,
                                                int act_row, int octets, int chunks, int tiles) {
  constexpr int NTS = SD / 16, DG = 8 / SG;  // destination tiles per stage, shares of them
  constexpr int TPW = NTS / DG, TU = TPW < 2 ? 1 : 2;  // tiles of a wave per stage, at a time
  constexpr int MS = 32 * SG;                // sources per workgroup
  __shared__ __align__(1024) uint8_t Bs[2][NTS * KC * 1024];  // [tile][128 channels][lane] fragments
  __shared__ __align__(16) float fj[1024], ij[1024];  // the chunk's destinations: at most eight times 128
  __shared__ int off[1024];
  __shared__ uint32_t marks[SG][8];              // [sources][128 destinations]
  __shared__ __align__(16) uint32_t all_soft[8];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int work = xcd_remap(blockIdx.x, gridDim.x);
  const int b = work / (chunks * tiles), rest = work - b * chunks * tiles, mt = rest / chunks, ck = rest - mt * chunks;
  const int m0 = mt * MS, kb = kc * 64, N = v.N, D = v.D;
  const int span = octets * 128, j0 = ck * span, j1 = min(j0 + span, D);
  const uint8_t *qb = q4 + (size_t)b * N * kb;
  const int2 *ib = order + (size_t)b * D;
  int jt[2];  // this thread's destinations of the chunk (requested first: others' addresses follow from them)
#pragma unroll
  for (int u = 0; u < 2; u++) {
    jt[u] = ib[min(j0 + min(tid + 512 * u, span - 1), D - 1)].x;
  }
  // sources as right operands: lane = source 16 i + c, 32 channels of group g
  const int sg = w % SG, dg = w / SG, mw = m0 + 32 * sg;
  u32x4 fs[2][KC];
  float es[2], ts[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int t = v.token(0, min(mw + 16 * i + c, N - 1));
    const float2 e = src[(size_t)b * N + t];
    es[i] = e.x;
    ts[i] = -e.y;
#pragma unroll
    for (int k = 0; k < KC; k++) fs[i][k] = *reinterpret_cast<const u32x4 *>(qb + (size_t)t * kb + min(k, kc - 1) * 64 + 16 * g);
  }
  const int nstage = (j1 - j0 + SD - 1) / SD, pieces = NTS * kc;
  for (int j = tid; j < span; j += 512) {  // (past the end: the last destination again)
    const int t = jt[(j - tid) >> 9];
    const float2 e = dst[(size_t)b * N + t];
    off[j] = t * kb;
    fj[j] = e.x;
    ij[j] = e.y;
  }
  wait_vmcnt<0>();
  // (no source here screens anything: every tile is marked, and whoever computes them writes all of A)
  if (block_all(ts[0] != ts[0] && ts[1] != ts[1], all_soft)) {
    if (tid < SG * octets) {
      const int r = tid / octets, o = tid - r * octets, n = min((j1 - j0 - 128 * o + 15) / 16, 8);
      if (m0 + 32 * r < N && n > 0)
        act[((size_t)b * ((N + 31) / 32) + m0 / 32 + r) * act_row + ck * octets + o] = (uint8_t)((1 << n) - 1);
    }
    return;
  }
  auto issue = [&](int st) {
    for (int p = w; p < pieces; p += 8) {  // piece: tile p / kc, channels 128 (p % kc) .. + 127
      const int tile = p / kc, k = p - tile * kc;
      load_to_lds16_at(qb + off[st * SD + 16 * tile + c] + k * 64 + 16 * g, lds_addr_of(&Bs[st & 1][(tile * KC + k) * 1024]));
    }
  };
  if (tid < SG * 8) marks[tid >> 3][tid & 7] = 0;
  // Zeros for this block of A, a stage's rows per stage: after its loads, so that the wait below (memory operations
  // count down in order) leaves them in flight.
  constexpr int EPC = 8, CPR = MS / EPC, ZS = SD * CPR / 512;  // packets per row, stores per thread
  const u32x4 zero = {0u, 0u, 0u, 0u};
  const int zm = min(m0 + (tid % CPR) * EPC, N - EPC), zr = tid / CPR;  // (past the end: the last packet again)
  issue(0);
  for (int st = 0; st < nstage; st++) {
    // the stage has landed; the other one is free
    if (st == 0) wait_vmcnt<0>(); else wait_vmcnt<ZS>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (st + 1 < nstage) issue(st + 1);
#pragma unroll
    for (int u = 0; u < ZS; u++)
      *reinterpret_cast<u32x4 *>(A + ((size_t)b * D + min(j0 + st * SD + zr + u * (512 / CPR), D - 1)) * N + zm) = zero;
    const uint8_t *bs = Bs[st & 1];
#pragma unroll
    for (int t2 = dg * TPW; t2 < (dg + 1) * TPW; t2 += TU) {  // (two tiles at a time: four chains of products)
      f32x4 acc[TU][2];
#pragma unroll
      for (int u = 0; u < TU; u++)
#pragma unroll
        for (int i = 0; i < 2; i++) acc[u][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KC; k++) {
        if (k < kc) {  // (uniform)
#pragma unroll
          for (int u = 0; u < TU; u++) {
            const u32x4 q = *reinterpret_cast<const u32x4 *>(bs + ((t2 + u) * KC + k) * 1024 + 16 * lane);
#pragma unroll
            for (int i = 0; i < 2; i++)
              acc[u][i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(four_bit(q), four_bit(fs[i][k]), acc[u][i], 4, 4, 0,
                                                                           0x7f7f7f7f, 0, 0x7f7f7f7f);
          }
        }
      }
      // lane: source c of half i, destinations 4 g + r of the tile
#pragma unroll
      for (int u = 0; u < TU; u++) {
        const int at = st * SD + 16 * (t2 + u) + 4 * g;
        const f32x4 f = *reinterpret_cast<const f32x4 *>(&fj[at]), q = *reinterpret_cast<const f32x4 *>(&ij[at]);
        float top = -1.0f;
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int r = 0; r < 4; r++)  // (NaN stays, and marks the tile)
            top = __builtin_elementwise_maximum(top, fmaf(ts[i], q[r], fmaf(es[i], f[r], acc[u][i][r])));
        // (tiles past the last destination repeat it: not marked)
        const int tile = st * NTS + t2 + u;
        if (__any(!(top < 0.f)) && lane == 0 && j0 + 16 * tile < j1) atomicOr(&marks[sg][tile >> 3], 1u << (tile & 7));
      }
    }
  }
  __syncthreads();
  if (tid < SG * octets) {
    const int r = tid / octets, o = tid - r * octets;
    if (m0 + 32 * r < N && j0 + 128 * o < D)
      act[((size_t)b * ((N + 31) / 32) + m0 / 32 + r) * act_row + ck * octets + o] = (uint8_t)marks[r][o];
  }
}

ScreenPlan plan_screen(const Shape &s, const Workspace &w) {
  ScreenPlan p{};
  // bf16 only: the full product's write pass subtracts a log-sum-exp rounded to fp32, in the last place of some thousands, so
  // that exact fp32 weights differ from its by up to 1e-4: more than fp32 layers with kept weights are held to.
  // (a merge region of one selection region has no far destinations; rows of a multiple of 128 bytes and at most 3072
  // channels are what the kernels take, and a list of marked tiles has room for 32768 destinations)
  if (s.dtype != TOMA_BF16 || s.R != 1 || s.P < 4 || s.C % 64 != 0 || s.C > 3072 || s.D > 32768 || !w.z_in_merge) return p;
  auto up256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
  p.kc = (s.C + 127) / 128;
  p.act_row = (s.D + 127) / 128;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += up256(bytes); return o; };
  p.q4 = take((size_t)s.B * s.N * p.kc * 64);
  p.src = take((size_t)s.B * s.N * sizeof(float2));
  p.dst = take((size_t)s.B * s.N * sizeof(float2));
  p.order = take((size_t)s.B * s.D * sizeof(int2));
  p.act = take((size_t)s.B * ((s.N + 31) / 32) * p.act_row);
  // Scratch from the start of the workspace: the selection is over, and no later stage has begun.
  if (off > w.total) return p;
  p.use = screen_pays(s);
  return p;
}

int launch_screen(const Shape &s, const ScreenPlan &p, const void *X, const int32_t *idx, void *A, char *ws, hipStream_t st) {
  const RegionView<bf16_t> v = make_view<bf16_t>(s, X);
  uint8_t *q4 = reinterpret_cast<uint8_t *>(ws + p.q4);
  int2 *order = reinterpret_cast<int2 *>(ws + p.order);
  float2 *src = reinterpret_cast<float2 *>(ws + p.src), *dst = reinterpret_cast<float2 *>(ws + p.dst);
  uint8_t *act = reinterpret_cast<uint8_t *>(ws + p.act);
  {
    KernelTimer kt(K_WBOUNDS, st);
    const dim3 grid((s.N + 31) / 32 * s.B);
    hipLaunchKernelGGL(k_fp4_bounds, grid, dim3(512), 0, st, v, idx, s.scale, s.n_loc, s.d_loc, q4, p.kc * 64, src, dst, order);
  }
  // 256 sources x 128 destinations per workgroup; 128 sources where that leaves CUs without one, more destinations
  // while four workgroups per CU remain
  const int all = p.act_row;
  const bool small = (long long)((s.N + 255) / 256) * all * s.B < 512;
  const int tiles = small ? (s.N + 127) / 128 : (s.N + 255) / 256;
  int octets = 1;
  while (octets < 8 && (long long)tiles * s.B * ((all + 2 * octets - 1) / (2 * octets)) >= 1024) octets *= 2;
  const int chunks = (all + octets - 1) / octets;
  const dim3 grid(tiles * chunks * s.B);
  KernelTimer kt(K_WSTATS, st);
#define TOMA_SCREEN(KC, SD)                                                                                             \
  if (small)                                                                                                            \
    hipLaunchKernelGGL((k_screen<KC, SD, 4>), grid, dim3(512), 0, st, v, order, q4, p.kc, src, dst, static_cast<bf16_t *>(A), \
                       act, p.act_row, octets, chunks, tiles);                                                          \
  else                                                                                                                  \
    hipLaunchKernelGGL((k_screen<KC, SD, 8>), grid, dim3(512), 0, st, v, order, q4, p.kc, src, dst, static_cast<bf16_t *>(A), \
                       act, p.act_row, octets, chunks, tiles)
  if (p.kc <= 5) { TOMA_SCREEN(5, 64); }
  else if (p.kc <= 10) { TOMA_SCREEN(10, 64); }
  else { TOMA_SCREEN(24, 32); }
#undef TOMA_SCREEN
  return launch_status();
}

}  // namespace toma

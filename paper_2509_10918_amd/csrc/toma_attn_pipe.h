// Attention of 64- and 128-wide bf16 heads: 32 queries per wave on the 32 x 32 x 16 products, with the products of
// one key tile and the softmax of another in one instruction stream.
//
// What bounds it.  Per 64 keys a wave of 32 queries issues 8 + 8 products of 32 clocks (head width 64) and about 100
// vector instructions, 32 of them exponentials of 8 clocks.  On this chip the two overlap when they alternate inside a
// wave (a product followed by two additions: 17 clocks per 16-clock product) and hardly when different waves of a SIMD
// are in different phases (23 clocks), so a step is written as two runs of products, each with the vector work that
// does not depend on it in between:
//     scores of tile t + 1   with the exponentials of tile t, their sums and packing, and the reads of V tile t
//     O += V P of tile t     with the maxima of tile t + 1 and the reads of K tile t + 2
// 32 queries per wave (not 16) halve the LDS reads per product: a tile's 16 KB are read by half as many waves.
// Queries come scaled by log2(e) / sqrt(head width) from the projection, so that a score is the exponent's argument.
#pragma once
#include "toma_gemm.h"

namespace toma {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Maximum / sum over the four 16-lane rows of a wave without LDS traffic: the gfx950 row-swap
// instructions exchange odd with even rows (16) and the upper with the lower half (32); after each
// swap the two results hold the two partners of every lane.
// Maxima as single instructions: fmaxf() would first copy each operand through v_max(x, x) to quiet signalling
// NaNs; the NaN-propagating maximum (v_maximum3_f32) takes operands as they are, and a score that is NaN makes
// its query's row NaN either way.  Builtins and no inline assembly: the compiler puts no wait states between a
// matrix product and inline assembly that reads its result (8 are due after a 16 x 16 x 32 bf16 product).
// The same speed as v_max3_f32 written as assembly.
__device__ __forceinline__ float max2_f32(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float max3_f32(float a, float b, float c) { return max2_f32(max2_f32(a, b), c); }
__device__ __forceinline__ float rows4_max_f32(float v) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float m = max2_f32(__builtin_bit_cast(float, (uint32_t)a[0]), __builtin_bit_cast(float, (uint32_t)a[1]));
  const uint32_t w = __builtin_bit_cast(uint32_t, m);
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return max2_f32(__builtin_bit_cast(float, (uint32_t)b[0]), __builtin_bit_cast(float, (uint32_t)b[1]));
}
__device__ __forceinline__ float rows4_sum_f32(float v) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float m = __builtin_bit_cast(float, (uint32_t)a[0]) + __builtin_bit_cast(float, (uint32_t)a[1]);
  const uint32_t w = __builtin_bit_cast(uint32_t, m);
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __builtin_bit_cast(float, (uint32_t)b[0]) + __builtin_bit_cast(float, (uint32_t)b[1]);
}

// LDS tiles of 64 rows (keys), PPR packets of 16 bytes per row; packet p of a row sits at p ^ swizzle(row).
// K is read 32 rows at a time, one packet each; V by transpose reads, four rows x 32 bytes per 16 lanes.
template <int PPR> __device__ __forceinline__ int attn_k_swz(int row) { return PPR == 8 ? (row >> 1) & 7 : row & 15; }
template <int PPR> __device__ __forceinline__ int attn_v_swz(int row) {
  return PPR == 8 ? (((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1) : ((row & 3) << 2) | (((row >> 2) & 1) << 1);
}

// Grid: (sample, head, block of 32 x waves queries); four to eight waves.  Lq queries attend to L keys.
template <int DH>
__global__ __launch_bounds__(512, 2) void k_attn_pipe(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ Kx,
                                                      const bf16_t *__restrict__ V, bf16_t *__restrict__ O, int Lq, int L,
                                                      int H, const float *__restrict__ Zs, int D, bf16_t *__restrict__ Oe) {
  constexpr int PPR = DH / 8;          // packets per row
  constexpr int KK = DH / 16;          // products along the head width per 32 keys
  constexpr int DT = DH / 32;          // 32-wide output tiles along the head width
  constexpr int STAGES = 4, TILE = 64 * DH, CH = PPR;  // ring; elements and 1 KiB chunks per tile
  constexpr int LW = 4, NI = CH / LW;  // waves that fetch; their chunks per tile
  constexpr bool kSplat = DH <= 64;    // the scores' accumulators start at minus the reference point (16 registers)
  constexpr int LK = DH <= 64 ? 4 : 2, LV = DH <= 64 ? 4 : 1;  // fragment groups read ahead of their products
  __shared__ __align__(1024) bf16_t Ks[STAGES][TILE];
  __shared__ __align__(1024) bf16_t Vs[STAGES][TILE];
  typedef s16x4 __attribute__((address_space(3))) *lds_s16x4_ptr;
  typedef short s16x8 __attribute__((ext_vector_type(8)));

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 31, h = lane >> 5;
  const int QB = (int)(blockDim.x >> 6) * 32;
  const int nq = (Lq + QB - 1) / QB;
  const int work = xcd_remap(blockIdx.x, gridDim.x);  // (the query blocks of a head share its K and V in one L2)
  const int qb = work % nq, hd = (work / nq) % H, b = work / (nq * H);
  const size_t head = ((size_t)b * H + hd) * L * DH;
  const bf16_t *Qh = Q + ((size_t)b * H + hd) * Lq * DH, *Kh = Kx + head, *Vh = V + head;
  const int q_w = qb * QB + w * 32, nt = (L + 63) / 64;

  // queries as right operands: lane = query c, channels 16 kk + 8 h .. + 7
  bf16x8 fq[KK];
  {
    const int q = min(q_w + c, Lq - 1);
#pragma unroll
    for (int kk = 0; kk < KK; kk++) fq[kk] = *reinterpret_cast<const bf16x8 *>(Qh + (size_t)q * DH + 16 * kk + 8 * h);
  }

  // ---- loads: the first LW waves, NI chunks of each tile; byte offsets from the tile's first row ----
  const bool loader = w < LW;
  const int wl = __builtin_amdgcn_readfirstlane(w & (LW - 1));
  const uint32_t ks_addr = lds_addr_of(&Ks[0][0]) + (uint32_t)wl * (NI * 1024);
  const uint32_t vs_addr = lds_addr_of(&Vs[0][0]) + (uint32_t)wl * (NI * 1024);
  constexpr int RPC = 64 / PPR;        // rows per chunk
  const int row0 = lane / PPR, slot0 = lane % PPR;
  const uint32_t k_off0 = (uint32_t)(row0 * PPR + (slot0 ^ attn_k_swz<PPR>(row0))) * 16;
  const uint32_t v_off0 = (uint32_t)(row0 * PPR + (slot0 ^ attn_v_swz<PPR>(row0))) * 16;
  // (the swizzle of chunk wl NI + t differs from the first chunk's by bits of t alone)
  static_assert(NI * RPC % 16 == 0, "a wave's chunks start at a multiple of 16 rows");
  auto k_off = [&](int t) { return k_off0 ^ (uint32_t)(attn_k_swz<PPR>(RPC * t) * 16); };
  auto v_off = [&](int t) { return v_off0 ^ (uint32_t)(attn_v_swz<PPR>(RPC * t) * 16); };
  auto load_tile = [&](const bf16_t *base, uint32_t off, uint32_t dst, int it, int t) {
    const int chunk = wl * NI + t;
    const bf16_t *src = base + (ptrdiff_t)it * TILE;
    uint32_t o = off + (uint32_t)(chunk * 1024);
    if ((it + 1) * 64 > L)  // (only the last tile: rows past the end repeat row L - 1 and are masked below)
      o -= (uint32_t)(max(it * 64 + chunk * RPC + lane / PPR - (L - 1), 0) * (DH * 2));
    load_to_lds16_from(src, o, dst + (uint32_t)(t * 1024));
  };
  auto issue_k = [&](int st, int it) {
    if (!loader) return;
#pragma unroll
    for (int t = 0; t < NI; t++) load_tile(Kh, k_off(t), ks_addr + (uint32_t)(st * TILE * 2), it, t);
  };
  auto issue_v = [&](int st, int it) {
    if (!loader) return;
#pragma unroll
    for (int t = 0; t < NI; t++) load_tile(Vh, v_off(t), vs_addr + (uint32_t)(st * TILE * 2), it, t);
  };
  // group j: V tile j and K tile j + 2 (the last K tile again past the end: every group has the same number of loads)
  auto issue_group = [&](int st, int j) { issue_k((st + 2) % STAGES, min(j + 2, nt - 1)); issue_v(st, j); };

  // ---- fragment reads ----
  // K: lane = key 32 kt + c, channels 16 kk + 8 h .. + 7
  const int k_lane = c * DH, k_slot = h ^ attn_k_swz<PPR>(c);
  auto read_k = [&](bf16x8 (&f)[2], int st, int kk) {
#pragma unroll
    for (int kt = 0; kt < 2; kt++)
      f[kt] = *reinterpret_cast<const bf16x8 *>(&Ks[st][k_lane + ((k_slot ^ (2 * kk)) * 8) + kt * 32 * DH]);
  };
  // V transposed: lane = channel 32 dt + c, keys 16 u + 4 h + 0 .. 3 and 16 u + 8 + 4 h + 0 .. 3 - the keys whose
  // probabilities the lanes of half h hold in registers 8 u .. 8 u + 7
  const int j4 = lane & 15, v_row = 4 * h + (j4 >> 2), v_pkt = 2 * ((lane >> 4) & 1) + ((j4 & 3) >> 1);
  const int v_lane = v_row * DH + (j4 & 1) * 4, v_slot = v_pkt ^ attn_v_swz<PPR>(v_row);
  auto read_v = [&](bf16x8 (&f)[DT], int st, int u) {
#pragma unroll
    for (int dt = 0; dt < DT; dt++) {
      const bf16_t *p = &Vs[st][v_lane + ((v_slot ^ (4 * dt)) * 8) + 16 * u * DH];
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 8 * DH));
      const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      f[dt] = __builtin_bit_cast(bf16x8, both);
    }
  };
  auto fence = [&]() { __builtin_amdgcn_sched_barrier(0); };
  auto meet = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto half_max = [&](float v) {  // over the two lanes that share a query
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_elementwise_maximum(__builtin_bit_cast(float, (uint32_t)a[0]), __builtin_bit_cast(float, (uint32_t)a[1]));
  };

  f32x16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; dt++) oacc[dt] = (f32x16)(0.f);
  float l_a = 0.f, l_b = 0.f;  // row sums of this lane's keys
  float m = 0.f;               // reference point of the exponentials, per query
  f32x16 minus_m;              // (kSplat: what the scores start from)
  constexpr float kSlack = 8.0f;
  const f32x16 zero16 = (f32x16)(0.f);

  // masks the keys past the end (the last tile only)
  auto mask = [&](f32x16 (&s)[2], int key0) {
#pragma unroll
    for (int kt = 0; kt < 2; kt++)
#pragma unroll
      for (int r = 0; r < 16; r++)
        if (key0 + 32 * kt + 8 * (r >> 2) + 4 * h + (r & 3) >= L) s[kt][r] = -__builtin_inff();
  };

  // ---- prologue: the first tile's scores and reference point ----
  wait_vmcnt<0>();  // the queries have landed: from here on only the ring's loads are outstanding
  issue_k(0, 0);
  issue_k(1, min(1, nt - 1));
  issue_group(0, 0);
  wait_vmcnt<2 * NI>();
  meet();
  if (nt > 1) issue_group(1, 1);  // (its K tile goes to stage 3)
  bf16x8 fk[LK][2], fv[LV][DT];
  f32x16 sa[2], sb[2];
#pragma unroll
  for (int kk = 0; kk < KK; kk++) {
    bf16x8 f[2];
    read_k(f, 0, kk);
#pragma unroll
    for (int kt = 0; kt < 2; kt++) sa[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[kt], fq[kk], kk == 0 ? zero16 : sa[kt], 0, 0, 0);
  }
#pragma unroll
  for (int g = 0; g < LK; g++) read_k(fk[g], 1, g);
  {
    float mx = __builtin_elementwise_maximum(sa[0][0], sa[1][0]);
#pragma unroll
    for (int r = 1; r < 16; r++) mx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mx, sa[0][r]), sa[1][r]);
    m = half_max(mx);  // (rows past the end repeat a key: they do not raise it)
    minus_m = (f32x16)(-m);
    if constexpr (kSplat) {
#pragma unroll
      for (int kt = 0; kt < 2; kt++)
#pragma unroll
        for (int r = 0; r < 16; r++) sa[kt][r] -= m;
    }
  }

  // One step.  s: scores of tile t (kSplat: minus the reference point); n: room for the next tile's.
  auto step = [&](auto stage_c, f32x16 (&s)[2], f32x16 (&n)[2], int t) {
    constexpr int ST = decltype(stage_c)::value;
    // this wave's part of group t has landed (group t + 1 may be in flight); after the barrier so has everyone's, and
    // every wave is done with V tile t - 2 and K tile t, whose stages the next group takes
    if (t + 1 < nt) wait_vmcnt<2 * NI>(); else wait_vmcnt<0>();
    meet();
    if (t + 2 < nt) issue_group((ST + 2) % STAGES, t + 2);
    if ((t + 1) * 64 > L) mask(s, t * 64);
    bf16x8 fp[4];
#pragma unroll
    for (int g = 0; g < LV; g++) read_v(fv[g], ST, g);
    fence();
    __builtin_amdgcn_s_setprio(0);
    // ---- scores of tile t + 1 (of no use, and not used, after the last) | exponentials of tile t ----
    constexpr int EP = 32 / (2 * KK);  // exponentials per product
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int kt = 0; kt < 2; kt++) {
        n[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[kk % LK][kt], fq[kk], kk == 0 ? (kSplat ? minus_m : zero16) : n[kt], 0, 0, 0);
        float e[EP];
#pragma unroll
        for (int i = 0; i < EP; i++) {
          const int at = (2 * kk + kt) * EP + i;
          e[i] = __builtin_amdgcn_exp2f(kSplat ? s[at >> 4][at & 15] : s[at >> 4][at & 15] - m);
        }
#pragma unroll
        for (int i = 0; i < EP; i += 2) { l_a += e[i]; l_b += e[i + 1]; }
#pragma unroll
        for (int i = 0; i < EP; i += 2) {
          const int at = (2 * kk + kt) * EP + i;
          const bf16x2 pk = __builtin_convertvector((__attribute__((ext_vector_type(2))) float){e[i], e[i + 1]}, bf16x2);
          fp[at >> 3][at & 7] = pk[0];
          fp[at >> 3][(at & 7) + 1] = pk[1];
        }
        if (kt == 1 && kk + LK < KK) read_k(fk[kk % LK], (ST + 1) % STAGES, kk + LK);
        fence();
      }
    // ---- O += V P of tile t | row sums of tile t, maxima of tile t + 1 ----
    __builtin_amdgcn_s_setprio(1);
    float mx = -__builtin_inff(), my = -__builtin_inff();
#pragma unroll
    for (int u = 0; u < 4; u++)
#pragma unroll
      for (int dt = 0; dt < DT; dt++) {
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv[u % LV][dt], fp[u], oacc[dt], 0, 0, 0);
        constexpr int NP = 4 * DT;     // products of this run
        const int i = u * DT + dt;
        // the first half: the next K fragments; the second: the maxima
        if (i < NP / 2) {
#pragma unroll
          for (int g = i * LK / (NP / 2); g < (i + 1) * LK / (NP / 2); g++) read_k(fk[g], (ST + 2) % STAGES, g);
        } else {
          constexpr int PER = 32 / (NP / 2);
#pragma unroll
          for (int q = 0; q < PER; q += 4) {
            const int at = (i - NP / 2) * PER + q;
            mx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mx, n[at >> 4][at & 15]), n[at >> 4][(at & 15) + 1]);
            my = __builtin_elementwise_maximum(__builtin_elementwise_maximum(my, n[at >> 4][(at & 15) + 2]), n[at >> 4][(at & 15) + 3]);
          }
        }
        if (dt == DT - 1 && u + LV < 4) read_v(fv[u % LV], ST, u + LV);
        fence();
      }
    mx = __builtin_elementwise_maximum(mx, my);
    // The reference point follows the running maximum lazily: it moves, and the sums so far are rescaled, only when
    // some lane's maximum has grown by more than 2^kSlack - almost never after the first tile.  The final O / l does
    // not depend on it.
    if (t + 1 < nt && __any(kSplat ? mx > kSlack : mx > m + kSlack)) {
      const float row = half_max(mx);
      const float up = kSplat ? fmaxf(row, 0.f) : fmaxf(row, m) - m;
      const float alpha = __builtin_amdgcn_exp2f(-up);
      l_a *= alpha;
      l_b *= alpha;
      if constexpr (kSplat) {
#pragma unroll
        for (int r = 0; r < 16; r++) minus_m[r] -= up;
#pragma unroll
        for (int kt = 0; kt < 2; kt++)
#pragma unroll
          for (int r = 0; r < 16; r++) n[kt][r] -= up;
      } else {
        m = fmaxf(row, m);
      }
#pragma unroll
      for (int dt = 0; dt < DT; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) oacc[dt][r] *= alpha;
    }
  };
  for (int t = 0; t < nt; t += 4) {
    step(std::integral_constant<int, 0>{}, sa, sb, t);
    if (t + 1 < nt) step(std::integral_constant<int, 1>{}, sb, sa, t + 1);
    if (t + 2 < nt) step(std::integral_constant<int, 2>{}, sa, sb, t + 2);
    if (t + 3 < nt) step(std::integral_constant<int, 3>{}, sb, sa, t + 3);
  }

  // ---- O[b][q][hd DH + channel]: lane holds query c, channels 32 dt + 8 (r / 4) + 4 h + r % 4 ----
  float l = l_a + l_b;
  {
    const uint32_t u = __builtin_bit_cast(uint32_t, l);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    l = __builtin_bit_cast(float, (uint32_t)a[0]) + __builtin_bit_cast(float, (uint32_t)a[1]);
  }
  const int q = q_w + c, Cw = H * DH;
  if (q >= Lq) return;
  float inv = 1.0f / l;
  if (Zs && q < D) inv /= fmaxf(Zs[(size_t)b * D + q], 1e-20f);  // unmerge input: O / Z
  // (extra-token rows straight to their own output when the caller has one)
  bf16_t *dst = (Oe && q >= D ? Oe + ((size_t)b * (Lq - D) + (q - D)) * Cw : O + ((size_t)b * Lq + q) * Cw) + hd * DH + 4 * h;
#pragma unroll
  for (int dt = 0; dt < DT; dt++)
#pragma unroll
    for (int r4 = 0; r4 < 4; r4++) {
      f32x4 v;
#pragma unroll
      for (int r = 0; r < 4; r++) v[r] = oacc[dt][4 * r4 + r] * inv;
      store4<bf16_t>(dst + 32 * dt + 8 * r4, v);
    }
}

// The same with 16 queries per wave on the 16 x 16 x 32 products, three waves to a SIMD (four to twelve waves per
// workgroup): half the work per wave, for launches that the larger kernel would spread unevenly over the SIMDs.
template <int DH>
__global__ __launch_bounds__(768, 3) void k_attn_pipe16(const bf16_t *__restrict__ Q, const bf16_t *__restrict__ Kx,
                                                      const bf16_t *__restrict__ V, bf16_t *__restrict__ O, int Lq, int L,
                                                      int H, const float *__restrict__ Zs, int D, bf16_t *__restrict__ Oe) {
  constexpr int PPR = DH / 8;          // packets per row
  constexpr int KK = DH / 32;          // products along the head width per 16 keys
  constexpr int DT = DH / 16;          // 16-wide output tiles along the head width
  constexpr int STAGES = 4, TILE = 64 * DH, CH = PPR;  // ring; elements and 1 KiB chunks per tile
  constexpr int LW = 4, NI = CH / LW;  // waves that fetch; their chunks per tile
  constexpr int LK = DH <= 64 ? 2 : 1, LV = DH <= 64 ? 2 : 1;  // fragment groups read ahead of their products
  __shared__ __align__(1024) bf16_t Ks[STAGES][TILE];
  __shared__ __align__(1024) bf16_t Vs[STAGES][TILE];
  typedef s16x4 __attribute__((address_space(3))) *lds_s16x4_ptr;
  typedef short s16x8 __attribute__((ext_vector_type(8)));

  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, h = lane >> 4;
  const int QB = (int)(blockDim.x >> 6) * 16;
  const int nq = (Lq + QB - 1) / QB;
  const int work = xcd_remap(blockIdx.x, gridDim.x);  // (the query blocks of a head share its K and V in one L2)
  const int qb = work % nq, hd = (work / nq) % H, b = work / (nq * H);
  const size_t head = ((size_t)b * H + hd) * L * DH;
  const bf16_t *Qh = Q + ((size_t)b * H + hd) * Lq * DH, *Kh = Kx + head, *Vh = V + head;
  const int q_w = qb * QB + w * 16, nt = (L + 63) / 64;

  // queries as right operands: lane = query c, channels 32 kk + 8 h .. + 7
  bf16x8 fq[KK];
  {
    const int q = min(q_w + c, Lq - 1);
#pragma unroll
    for (int kk = 0; kk < KK; kk++) fq[kk] = *reinterpret_cast<const bf16x8 *>(Qh + (size_t)q * DH + 32 * kk + 8 * h);
  }

  // ---- loads: the first LW waves, NI chunks of each tile; byte offsets from the tile's first row ----
  const bool loader = w < LW;
  const int wl = __builtin_amdgcn_readfirstlane(w & (LW - 1));
  const uint32_t ks_addr = lds_addr_of(&Ks[0][0]) + (uint32_t)wl * (NI * 1024);
  const uint32_t vs_addr = lds_addr_of(&Vs[0][0]) + (uint32_t)wl * (NI * 1024);
  constexpr int RPC = 64 / PPR;        // rows per chunk
  const int row0 = lane / PPR, slot0 = lane % PPR;
  const uint32_t k_off0 = (uint32_t)(row0 * PPR + (slot0 ^ attn_k_swz<PPR>(row0))) * 16;
  const uint32_t v_off0 = (uint32_t)(row0 * PPR + (slot0 ^ attn_v_swz<PPR>(row0))) * 16;
  // (the swizzle of chunk wl NI + t differs from the first chunk's by bits of t alone)
  static_assert(NI * RPC % 16 == 0, "a wave's chunks start at a multiple of 16 rows");
  auto k_off = [&](int t) { return k_off0 ^ (uint32_t)(attn_k_swz<PPR>(RPC * t) * 16); };
  auto v_off = [&](int t) { return v_off0 ^ (uint32_t)(attn_v_swz<PPR>(RPC * t) * 16); };
  auto load_tile = [&](const bf16_t *base, uint32_t off, uint32_t dst, int it, int t) {
    const int chunk = wl * NI + t;
    const bf16_t *src = base + (ptrdiff_t)it * TILE;
    uint32_t o = off + (uint32_t)(chunk * 1024);
    if ((it + 1) * 64 > L)  // (only the last tile: rows past the end repeat row L - 1 and are masked below)
      o -= (uint32_t)(max(it * 64 + chunk * RPC + lane / PPR - (L - 1), 0) * (DH * 2));
    load_to_lds16_from(src, o, dst + (uint32_t)(t * 1024));
  };
  auto issue_k = [&](int st, int it) {
    if (!loader) return;
#pragma unroll
    for (int t = 0; t < NI; t++) load_tile(Kh, k_off(t), ks_addr + (uint32_t)(st * TILE * 2), it, t);
  };
  auto issue_v = [&](int st, int it) {
    if (!loader) return;
#pragma unroll
    for (int t = 0; t < NI; t++) load_tile(Vh, v_off(t), vs_addr + (uint32_t)(st * TILE * 2), it, t);
  };
  // group j: V tile j and K tile j + 2 (the last K tile again past the end: every group has the same number of loads)
  auto issue_group = [&](int st, int j) { issue_k((st + 2) % STAGES, min(j + 2, nt - 1)); issue_v(st, j); };

  // ---- fragment reads ----
  // K: lane = key 16 kt + c, channels 32 kk + 8 h .. + 7
  const int k_lane = c * DH, k_slot = h ^ attn_k_swz<PPR>(c);
  auto read_k = [&](bf16x8 (&f)[4], int st, int kk) {
#pragma unroll
    for (int kt = 0; kt < 4; kt++)  // (sixteen rows further on the swizzle is the same)
      f[kt] = *reinterpret_cast<const bf16x8 *>(&Ks[st][k_lane + ((k_slot ^ (4 * kk)) * 8) + kt * 16 * DH]);
  };
  // V transposed: lane = channel 16 dt + c, keys 32 u + 4 h + 0 .. 3 and 32 u + 16 + 4 h + 0 .. 3 - the keys whose
  // probabilities the lanes of group h hold in score tiles 2 u and 2 u + 1
  const int j4 = lane & 15, v_row = 4 * h + (j4 >> 2), v_pkt = (j4 & 3) >> 1;
  const int v_lane = v_row * DH + (j4 & 1) * 4, v_slot = v_pkt ^ attn_v_swz<PPR>(v_row);
  auto read_v = [&](bf16x8 (&f)[DT], int st, int u) {
#pragma unroll
    for (int dt = 0; dt < DT; dt++) {
      const bf16_t *p = &Vs[st][v_lane + ((v_slot ^ (2 * dt)) * 8) + 32 * u * DH];
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 16 * DH));
      const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      f[dt] = __builtin_bit_cast(bf16x8, both);
    }
  };
  auto fence = [&]() { __builtin_amdgcn_sched_barrier(0); };
  auto meet = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  f32x4 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; dt++) oacc[dt] = (f32x4)(0.f);
  float l_a = 0.f, l_b = 0.f;  // row sums of this lane's keys
  f32x4 minus_m;               // minus the reference point of the exponentials: what the scores start from
  constexpr float kSlack = 8.0f;
  const f32x4 zero4 = (f32x4)(0.f);

  // masks the keys past the end (the last tile only)
  auto mask = [&](f32x4 (&s)[4], int key0) {
#pragma unroll
    for (int kt = 0; kt < 4; kt++)
#pragma unroll
      for (int r = 0; r < 4; r++)
        if (key0 + 16 * kt + 4 * h + r >= L) s[kt][r] = -__builtin_inff();
  };

  // ---- prologue: the first tile's scores and reference point ----
  wait_vmcnt<0>();  // the queries have landed: from here on only the ring's loads are outstanding
  issue_k(0, 0);
  issue_k(1, min(1, nt - 1));
  issue_group(0, 0);
  wait_vmcnt<2 * NI>();
  meet();
  if (nt > 1) issue_group(1, 1);  // (its K tile goes to stage 3)
  bf16x8 fk[LK][4], fv[LV][DT];
  f32x4 sa[4], sb[4];
#pragma unroll
  for (int kk = 0; kk < KK; kk++) {
    bf16x8 f[4];
    read_k(f, 0, kk);
#pragma unroll
    for (int kt = 0; kt < 4; kt++) sa[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[kt], fq[kk], kk == 0 ? zero4 : sa[kt], 0, 0, 0);
  }
#pragma unroll
  for (int g = 0; g < LK; g++) read_k(fk[g], 1, g);
  {
    float mx = sa[0][0];
#pragma unroll
    for (int r = 1; r < 16; r++) mx = max2_f32(mx, sa[r >> 2][r & 3]);
    const float m = rows4_max_f32(mx);  // (rows past the end repeat a key: they do not raise it)
    minus_m = (f32x4)(-m);
#pragma unroll
    for (int kt = 0; kt < 4; kt++)
#pragma unroll
      for (int r = 0; r < 4; r++) sa[kt][r] -= m;
  }

  // One step.  s: scores of tile t minus the reference point; n: room for the next tile's.
  auto step = [&](auto stage_c, f32x4 (&s)[4], f32x4 (&n)[4], int t) {
    constexpr int ST = decltype(stage_c)::value;
    // this wave's part of group t has landed (group t + 1 may be in flight); after the barrier so has everyone's, and
    // every wave is done with V tile t - 2 and K tile t, whose stages the next group takes
    if (t + 1 < nt) wait_vmcnt<2 * NI>(); else wait_vmcnt<0>();
    meet();
    if (t + 2 < nt) issue_group((ST + 2) % STAGES, t + 2);
    if ((t + 1) * 64 > L) mask(s, t * 64);
    bf16x8 fp[2];
#pragma unroll
    for (int g = 0; g < LV; g++) read_v(fv[g], ST, g);
    fence();
    __builtin_amdgcn_s_setprio(0);
    // ---- scores of tile t + 1 (of no use, and not used, after the last) | exponentials of tile t ----
    constexpr int EP = 16 / (4 * KK);  // exponentials per product
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int kt = 0; kt < 4; kt++) {
        n[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fk[kk % LK][kt], fq[kk], kk == 0 ? minus_m : n[kt], 0, 0, 0);
#pragma unroll
        for (int i = 0; i < EP; i++) {
          const int at = (4 * kk + kt) * EP + i;
          const float e = __builtin_amdgcn_exp2f(s[at >> 2][at & 3]);
          s[at >> 2][at & 3] = e;
          if (at & 1) l_b += e; else l_a += e;
          if (at & 1) {  // score tiles 2 u and 2 u + 1 make the eight slots of fragment u
            const bf16x2 pk = __builtin_convertvector((__attribute__((ext_vector_type(2))) float){s[at >> 2][(at & 3) - 1], e}, bf16x2);
            fp[at >> 3][(at & 7) - 1] = pk[0];
            fp[at >> 3][at & 7] = pk[1];
          }
        }
        if (kt == 3 && kk + LK < KK) read_k(fk[kk % LK], (ST + 1) % STAGES, kk + LK);
        fence();
      }
    // ---- O += V P of tile t | row sums of tile t, maxima of tile t + 1 ----
    __builtin_amdgcn_s_setprio(1);
    float mx = -__builtin_inff(), my = -__builtin_inff();
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
      for (int dt = 0; dt < DT; dt++) {
        oacc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fv[u % LV][dt], fp[u], oacc[dt], 0, 0, 0);
        constexpr int NP = 2 * DT;     // products of this run
        const int i = u * DT + dt;
        // the first half: the next K fragments; the second: the maxima
        if (i < NP / 2) {
#pragma unroll
          for (int g = i * LK / (NP / 2); g < (i + 1) * LK / (NP / 2); g++) read_k(fk[g], (ST + 2) % STAGES, g);
        } else {
          constexpr int PER = 16 / (NP / 2);
#pragma unroll
          for (int q = 0; q < PER; q += 2) {
            const int at = (i - NP / 2) * PER + q;
            if (q & 2) my = max3_f32(my, n[at >> 2][at & 3], n[at >> 2][(at & 3) + 1]);
            else mx = max3_f32(mx, n[at >> 2][at & 3], n[at >> 2][(at & 3) + 1]);
          }
        }
        if (dt == DT - 1 && u + LV < 2) read_v(fv[u % LV], ST, u + LV);
        fence();
      }
    mx = max2_f32(mx, my);
    // The reference point follows the running maximum lazily: it moves, and the sums so far are rescaled, only when
    // some lane's maximum has grown by more than 2^kSlack - almost never after the first tile.  The final O / l does
    // not depend on it.
    if (t + 1 < nt && __any(mx > kSlack)) {
      const float up = fmaxf(rows4_max_f32(mx), 0.f);
      const float alpha = __builtin_amdgcn_exp2f(-up);
      l_a *= alpha;
      l_b *= alpha;
#pragma unroll
      for (int r = 0; r < 4; r++) minus_m[r] -= up;
#pragma unroll
      for (int kt = 0; kt < 4; kt++)
#pragma unroll
        for (int r = 0; r < 4; r++) n[kt][r] -= up;
#pragma unroll
      for (int dt = 0; dt < DT; dt++)
#pragma unroll
        for (int r = 0; r < 4; r++) oacc[dt][r] *= alpha;
    }
  };
  for (int t = 0; t < nt; t += 4) {
    step(std::integral_constant<int, 0>{}, sa, sb, t);
    if (t + 1 < nt) step(std::integral_constant<int, 1>{}, sb, sa, t + 1);
    if (t + 2 < nt) step(std::integral_constant<int, 2>{}, sa, sb, t + 2);
    if (t + 3 < nt) step(std::integral_constant<int, 3>{}, sb, sa, t + 3);
  }

  // ---- O[b][q][hd DH + channel]: lane holds query c, channels 16 dt + 4 h + r ----
  const float l = rows4_sum_f32(l_a + l_b);
  const int q = q_w + c, Cw = H * DH;
  if (q >= Lq) return;
  float inv = 1.0f / l;
  if (Zs && q < D) inv /= fmaxf(Zs[(size_t)b * D + q], 1e-20f);  // unmerge input: O / Z
  // (extra-token rows straight to their own output when the caller has one)
  bf16_t *dst = (Oe && q >= D ? Oe + ((size_t)b * (Lq - D) + (q - D)) * Cw : O + ((size_t)b * Lq + q) * Cw) + hd * DH + 4 * h;
#pragma unroll
  for (int dt = 0; dt < DT; dt++) store4<bf16_t>(dst + 16 * dt, oacc[dt] * inv);
}

}  // namespace toma

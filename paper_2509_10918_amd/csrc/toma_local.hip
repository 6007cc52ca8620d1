// Merge weights and merge of small merge regions in one kernel.
//
// A region-local merge of a few dozen to a few hundred tokens is a handful of 16 x 16 tiles: as separate launches
// (statistics, log-sum-exp, weights, their row sums, merge) it is five dependent chains of loads, in which the logits are
// computed twice.  Here a workgroup (8 waves) takes one region and a slice of its channels:
//   1. all logits of the region, its source and destination rows streamed through a ring in LDS (three or four stages of
//      128 bytes of every row); the steps of its own slice stay in LDS;
//   2. the softmax over destinations of every source, the weights as stored in LDS;
//   3. the merge of its slice from the weights and rows in LDS, Z from the same product (a fragment of ones).
// The logits are computed once per slice, that is several times over: a region's are a few MFLOP, and the slices are what
// fills the chip (SDXL's second stage: 32 regions, seven slices).  Every slice adds them in the same order, so that all
// have the same weights.  What bounds it is the chain of K steps, 0.3 to 1 us each (wait, barrier, reads, products of up to
// eight tiles per wave); a deeper ring changed nothing (six stages: 14.2 us where three took 13.6), branches inside the
// step cost a fifth of it.  Measured (us, the separate kernels and this one): regions of 64 tokens with 32 destinations,
// width 1280, 128 regions 43.5 and 16.9; 64 with 16, 32 regions 28.8 and 13.0; 96 with 29, width 352, 45 regions 30 and 10;
// 16 with 8, width 320, 2048 regions 96 and 26.
// bf16 only.  fp32 gained as well (64 with 32, width 640, 48 regions 46 and 20 us), but the kernels it would replace store
// exp(logit - lse) with a log-sum-exp rounded to fp32 (WeightsPol, the write pass), up to 1e-4 of a weight away from the
// softmax made here: fp32 weights, and layers that keep them, would have changed by more than the 1e-5 that fp32 layers with
// kept weights are held to.  (The one-pass kernel and the recomputed weights do not round there: it is the write pass that
// would have to change first.)
#include <type_traits>

#include "toma_gemm.h"
#include "toma_internal.h"
#include "toma_region.h"

namespace toma {

constexpr int kLocalLds = 156 * 1024, kLocalLds2 = 78 * 1024;  // (one workgroup per CU, or two)

// LDS of a region: the ring (whose room the logits and weights take over) and the slice's steps of the source rows
struct LocalPlan { int nti, ntj, steps, stages, slices, per_slice; size_t ring, lds; };
static bool plan_local(int regions, int Nr, int Dr, int C, LocalPlan *best) {
  constexpr int es = 2;
  LocalPlan p;
  p.nti = Nr / 16;
  p.ntj = (Dr + 15) / 16;
  const int rows = Nr + 16 * p.ntj, Nrp = (Nr + 31) / 32 * 32;
  if (Nr % 16 != 0 || rows > 256) return false;
  p.steps = (C * es + 127) / 128;
  const size_t logits = ((size_t)Nr * (16 * p.ntj + 1) * 4 + 15) & ~(size_t)15;
  const size_t weights = (size_t)16 * p.ntj * (Nrp + 16 / es) * es, step = (size_t)Nrp * 128;
  bool found = false;
  for (int stages = rows <= 128 ? 4 : 3; stages >= 3; stages--) {
    p.stages = stages;
    p.ring = (std::max((size_t)stages * rows * 128, logits + weights) + 1023) & ~(size_t)1023;
    if (p.ring + step > (size_t)kLocalLds) continue;
    const int most = (int)((kLocalLds - p.ring) / step);
    // a workgroup per CU, as far as the steps go; no more steps of a slice than the LDS keeps
    p.slices = std::max(std::min(p.steps, std::max(256 / regions, 1)), (p.steps + most - 1) / most);
    p.per_slice = (p.steps + p.slices - 1) / p.slices;
    p.slices = (p.steps + p.per_slice - 1) / p.per_slice;
    p.lds = p.ring + p.per_slice * step;
    if (!found || p.slices < best->slices) *best = p;
    found = true;
  }
  return found;
}

// NL: load instructions per wave and step (64 rows each); TPW: logit tiles per wave; ST: stages of the ring
template <int NL, int TPW, int ST, int LDSB>
__global__ __launch_bounds__(512) void k_local_merge(const RegionView<bf16_t> v, const int32_t *__restrict__ idx, float scale,
                                                     bf16_t *__restrict__ A, float *__restrict__ Z, bf16_t *__restrict__ Xm, int ntj,
                                                     int slices, int per_slice, int ring_bytes) {
  typedef bf16_t T;
  constexpr int ES = (int)sizeof(T), EPS = 128 / ES, EPP = 16 / ES, NH = 2;
  constexpr int CPS = EPS / 16;  // 16-channel tiles per step
  __shared__ __align__(1024) char lds[LDSB];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int work = xcd_remap(blockIdx.x, gridDim.x);  // (the slices of a region share its rows in one L2)
  const int z = work / slices, slice = work - z * slices, b = z / v.R, rho = z % v.R;
  const int Nr = v.Nr, Dr = v.Dr, C = v.C, Drp = 16 * ntj, rows = Nr + Drp, Nrp = (Nr + 31) / 32 * 32;
  const int steps = (C * ES + 127) / 128, k0 = slice * per_slice, k1 = min(k0 + per_slice, steps);
  const int tail = C * ES - (steps - 1) * 128;  // bytes of the last step: 128, or 64 (C an odd multiple of 32)
  const T *Xb = v.X + (size_t)b * v.N * C;
  char *kept = lds + ring_bytes;

  // ---- loads: wave w takes the pieces w, w + 8, ... (8 rows x 128 bytes; the last one again past the end) of a step ----
  const int pieces = rows / 8;
  uint32_t off[NL];
  int piece[NL], pkt[NL];
#pragma unroll
  for (int t = 0; t < NL; t++) {
    piece[t] = min(w + 8 * t, pieces - 1);
    const int row = piece[t] * 8 + (lane >> 3);
    int tok;
    if (row < Nr) {
      tok = v.token(rho, row);
    } else {  // (rows past the last destination repeat it)
      tok = idx[(size_t)b * v.D + rho * Dr + min(row - Nr, Dr - 1)];
      tok = tok < 0 ? 0 : (tok >= v.N ? v.N - 1 : tok);
    }
    pkt[t] = (lane & 7) ^ (row & 7);
    off[t] = (uint32_t)tok * (uint32_t)C + (uint32_t)(pkt[t] * EPP);
  }
  const uint32_t lds0 = lds_addr_of(lds);
  const int stage_bytes = rows * 128, kept_bytes = Nrp * 128, own = k1 - k0;
  bool source[NL];
#pragma unroll
  for (int t = 0; t < NL; t++) source[t] = piece[t] * 8 < Nr;
  // (ring: the stage of step s, kept along by the callers)
  auto issue = [&](int s, int ring) {
    const int back = s == steps - 1 && tail == 64 ? 4 * EPP : 0;  // (the second half of a half step: the first half again)
    const bool mine = (uint32_t)(s - k0) < (uint32_t)own;
    const int at_own = ring_bytes + (s - k0) * kept_bytes;
#pragma unroll
    for (int t = 0; t < NL; t++)
      load_to_lds16_at(Xb + off[t] + s * EPS - (pkt[t] >= 4 ? back : 0),
                       lds0 + (uint32_t)__builtin_amdgcn_readfirstlane((mine && source[t] ? at_own : ring * stage_bytes) + piece[t] * 1024));
  };
  // logit tiles of this wave: consecutive ones, which mostly share their sources' fragment (the last tile again past the
  // end: no branches inside a step)
  const int ntiles = Nr / 16 * ntj, per_wave = (ntiles + 7) / 8, id0 = w * per_wave, id1 = min(id0 + per_wave, ntiles);
  int ti[TPW], tj[TPW];
#pragma unroll
  for (int q = 0; q < TPW; q++) {
    const int id = min(id0 + q, ntiles - 1);
    ti[q] = id / ntj;
    tj[q] = id - ti[q] * ntj;
  }
  f32x4 acc[TPW];
#pragma unroll
  for (int q = 0; q < TPW; q++) acc[q] = (f32x4){0.f, 0.f, 0.f, 0.f};
  auto products = [&](int s, int ring, auto nh) {
    if (id0 >= ntiles) return;  // (uniform)
    const char *stage = lds + ring * stage_bytes;
    const T *src = reinterpret_cast<const T *>((uint32_t)(s - k0) < (uint32_t)own ? kept + (s - k0) * kept_bytes : stage);
    const T *dst = reinterpret_cast<const T *>(stage + Nr * 128);
#pragma unroll
    for (int h = 0; h < decltype(nh)::value; h++) {
#pragma unroll
      for (int q = 0; q < TPW; q++) {
        Frag<T> fa, fb;
        frag_load_kc_sw(fa, src, 16 * ti[q] + c, 32 * h + 8 * g);
        frag_load_kc_sw(fb, dst, 16 * tj[q] + c, 32 * h + 8 * g);
        mma16(acc[q], fa, fb);  // lane: destination c, sources 4 g + r
      }
    }
  };
  wait_vmcnt<0>();
#pragma unroll
  for (int s = 0; s < ST - 1; s++)
    if (s < steps) issue(s, s);
  // rows that pad the slice's tiles to whole fragments
  for (int e = tid; e < (k1 - k0) * (Nrp - Nr) * 8; e += 512) {
    const int per = (Nrp - Nr) * 8, st = e / per, q = e - st * per;
    *reinterpret_cast<u32x4 *>(kept + (size_t)st * Nrp * 128 + (size_t)Nr * 128 + q * 16) = (u32x4){0u, 0u, 0u, 0u};
  }
  const int whole = steps - (tail == 64 ? 1 : 0);
  int s = 0, ring = 0;
  for (; s + ST - 1 < steps; s++) {
    // step s has landed (the ST - 2 after it may be in flight), and every wave is done with step s - 1
    wait_vmcnt<NL * (ST - 2)>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    issue(s + ST - 1, ring == 0 ? ST - 1 : ring - 1);
    products(s, ring, std::integral_constant<int, NH>{});
    ring = ring == ST - 1 ? 0 : ring + 1;
  }
  wait_vmcnt<0>();
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  for (; s < whole; s++) {
    products(s, ring, std::integral_constant<int, NH>{});
    ring = ring == ST - 1 ? 0 : ring + 1;
  }
  if (s < steps) products(s, ring, std::integral_constant<int, 1>{});
  __syncthreads();  // the ring's room is free

  // ---- softmax over the destinations of every source; weights destination-major in LDS ----
  float *lg = reinterpret_cast<float *>(lds);
  const int ldl = Drp + 1, ldp = Nrp + EPP;
  T *P = reinterpret_cast<T *>(lds + (((size_t)Nr * ldl * 4 + 15) & ~(size_t)15));
#pragma unroll
  for (int q = 0; q < TPW; q++) {
    if (id0 + q < id1) {
#pragma unroll
      for (int r = 0; r < 4; r++) lg[(16 * ti[q] + 4 * g + r) * ldl + 16 * tj[q] + c] = acc[q][r];
    }
  }
  __syncthreads();
  const float k2 = scale * 1.44269504088896341f;
  for (int s = tid >> 3; s < Nrp; s += 64) {  // eight lanes per source
    const float *row = lg + s * ldl;
    const bool live = s < Nr;
    float m = -__builtin_inff();
    if (live)
      for (int j = tid & 7; j < Dr; j += 8) m = fmaxf(m, row[j]);
    m = fmaxf(m, dpp_f32<0xB1>(m));
    m = fmaxf(m, dpp_f32<0x4E>(m));
    m = fmaxf(m, __shfl_xor(m, 4, 64));
    const float mk = m * k2;
    float sum = 0.f;
    if (live)
      for (int j = tid & 7; j < Dr; j += 8) sum += __builtin_amdgcn_exp2f(fmaf(row[j], k2, -mk));
    sum += dpp_f32<0xB1>(sum);
    sum += dpp_f32<0x4E>(sum);
    sum += __shfl_xor(sum, 4, 64);
    const float inv = 1.0f / sum;
    for (int j = tid & 7; j < Drp; j += 8)
      P[j * ldp + s] = from_f32<T>(live && j < Dr ? __builtin_amdgcn_exp2f(fmaf(row[j], k2, -mk)) * inv : 0.f);
  }
  __syncthreads();

  // ---- the weights leave, the rows shared out over the region's slices ----
  {
    const int cpr = Nr / EPP;
    for (int e = tid; e < (Dr - slice + slices - 1) / slices * cpr; e += 512) {
      const int j = slice + e / cpr * slices, u = e % cpr;
      *reinterpret_cast<u32x4 *>(A + ((size_t)z * Dr + j) * Nr + u * EPP) = *reinterpret_cast<const u32x4 *>(P + j * ldp + u * EPP);
    }
  }
  // ---- merge of this slice: 16 destinations x 16 channels per product, K over the sources ----
  Frag<T> ones;
#pragma unroll
  for (int e = 0; e < 8; e++) ones.v[e] = from_f32<T>(1.0f);
  const int nct = (k1 - k0) * CPS;
  for (int id = w; id < nct * ntj; id += 8) {
    const int ct = id / ntj, tj = id - ct * ntj, st = ct / CPS, nb = (ct - st * CPS) * 16;
    const T *x = reinterpret_cast<const T *>(kept + (size_t)st * Nrp * 128);
    f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f}, rs = o;
    for (int kk = 0; kk < Nrp / 32; kk++) {
      Frag<T> fa, fb;
      frag_load_kc(fa, P + (16 * tj + c) * ldp + 32 * kk + 8 * g);
      const int ra = 32 * kk + 8 * g;
      typedef s16x4 __attribute__((address_space(3))) *lds_s16x4_ptr;
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      const int r = ra + (c >> 2), col = nb + 4 * (c & 3);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(x + SwzTile<T>::kc(r, col >> 3) + (col & 7)));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(x + SwzTile<T>::kc(r + 4, col >> 3) + (col & 7)));
      const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      fb.v = __builtin_bit_cast(bf16x8, both);
      mma16(o, fb, fa);    // lane: destination c, channels 4 g + r
      mma16(rs, ones, fa);  // the destination's row sum
    }
    const int m = 16 * tj + c, n = (k0 + st) * EPS + nb + 4 * g;
    if (m < Dr) {
      if (ct == 0 && k0 == 0 && g == 0) Z[(size_t)b * v.D + rho * Dr + m] = rs[0];
      if (n < C) store4<T>(Xm + ((size_t)b * v.D + rho * Dr + m) * C + n, o * (1.0f / fmaxf(rs[0], 1e-20f)));
    }
  }
}

// Where it pays.  In us, fitted to traces of both over regions of 16 to 192 tokens with 1 to 8 tiles per wave, widths of
// 64 to 1280 and grids of up to 1280 workgroups: per round of one or two workgroups per CU, a fixed part, the softmax and
// the K steps; against the fixed cost of four or five kernels, their K steps, the passes over X and a block tile at least
// per region.  Both sides at the line: 144 tokens with 72 destinations, width 1280, 32 regions 35.7 and 40.1, 128 regions
// (four rounds) 118 and 74; 128 with 112, width 1280, 35.3 and 31.6.  Destinations in one block of 128 have a one-pass
// kernel (128 tokens with 128: 11 us against 15).
bool local_merge_fits(const Shape &s) {
  const int regions = s.B * s.R;
  LocalPlan p;
  if (s.dtype != TOMA_BF16 || !plan_local(regions, s.Nr, s.Dr, s.C, &p)) return false;
  if (weights_single_pass(s.Nr, s.Dr, s.C, regions, 2)) return false;
  const int per_wave = (p.nti * p.ntj + 7) / 8, at_once = p.lds <= (size_t)kLocalLds2 ? 512 : 256;
  const double rounds = (double)(((long long)regions * p.slices + at_once - 1) / at_once), mb = (double)s.B * s.N * s.C * 2e-6;
  const double here = rounds * (5.0 + 1.2 * per_wave + p.steps * (0.25 + 0.1 * per_wave));
  return here < 0.95 * (17.0 + 0.55 * p.steps + 0.6 * mb + 0.03 * regions);
}

int launch_local_merge(const Shape &s, const void *X, const int32_t *idx, void *A, float *Z, void *Xm, hipStream_t st) {
  LocalPlan p;
  if (s.dtype != TOMA_BF16 || !plan_local(s.B * s.R, s.Nr, s.Dr, s.C, &p)) return TOMA_ERR_UNSUPPORTED;
  const RegionView<bf16_t> v = make_view<bf16_t>(s, X);
  const int rows = s.Nr + 16 * p.ntj, per_wave = (p.nti * p.ntj + 7) / 8;
  const dim3 grid((unsigned)(s.B * s.R * p.slices));
  KernelTimer kt(K_LOCAL_MERGE, st);
#define TOMA_LOCAL_LDS(NL, TPW, ST, LDSB)                                                                           \
  hipLaunchKernelGGL((k_local_merge<NL, TPW, ST, LDSB>), grid, dim3(512), 0, st, v, idx, s.scale,                    \
                     static_cast<bf16_t *>(A), Z, static_cast<bf16_t *>(Xm), p.ntj, p.slices, p.per_slice, (int)p.ring)
#define TOMA_LOCAL(NL, TPW, ST)                                                                                     \
  do {                                                                                                              \
    if (p.lds <= (size_t)kLocalLds2) TOMA_LOCAL_LDS(NL, TPW, ST, kLocalLds2);                                       \
    else TOMA_LOCAL_LDS(NL, TPW, ST, kLocalLds);                                                                    \
  } while (0)
  if (rows <= 64 && per_wave <= 1 && p.stages == 4) TOMA_LOCAL(1, 1, 4);
  else if (rows <= 128 && per_wave <= 2 && p.stages == 4) TOMA_LOCAL(2, 2, 4);
  else if (rows <= 192 && per_wave <= 4 && p.stages == 3) TOMA_LOCAL(3, 4, 3);
  else if (per_wave <= 6 && p.stages == 3) TOMA_LOCAL(4, 6, 3);
  else if (per_wave <= 8 && p.stages == 3) TOMA_LOCAL(4, 8, 3);
  else return TOMA_ERR_UNSUPPORTED;
#undef TOMA_LOCAL_LDS
#undef TOMA_LOCAL
  return launch_status();
}

}  // namespace toma

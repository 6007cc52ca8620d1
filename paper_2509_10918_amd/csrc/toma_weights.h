// Products of 32 source rows with gathered destination rows, the inner loop of the merge weights.
// A K step is 128 bytes of every row: two 32-channel fragments (bf16) or one (fp32).  A destination
// row is used by one wave only: every wave streams its own rows through a PRIVATE ring of LDS
// stages (up to two MFMA tiles = 4 KiB each) with the load-to-LDS path, three stages ahead of the
// products, and only its own s_waitcnt orders them.  The 32 source rows of a step are shared: four
// waves fetch them, three steps ahead, and the workgroup meets once per K step.
#pragma once
#include "toma_gemm.h"
#include "toma_region.h"

namespace toma {

// LDS of the product: a private ring of stages per wave (sized for two tiles per stage) and a ring of the steps' 32
// source rows.
template <typename T> struct WeightsLds {
  static constexpr int EPS = 128 / (int)sizeof(T);  // elements per K step
  T b[8][4][2 * 16 * EPS];
  T a[4][32 * EPS];
};
// acc[i][j]: products of source rows 16 i + 4 g + r of the block at m0 with the wave's destination tile j, whose 16 rows
// are the tokens token(j, 0) .. token(j, 15)
template <typename T, int NJ, typename TokenFn>
__device__ __forceinline__ void weights_products(f32x4 (&acc)[2][NJ], WeightsLds<T> &lds, const RegionView<T> &v,
                                                 int b, int rho, int m0, TokenFn token) {
  constexpr int ES = (int)sizeof(T), EPS = 128 / ES;   // elements per K step
  constexpr int EPP = 16 / ES;
  constexpr int NH = ES == 2 ? 2 : 1;                  // fragments per row per K step
  constexpr int JS = NJ < 2 ? 1 : 2;                   // MFMA tiles per stage
  constexpr int SPS = NJ / JS;                         // stages per K step
  constexpr int RS = 4;                                // ring stages per wave
  constexpr int LPS = 2 * JS;                          // load instructions (1 KiB) per stage
  T(&Bs)[8][4][2 * 16 * EPS] = lds.b;
  T(&As)[4][32 * EPS] = lds.a;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, g = lane >> 4, c = lane & 15;
  const T *Xb = v.X + (size_t)b * v.N * v.C;
  // what this lane fetches of a 1 KiB chunk (8 rows x 128 bytes): row lane / 8, and the packet that
  // the swizzle places at position lane % 8 of that row
  const int l_row = lane >> 3;
  const int l_pkt = ((lane & 7) ^ (l_row & 7)) * EPP;
  // Element offsets (inside the sample) of the packets this lane fetches of its wave's destination
  // rows, one per (stage of a K step, chunk): the same for every K step, so they stay in registers.
  int roff[SPS][LPS];
#pragma unroll
  for (int q = 0; q < SPS; q++)
#pragma unroll
    for (int ch = 0; ch < LPS; ch++) {
      roff[q][ch] = token(q * JS + (ch >> 1), 8 * (ch & 1) + l_row) * v.C + l_pkt;
    }
  // source rows: wave w < 4 fetches rows 8 w .. 8 w + 7 of every step
  const T *a_src = Xb + (size_t)v.token(rho, min(m0 + 8 * (w & 3) + l_row, v.Nr - 1)) * v.C + l_pkt;
  const int nsteps = v.C / EPS, U = nsteps * SPS;
  // LDS byte addresses (scalar registers) of this wave's ring and of its part of the source rows
  const uint32_t w_s = (uint32_t)__builtin_amdgcn_readfirstlane(w);
  const uint32_t bs_lds = lds_addr_of(&Bs[0][0][0]) + w_s * (RS * 2 * 16 * EPS * ES);
  const uint32_t as_lds = lds_addr_of(&As[0][0]) + (w_s & 3) * 1024;
  auto issue_a = [&](int s) { load_to_lds16_at(a_src + s * EPS, as_lds + (uint32_t)(s & 3) * (32 * EPS * ES)); };
  // stage u = s * SPS + q of the ring (q is a compile-time constant at every call)
  auto issue_b = [&](int s, int q) {
    const uint32_t dst = bs_lds + (uint32_t)((s * SPS + q) & (RS - 1)) * (2 * 16 * EPS * ES);
    const T *src = Xb + s * EPS;
#pragma unroll
    for (int ch = 0; ch < LPS; ch++) load_to_lds16_at(src + roff[q][ch], dst + ch * 1024);
  };
  auto fence = [&]() { asm volatile("" ::: "memory"); };

#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < NJ; j++) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

  // the index loads above have returned (their values were used): from here on vmcnt counts
  // only ring loads
  wait_vmcnt<0>();
  if (w < 4) {
#pragma unroll
    for (int s = 0; s < 3; s++)
      if (s < nsteps) issue_a(s);
  }
#pragma unroll
  for (int u = 0; u < RS - 1; u++)
    if (u < U) issue_b(u / SPS, u % SPS);
  wait_vmcnt<0>();
  fence();
  __builtin_amdgcn_s_barrier();
  fence();

  for (int s = 0; s < nsteps; s++) {
    if (w < 4 && s + 3 < nsteps) issue_a(s + 3);  // (the slot of step s - 1, which every wave is done with)
    Frag<T> fa[2][NH];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int h = 0; h < NH; h++) frag_load_kc_sw(fa[i][h], As[s & 3], 16 * i + c, 32 * h + 8 * g);
#pragma unroll
    for (int q = 0; q < SPS; q++) {
      const int u = s * SPS + q;
      if (u + RS - 1 < U) issue_b(s + (q + RS - 1) / SPS, (q + RS - 1) % SPS);
      // this wave's loads of stage u are the oldest outstanding ones
      // (short steps: as many source rows are in flight behind it; elsewhere the wait covers them too)
      const int younger = min(U - 1 - u, RS - 1);
      if (SPS == 1 && w < 4) {
        if (younger >= 3) wait_vmcnt<3 * (LPS + 1)>();
        else if (younger == 2) wait_vmcnt<2 * (LPS + 1)>();
        else if (younger == 1) wait_vmcnt<LPS + 1>();
        else wait_vmcnt<0>();
      } else {
        if (younger >= 3) wait_vmcnt<3 * LPS>();
        else if (younger == 2) wait_vmcnt<2 * LPS>();
        else if (younger == 1) wait_vmcnt<LPS>();
        else wait_vmcnt<0>();
      }
      fence();
      const T *bt = Bs[w][u & (RS - 1)];
#pragma unroll
      for (int t = 0; t < JS; t++)
#pragma unroll
        for (int h = 0; h < NH; h++) {
          Frag<T> fb;
          frag_load_kc_sw(fb, bt, 16 * t + c, 32 * h + 8 * g);
#pragma unroll
          for (int i = 0; i < 2; i++) mma16(acc[i][q * JS + t], fa[i][h], fb);
        }
      // the fragment reads of this stage have returned before its slot is refilled (next trip)
      __builtin_amdgcn_s_waitcnt(0xc07f);
      fence();
    }
    // The next step's source rows have landed - two steps and this one issued loads after them, where there were any
    // left to issue - and every wave is done with this step's.
    constexpr int kAfterA = 2 + 3 * SPS * LPS < 60 ? 2 + 3 * SPS * LPS : 60;
    if ((s + 1) * SPS + RS - 1 <= U && s + 3 < nsteps) wait_vmcnt<kAfterA>();
    else wait_vmcnt<0>();
    fence();
    __builtin_amdgcn_s_barrier();
    fence();
  }
}

}  // namespace toma

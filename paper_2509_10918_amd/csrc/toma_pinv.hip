// Moore-Penrose unmerge (paper Sec. 4.2.2, first display): Y = A~^+ X' with A~ = A / Z the
// row-normalised merge matrix of a merge region (Dr destinations x Nr sources, Dr <= 128) and A~^+ its
// pseudo-inverse with singular values <= rcond * largest treated as zero.  The paper measures this
// against the transpose unmerge and rejects it for its cost; it is here so that the comparison can be
// made on this hardware too.
//
//   A~^+ = A~^T (A~ A~^T)^+ :  G = A~ A~^T is Dr x Dr, symmetric, positive semi-definite.
//   k_pinv_eig    one workgroup per (sample, merge region): G in double precision in LDS, its
//                 eigen-decomposition G = V diag(lambda) V^T by cyclic Jacobi rotations (every
//                 sweep rotates all pairs, up to 64 disjoint pairs at a time in round-robin order), then
//                 G^+ = sum over lambda_k > rcond^2 lambda_max of v_k v_k^T / lambda_k  (lambda =
//                 sigma^2, so this is the singular-value rule).  Rank deficiency of any kind - rows of
//                 A~ that are zero because nobody chose a destination, duplicated or nearly dependent
//                 rows - ends up as eigenvalues below the cut.
//   k_pinv_apply  one workgroup per (region, 32 channels): w = G^+ X' (double), then
//                 Y[token(s)] = sum_j A_js w_j / Z_j, written at the tokens' grid positions; both products
//                 on the fp64 matrix cores.
// Everything between the stored operands and the rounding of Y is double precision: the merge
// matrices of a small temperature have a few singular values of 1e-4 ... 1e-12 next to a bulk in
// [0.2, 1], and the cut has to tell them apart.
#include <algorithm>

#include "toma_common.h"
#include "toma_internal.h"

namespace toma {

constexpr int kPinvMax = 128;            // destinations per merge region this path takes
constexpr int kPinvThreads = 1024;       // (at most; pinv_threads)
constexpr int kPinvChunk = 16;           // sources per staging step of G = A A^T

template <typename T> struct PinvView {
  const T *A;          // [B*R][Dr][Nr]
  const float *Z;      // [B][D]
  RegionMap map;
  int N, C, D, R, Nr, Dr, n_loc;
  // grid index of source s of merge region rho (sources region by region, local order inside)
  __device__ __forceinline__ int token(int rho, int s) const {
    return R != 1 ? map.token(rho, s) : map.token(s / n_loc, s % n_loc);
  }
};

__device__ __forceinline__ double wave_sum_f64(double v) {
  v += __shfl_xor(v, 1, 64); v += __shfl_xor(v, 2, 64); v += __shfl_xor(v, 4, 64);
  v += __shfl_xor(v, 8, 64); v += __shfl_xor(v, 16, 64); v += __shfl_xor(v, 32, 64);
  return v;
}

// (row, column) of the elements tid, tid + nthreads, ... of a matrix of `cols` columns, without a division
// per element
struct RowCol {
  int i, j;
  const int cols, di, dj;
  __device__ __forceinline__ RowCol(int tid, int nthreads, int cols_)
      : i(tid / cols_), j(tid % cols_), cols(cols_), di(nthreads / cols_), dj(nthreads % cols_) {}
  __device__ __forceinline__ void next() {
    i += di; j += dj;
    if (j >= cols) { j -= cols; i++; }
  }
};

// Jacobi rotation of the pair with diagonal app, aqq and coupling apq.  The angle only has to be close (what
// is left of apq goes in the next sweep), so it is taken from the hardware's reciprocal and reciprocal root,
// about 2^-26; c = 1 / sqrt(1 + t^2) gets two Newton steps and s = t c, so that c^2 + s^2 = 1 to the last bits
// and V stays orthogonal.
__device__ __forceinline__ void jacobi_rotation(double app, double aqq, double apq, double &c, double &s) {
  const double th = 0.5 * (aqq - app) * __builtin_amdgcn_rcp(apq), ath = fabs(th), h = ath * ath + 1.0;
  const double t1 = ath < 1e8 ? __builtin_amdgcn_rcp(ath + h * __builtin_amdgcn_rsq(h)) : 0.5 * __builtin_amdgcn_rcp(ath);
  const double t = th >= 0.0 ? t1 : -t1, u = t * t + 1.0;
  double y = __builtin_amdgcn_rsq(u);
  y = y * (1.5 - 0.5 * u * y * y);
  y = y * (1.5 - 0.5 * u * y * y);
  c = y;
  s = t * y;
}

// The rounds of a sweep are a serial chain (rotations from the diagonal, barrier, update, barrier), and that
// chain bounds the kernel: so a round updates every 2 x 2 block of G from both sides at once - block (k, l)
// holds the rows of pair k and the columns of pair l, which no other block touches - together with the
// eigenvector rows, and the workgroup has no more waves than the blocks need.  V_LDS: G and V^T both fit the
// LDS (Dr <= 96); above that V^T stays in global memory.  SDXL-2's regions (Dr = 32, 32 workgroups): 79 us with
// rows and columns in turn, V^T in global memory and 1024 threads, 58 us so.
template <typename T, bool V_LDS>
__global__ __launch_bounds__(kPinvThreads) void k_pinv_eig(const PinvView<T> v, double rcond, double *__restrict__ Vt_all,
                                                          double *__restrict__ Ginv_all) {
  // G with a padded row stride (column walks would otherwise hit one bank)
  extern __shared__ __align__(16) double lds[];
  const int n = v.Dr, LD = n + 1, nthr = blockDim.x;
  const int np = n + (n & 1), m = np - 1, half = np / 2;  // an odd n plays against a dummy that never rotates
  double *G = lds;                                        // [n][LD]
  double *stage = G + (size_t)n * LD;                     // [kPinvChunk][n] weights of the current sources, as doubles
  double *rot_cs = stage + (size_t)n * kPinvChunk;        // [half][2]: c, s of the round's rotations
  double *red = rot_cs + 2 * half;                        // [kPinvThreads / 64][2]
  int *rot_pq = reinterpret_cast<int *>(red + 2 * (kPinvThreads / 64));  // [half][2]: p, q
  double *v_lds = red + 2 * (kPinvThreads / 64) + half;   // [n][n] with V_LDS
  const int tid = threadIdx.x, z = blockIdx.x, b = z / v.R, rho = z % v.R;
  const T *A = v.A + (size_t)z * n * v.Nr;
  const float *Zr = v.Z + (size_t)b * v.D + (size_t)rho * n;
  double *Vt = V_LDS ? v_lds : Vt_all + (size_t)z * n * n, *Ginv = Ginv_all + (size_t)z * n * n;

  // ---- G = diag(1/Z) A A^T diag(1/Z) ----
  for (RowCol e(tid, nthr, n); e.i < n; e.next()) {
    G[e.i * LD + e.j] = 0.0;
    Vt[e.i * n + e.j] = e.i == e.j ? 1.0 : 0.0;
  }
  for (int s0 = 0; s0 < v.Nr; s0 += kPinvChunk) {
    __syncthreads();
    for (int e = tid; e < n * kPinvChunk; e += nthr) {
      const int j = e / kPinvChunk, s = e % kPinvChunk;
      stage[s * n + j] = s0 + s < v.Nr ? (double)to_f32(A[(size_t)j * v.Nr + s0 + s]) : 0.0;
    }
    __syncthreads();
    for (RowCol e(tid, nthr, n); e.i < n; e.next()) {
      if (e.j < e.i) continue;  // upper triangle; mirrored below
      double acc = 0.0;
#pragma unroll
      for (int s = 0; s < kPinvChunk; s++) acc += stage[s * n + e.i] * stage[s * n + e.j];
      G[e.i * LD + e.j] += acc;
    }
  }
  __syncthreads();
  for (RowCol e(tid, nthr, n); e.i < n; e.next()) {
    if (e.j < e.i) continue;
    const double g = G[e.i * LD + e.j] / ((double)fmaxf(Zr[e.i], 1e-20f) * (double)fmaxf(Zr[e.j], 1e-20f));
    G[e.i * LD + e.j] = g;
    G[e.j * LD + e.i] = g;
  }
  __syncthreads();

  // ---- cyclic Jacobi: G <- J^T G J, V <- V J for every pair (p, q), until the off-diagonal part is gone ----
  for (int sweep = 0; sweep < 40; sweep++) {
    double off = 0.0, dia = 0.0;
    for (RowCol e(tid, nthr, n); e.i < n; e.next()) {
      const double g = G[e.i * LD + e.j];
      if (e.i == e.j) dia += g * g; else off += g * g;
    }
    off = wave_sum_f64(off);
    dia = wave_sum_f64(dia);
    if ((tid & 63) == 0) { red[2 * (tid >> 6)] = off; red[2 * (tid >> 6) + 1] = dia; }
    __syncthreads();
    off = 0.0; dia = 0.0;
    for (int i = 0; i < nthr / 64; i++) { off += red[2 * i]; dia += red[2 * i + 1]; }  // fixed order
    if (off <= 1e-26 * dia || dia == 0.0) break;  // uniform: every thread holds the same sums
    for (int r = 0; r < m; r++) {
      if (tid < half) {
        int p = r + tid, q = r - tid;
        if (p >= m) p -= m;
        if (q < 0) q += m;
        if (tid == 0) p = m;
        double c = 1.0, s = 0.0;
        if (p < n && q < n) {
          const double apq = G[p * LD + q], app = G[p * LD + p], aqq = G[q * LD + q];
          if (fabs(apq) > 1e-300 && apq * apq > 1e-40 * fabs(app * aqq)) jacobi_rotation(app, aqq, apq, c, s);
        } else {
          p = q = -1;
        }
        rot_pq[2 * tid] = p; rot_pq[2 * tid + 1] = q;
        rot_cs[2 * tid] = c; rot_cs[2 * tid + 1] = s;
      }
      __syncthreads();
      // the 2 x 2 blocks of G <- J^T G J
      for (RowCol e(tid, nthr, half); e.i < half; e.next()) {
        const double ck = rot_cs[2 * e.i], sk = rot_cs[2 * e.i + 1], cl = rot_cs[2 * e.j], sl = rot_cs[2 * e.j + 1];
        if (sk == 0.0 && sl == 0.0) continue;
        const int pk = rot_pq[2 * e.i], qk = rot_pq[2 * e.i + 1], pl = rot_pq[2 * e.j], ql = rot_pq[2 * e.j + 1];
        if (n & 1) {
          // the pair with the dummy: its one real row or column (the partner of the round) only turns from the other side
          const int ok = pk < 0 ? r : pk, ol = pl < 0 ? r : pl;
          if (pk < 0 && pl < 0) continue;
          if (pk < 0) {
            const double gp = G[ok * LD + pl], gq = G[ok * LD + ql];
            G[ok * LD + pl] = cl * gp - sl * gq;
            G[ok * LD + ql] = sl * gp + cl * gq;
            continue;
          }
          if (pl < 0) {
            const double gp = G[pk * LD + ol], gq = G[qk * LD + ol];
            G[pk * LD + ol] = ck * gp - sk * gq;
            G[qk * LD + ol] = sk * gp + ck * gq;
            continue;
          }
        }
        const double gpp = G[pk * LD + pl], gpq = G[pk * LD + ql], gqp = G[qk * LD + pl], gqq = G[qk * LD + ql];
        const double hpp = ck * gpp - sk * gqp, hqp = sk * gpp + ck * gqp;  // rows
        const double hpq = ck * gpq - sk * gqq, hqq = sk * gpq + ck * gqq;
        G[pk * LD + pl] = cl * hpp - sl * hpq;                              // columns
        G[pk * LD + ql] = sl * hpp + cl * hpq;
        G[qk * LD + pl] = cl * hqp - sl * hqq;
        G[qk * LD + ql] = sl * hqp + cl * hqq;
      }
      // the same rotations on the eigenvector rows of V^T
      for (RowCol e(tid, nthr, n); e.i < half; e.next()) {
        const double s = rot_cs[2 * e.i + 1];
        if (s == 0.0) continue;
        const int p = rot_pq[2 * e.i], q = rot_pq[2 * e.i + 1];
        const double c = rot_cs[2 * e.i], vp = Vt[p * n + e.j], vq = Vt[q * n + e.j];
        Vt[p * n + e.j] = c * vp - s * vq;
        Vt[q * n + e.j] = s * vp + c * vq;
      }
      __syncthreads();
    }
  }

  // ---- G^+ = sum over the eigenvalues above the cut of v_k v_k^T / lambda_k ----
  double lmax = 0.0;
  for (int k = 0; k < n; k++) lmax = fmax(lmax, G[k * LD + k]);
  const double cut = rcond * rcond * lmax;
  __syncthreads();  // (the rotations' last writes of V^T are visible to the whole workgroup)
  for (int k = tid; k < n; k += nthr) {
    const double l = G[k * LD + k];
    stage[k] = (l > cut && l > 0.0) ? 1.0 / l : 0.0;
  }
  __threadfence_block();
  __syncthreads();
  for (RowCol e(tid, nthr, n); e.i < n; e.next()) {
    double acc = 0.0;
    for (int k = 0; k < n; k++) acc += Vt[k * n + e.i] * Vt[k * n + e.j] * stage[k];
    Ginv[e.i * n + e.j] = acc;
  }
}

constexpr int kPinvCols = 32;              // channels per workgroup of the apply kernel
constexpr int kPinvLd = kPinvCols + 16;    // row stride of its LDS tile: two k-groups of a fragment fall on different banks

// Both products on v_mfma_f64_16x16x4_f64 (operands: row or column = lane % 16, k = lane / 16; result: column
// lane % 16, rows lane / 16 + 4 r).  The scalar loops this replaces (one fp64 multiply-add per LDS read, in one
// serial chain) took 52 us on SDXL-2's 32 regions x 40 channel blocks, these take 17 us.
template <typename T>
__global__ __launch_bounds__(256) void k_pinv_apply(const PinvView<T> v, const double *__restrict__ Ginv_all,
                                                   const T *__restrict__ O, int o_rows, T *__restrict__ Y) {
  extern __shared__ __align__(16) double xs[];  // [n rounded up to 16][kPinvLd]: X' chunk, then w = G^+ X' / Z in its place
  const int n = v.Dr, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, g = lane >> 4, c16 = lane & 15;
  const int tiles = (n + 15) / 16;
  const int z = blockIdx.y, b = z / v.R, rho = z % v.R, c0 = blockIdx.x * kPinvCols;
  const double *Ginv = Ginv_all + (size_t)z * n * n;
  const float *Zr = v.Z + (size_t)b * v.D + (size_t)rho * n;
  for (int e = tid; e < 16 * tiles * kPinvCols; e += 256) {
    const int j = e / kPinvCols, c = e % kPinvCols;
    xs[j * kPinvLd + c] =
        j < n && c0 + c < v.C ? (double)to_f32(O[((size_t)b * o_rows + (size_t)rho * n + j) * v.C + c0 + c]) : 0.0;
  }
  __syncthreads();
  constexpr int kPer = kPinvMax / 16 * (kPinvCols / 16) / 4;  // 16 x 16 tiles of w per wave
  f64x4 acc[kPer];
#pragma unroll
  for (int u = 0; u < kPer; u++) {
    const int t = wv + 4 * u, i0 = 16 * (t >> 1), ct = 16 * (t & 1);
    acc[u] = (f64x4){0.0, 0.0, 0.0, 0.0};
    if (i0 >= n) continue;  // (wave-uniform)
    const bool row_ok = i0 + c16 < n;
    for (int k0 = 0; k0 < n; k0 += 16) {
      double a[4];
#pragma unroll
      for (int q = 0; q < 4; q++) {  // G^+ is symmetric: sixteen consecutive words of row k
        const int k = k0 + 4 * q + g;
        a[q] = row_ok && k < n ? Ginv[(size_t)k * n + i0 + c16] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < 4; q++)
        acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], xs[(k0 + 4 * q + g) * kPinvLd + ct + c16], acc[u], 0, 0, 0);
    }
  }
  __syncthreads();
  int finite = 1;
#pragma unroll
  for (int u = 0; u < kPer; u++) {
    const int t = wv + 4 * u, i0 = 16 * (t >> 1), ct = 16 * (t & 1);
    if (i0 >= n) continue;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int i = i0 + g + 4 * r;
      const double w = i < n ? acc[u][r] / (double)fmaxf(Zr[i], 1e-20f) : 0.0;
      finite &= fabs(w) <= 1.7976931348623157e308;
      xs[i * kPinvLd + ct + c16] = w;
    }
  }
  finite = __syncthreads_and(finite);
  const T *A = v.A + (size_t)z * n * v.Nr;
  if (finite) {
    // a wave takes sixteen sources and all 32 channels
    for (int s0 = 16 * wv; s0 < v.Nr; s0 += 64) {
      const bool src_ok = s0 + c16 < v.Nr;
      f64x4 y[2] = {(f64x4){0.0, 0.0, 0.0, 0.0}, (f64x4){0.0, 0.0, 0.0, 0.0}};
      for (int j0 = 0; j0 < n; j0 += 16) {
        double a[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const int j = j0 + 4 * q + g;
          a[q] = src_ok && j < n ? (double)to_f32(A[(size_t)j * v.Nr + s0 + c16]) : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
          for (int h = 0; h < 2; h++)
            y[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], xs[(j0 + 4 * q + g) * kPinvLd + 16 * h + c16], y[h], 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int s = s0 + g + 4 * r;
        if (s >= v.Nr) continue;
        T *dst = Y + ((size_t)b * v.N + v.token(rho, s)) * v.C + c0 + c16;
#pragma unroll
        for (int h = 0; h < 2; h++)
          if (c0 + 16 * h + c16 < v.C) dst[16 * h] = from_f32<T>((float)y[h][r]);
      }
    }
    return;
  }
  // an infinity or NaN among the w: a weight of zero must not meet it (0 * inf), so zeros are passed over
  for (int e = tid; e < v.Nr * kPinvCols; e += 256) {
    const int s = e / kPinvCols, c = e % kPinvCols;
    if (c0 + c >= v.C) continue;
    double acc1 = 0.0;
    for (int j = 0; j < n; j++) {
      const double a = (double)to_f32(A[(size_t)j * v.Nr + s]);
      if (a != 0.0) acc1 += a * xs[j * kPinvLd + c];
    }
    Y[((size_t)b * v.N + v.token(rho, s)) * v.C + c0 + c] = from_f32<T>((float)acc1);
  }
}

size_t pinv_workspace_bytes(const Shape &s) {
  if (s.Dr > kPinvMax) return 0;
  return (size_t)2 * s.B * s.R * s.Dr * s.Dr * sizeof(double);
}

template <typename T>
static int pinv_typed(const Shape &s, const void *A, const float *Z, const void *O, int o_rows, float rcond, void *Y,
                      char *ws, const Workspace &w, hipStream_t st) {
  PinvView<T> v;
  v.A = static_cast<const T *>(A); v.Z = Z;
  v.map = RegionMap{s.W, s.tile_h, s.tile_w, s.W / s.tile_w};
  v.N = s.N; v.C = s.C; v.D = s.D; v.R = s.R; v.Nr = s.Nr; v.Dr = s.Dr; v.n_loc = s.n_loc;
  double *Vt = reinterpret_cast<double *>(ws + w.pinv);
  double *Ginv = Vt + (size_t)s.B * s.R * s.Dr * s.Dr;
  const int n = s.Dr, half = (n + 1) / 2;
  const size_t lds_g = sizeof(double) * ((size_t)n * (n + 1) + (size_t)n * kPinvChunk + 2 * half + 2 * (kPinvThreads / 64) + half);
  const size_t lds_v = sizeof(double) * (size_t)n * n;
  // V^T beside G where both fit; the workgroup has a thread for every 2 x 2 block, within 256 to 1024
  const bool v_lds = n <= 96;
  const size_t lds = lds_g + (v_lds ? lds_v : 0);
  const int threads = std::min(kPinvThreads, std::max(256, (half * half + 63) / 64 * 64));
  auto *kern = v_lds ? k_pinv_eig<T, true> : k_pinv_eig<T, false>;
  // (more than 64 KiB of dynamic LDS has to be granted per kernel)
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
      hipSuccess)
    return TOMA_ERR_LAUNCH;
  {
    KernelTimer kt(K_PINV_EIG, st);
    hipLaunchKernelGGL(kern, dim3(s.B * s.R), dim3(threads), lds, st, v, (double)rcond, Vt, Ginv);
  }
  {
    KernelTimer kt(K_PINV_APPLY, st);
    hipLaunchKernelGGL((k_pinv_apply<T>), dim3((s.C + kPinvCols - 1) / kPinvCols, s.B * s.R), dim3(256),
                       sizeof(double) * (size_t)((n + 15) / 16 * 16) * kPinvLd, st, v, Ginv, static_cast<const T *>(O), o_rows,
                       static_cast<T *>(Y));
  }
  return launch_status();
}

int launch_unmerge_pinv(const Shape &s, const void *A, const float *Z, const void *O, int o_rows, float rcond, void *Y,
                        char *ws, const Workspace &w, hipStream_t st) {
  if (s.Dr > kPinvMax) return TOMA_ERR_UNSUPPORTED;
  return s.dtype == TOMA_BF16 ? pinv_typed<bf16_t>(s, A, Z, O, o_rows, rcond, Y, ws, w, st)
                              : pinv_typed<float>(s, A, Z, O, o_rows, rcond, Y, ws, w, st);
}

}  // namespace toma

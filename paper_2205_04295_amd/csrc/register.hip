// Subpixel registration (Methods, "Adam-based position refinement": the
// 2-D phase correlation of Guizar-Sicairos et al. 2008, refined by a
// matrix-product DFT evaluated only around the coarse peak, no zero-padding)
// and the modified Adam step of Alg. 1 (Eq. 8-9), on gfx950.
//
// The whole registration runs in double precision so that its integer peaks
// (coarse lag and upsampled-window argmax) are those of an exact evaluation:
// float rounding of the 65536-term sums is larger than the gap between
// neighbouring samples near the peak of the upsampled surface.
//
// Pipeline for a batch of B (ref, mov) pairs of N x N complex64 patches:
//   k_reg_rows   row FFTs of ref and mov (complex128)
//   k_reg_cols   column FFTs, X = F(ref) conj(F(mov)) [phase-normalised],
//                stored; inverse column FFT of X
//   k_reg_coarse inverse row FFT -> |F^-1 X|^2, per-row first maximum
//   k_reg_s0     first maximum in row-major order -> signed integer lag s0
//   k_reg_gemm1  T = K (X . e^{2 pi i k.s0/N})   [U x N] x [N x N]
//   k_reg_gemm2  C = T K^T, per-tile first maximum of |C|^2
//   k_reg_final  window argmax (u*, v*) -> shift s0 + ((u*, v*) - c)/up
// (windows from 32 samples on: k_reg_fold, k_reg_fold1 and k_reg_fold2 for the
// two GEMMs, a quarter of the multiplications by symmetry, on matrix cores)
// with K[u][k] = exp(+2 pi i k (u - c) / (N up)), k the signed frequency,
// U = ceil(1.5 up), c = floor(U/2): the coarse lag is folded into X as a
// diagonal phase so one K serves every pair.
#include <algorithm>
#include <cmath>

#include "register.hpp"

namespace mrpie {

__device__ __forceinline__ int signed_freq(int k, int N) { return k < (N + 1) / 2 ? k : k - N; }

// first-maximum order: larger value first; equal values -> smaller index
__device__ __forceinline__ bool better(double v, long long i, double bv, long long bi) {
  return v > bv || (v == bv && i < bi);
}

struct ArgMax {
  double v;
  long long i;
};

// first-maximum argmax over one wave (all lanes get the result)
__device__ __forceinline__ ArgMax wave_argmax(double v, long long i) {
  for (int o = 32; o > 0; o >>= 1) {
    const double ov = __shfl_xor(v, o, 64);
    const long long oi = __shfl_xor(i, o, 64);
    if (better(ov, oi, v, i)) { v = ov; i = oi; }
  }
  return ArgMax{v, i};
}

// workgroup argmax with the first-maximum rule (all threads get the result)
__device__ __forceinline__ ArgMax block_argmax(double v, long long i, double* rv, long long* ri) {
  const ArgMax wm = wave_argmax(v, i);
  v = wm.v;
  i = wm.i;
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { rv[w] = v; ri[w] = i; }
  __syncthreads();
  ArgMax r{rv[0], ri[0]};
  for (int k = 1; k < nw; ++k)
    if (better(rv[k], ri[k], r.v, r.i)) { r.v = rv[k]; r.i = ri[k]; }
  return r;
}

// ---------------------------------------------------------------- FFT passes
// Row passes take kRegRW rows per workgroup (one wave per row at N = 256),
// so every thread of the workgroup has a butterfly in every radix-4 stage.
constexpr int kRegRW = 4;

template <int N>
__global__ __launch_bounds__(256) void k_reg_rows(const RegArgs a) {
  __shared__ double2 tw[N];
  __shared__ double2 A[kRegRW * N], B[kRegRW * N];
  const int r0 = blockIdx.x * kRegRW, b = blockIdx.y, which = blockIdx.z;
  const float2* src = (which == 0 ? a.ref : a.mov) + ((size_t)b * N + r0) * N;
  load_twiddles<N>(tw);
  for (int i = threadIdx.x; i < kRegRW * N; i += blockDim.x) {
    const float2 v = src[i];
    A[i] = make_double2((double)v.x, (double)v.y);
  }
  __syncthreads();
  double2* R = fft_lds<N, false>(A, B, kRegRW, tw);
  double2* dst = a.work + (((size_t)b * 2 + which) * N + r0) * N;
  for (int i = threadIdx.x; i < kRegRW * N; i += blockDim.x) dst[i] = R[i];
}

// CW adjacent columns per workgroup, so every access moves CW * 16
// contiguous bytes of a row; pixel q of the group is row k = q / CW, column
// c = q % CW.  LDS (dynamic): twiddles, then one buffer of 2 CW transforms
// (ref and mov of each column) transformed in place (the same butterflies
// as the ping-pong plan, half the LDS: twice the workgroups per CU).
constexpr int kRegCW = 4;
constexpr size_t reg_cols_lds(int N) { return (size_t)(N + 2 * kRegCW * N) * 16; }

template <int N>
__global__ __launch_bounds__(256) void k_reg_cols(const RegArgs a) {
  constexpr int CW = kRegCW, PIX = (N * CW + 255) / 256;
  extern __shared__ double2 dsm[];
  double2* tw = dsm;
  double2* A = tw + N;           // ref column c at c * N, mov at (CW + c) * N
  const int u0 = blockIdx.x * CW, b = blockIdx.y, tid = threadIdx.x;
  double2* w0 = a.work + (size_t)b * 2 * N * N;  // ref spectra -> later F^-1 over columns of X
  double2* w1 = w0 + (size_t)N * N;              // mov spectra -> later X
  load_twiddles<N>(tw);
#pragma unroll
  for (int i = 0; i < PIX; ++i) {
    const int q = tid + 256 * i, k = q / CW, c = q - k * CW;
    if (q >= N * CW) continue;
    A[c * N + k] = w0[(size_t)k * N + u0 + c];
    A[(CW + c) * N + k] = w1[(size_t)k * N + u0 + c];
  }
  __syncthreads();
  fft_lds_inplace<N, false, true, 2 * CW, 256>(A, 2 * CW, tw);
  const double2* F = A;
  double2* G = A;  // X over the ref transforms: each thread rewrites only the pixels it reads
#pragma unroll
  for (int i = 0; i < PIX; ++i) {
    const int q = tid + 256 * i, k = q / CW, c = q - k * CW;
    if (q >= N * CW) continue;
    double2 x = cmulc(F[c * N + k], F[(CW + c) * N + k]);  // F(ref) conj(F(mov))
    if (a.norm) {
      const double m = hypot(x.x, x.y);
      x = m > 0.0 ? make_double2(x.x / m, x.y / m) : make_double2(0.0, 0.0);
    }
    w1[(size_t)k * N + u0 + c] = x;
    G[c * N + k] = x;
  }
  __syncthreads();
  fft_lds_inplace<N, true, true, CW, 256>(G, CW, tw);
  const double2* H = G;
#pragma unroll
  for (int i = 0; i < PIX; ++i) {
    const int q = tid + 256 * i, k = q / CW, c = q - k * CW;
    if (q >= N * CW) continue;
    w0[(size_t)k * N + u0 + c] = H[c * N + k];
  }
}

// kRegRW rows per workgroup; wave w scans row r0 + w of the inverse
// transform for its first maximum (requires 64 kRegRW threads).
template <int N>
__global__ __launch_bounds__(256) void k_reg_coarse(const RegArgs a) {
  __shared__ double2 tw[N];
  __shared__ double2 A[kRegRW * N], B[kRegRW * N];
  const int r0 = blockIdx.x * kRegRW, b = blockIdx.y;
  const double2* src = a.work + ((size_t)b * 2 * N + r0) * N;
  load_twiddles<N>(tw);
  for (int i = threadIdx.x; i < kRegRW * N; i += blockDim.x) A[i] = src[i];
  __syncthreads();
  double2* R = fft_lds<N, true>(A, B, kRegRW, tw);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, r = r0 + w;
  double v = -1.0;
  long long idx = (long long)r * N + N;
  for (int i = lane; i < N; i += 64) {
    const double m = cabs2(R[w * N + i]);
    const long long ii = (long long)r * N + i;
    if (better(m, ii, v, idx)) { v = m; idx = ii; }
  }
  const ArgMax m = wave_argmax(v, idx);
  if (lane == 0) {
    a.rowmax_v[(size_t)b * N + r] = m.v;
    a.rowmax_i[(size_t)b * N + r] = m.i;
  }
}

__global__ __launch_bounds__(256) void k_reg_s0(const RegArgs a, int N) {
  __shared__ double rv[16];
  __shared__ long long ri[16];
  const int b = blockIdx.x;
  double v = -1.0;
  long long idx = (long long)N * N;
  for (int r = threadIdx.x; r < N; r += blockDim.x) {
    const double m = a.rowmax_v[(size_t)b * N + r];
    const long long ii = a.rowmax_i[(size_t)b * N + r];
    if (better(m, ii, v, idx)) { v = m; idx = ii; }
  }
  const ArgMax m = block_argmax(v, idx, rv, ri);
  if (threadIdx.x == 0) {
    const int py = (int)(m.i / N), px = (int)(m.i % N);
    a.s0[2 * b] = py > N / 2 ? py - N : py;
    a.s0[2 * b + 1] = px > N / 2 ? px - N : px;
    a.peak[4 * b] = py;
    a.peak[4 * b + 1] = px;
  }
}

// K[u][k] = exp(+2 pi i k_signed (u - c) / (N up)), u < U
__global__ void k_reg_kmat(const RegArgs a, int N) {
  const int U = a.U;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < U * N; i += gridDim.x * blockDim.x) {
    const int u = i / N, k = i - u * N;
    const double ph = 2.0 * (double)signed_freq(k, N) * (double)(u - a.c) / ((double)N * (double)a.up);
    double s, c;
    sincospi(ph, &s, &c);
    a.K[i] = make_double2(c, s);
  }
}

// The two GEMMs as plain vector code, for windows too small for the folded
// ones below.  Register blocks of 2 x 4 and 2 x 2.
// T[b][u][kx] = sum_ky K[u][ky] X[b][ky][kx] e^{2 pi i (ky s0y + kx s0x)/N}
// Tile: 32 u x 64 kx per workgroup, ky in chunks of 16 staged in LDS;
// each of the 16 x 16 threads accumulates a 2 x 4 block.
constexpr int G1_RI = 2, G1_RJ = 4, G1_TX = 16 * G1_RJ, G1_KC = 16;
template <int N>
__global__ __launch_bounds__(256) void k_reg_gemm1(const RegArgs a) {
  constexpr int G1_TU = 16 * G1_RI;
  __shared__ double2 Ks[G1_TU][G1_KC + 1];
  __shared__ double2 Xs[G1_KC][G1_TX + 1];
  __shared__ double2 tw[N];  // exp(-2 pi i e / N): the lag phase is an N-th root of unity
  const int b = blockIdx.z;
  const int u0 = blockIdx.y * G1_TU, x0 = blockIdx.x * G1_TX;
  const int U = a.U;
  const double2* X = a.work + ((size_t)b * 2 + 1) * N * N;
  const int s0y = a.s0[2 * b], s0x = a.s0[2 * b + 1];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;  // 16 x 16 threads
  double2 acc[G1_RI][G1_RJ];
#pragma unroll
  for (int i = 0; i < G1_RI; ++i)
#pragma unroll
    for (int j = 0; j < G1_RJ; ++j) acc[i][j] = make_double2(0.0, 0.0);
  load_twiddles<N>(tw);
  __syncthreads();
  for (int k0 = 0; k0 < N; k0 += G1_KC) {
    for (int i = threadIdx.x; i < G1_TU * G1_KC; i += blockDim.x) {
      const int uu = i / G1_KC, kk = i - uu * G1_KC;
      const int u = u0 + uu;
      Ks[uu][kk] = u < U ? a.K[(size_t)u * N + k0 + kk] : make_double2(0.0, 0.0);
    }
    for (int i = threadIdx.x; i < G1_KC * G1_TX; i += blockDim.x) {
      const int kk = i / G1_TX, xx = i - kk * G1_TX;
      const int ky = k0 + kk, kx = x0 + xx;
      if (kx >= N) { Xs[kk][xx] = make_double2(0.0, 0.0); continue; }
      const double2 x = X[(size_t)ky * N + kx];
      // e^{2 pi i e / N} with e = (ky s0y + kx s0x) mod N = conj(tw[e])
      int e = (signed_freq(ky, N) * s0y + signed_freq(kx, N) * s0x) % N;
      e += e < 0 ? N : 0;
      Xs[kk][xx] = cmulc(x, tw[e]);
    }
    __syncthreads();
#pragma unroll 4
    for (int kk = 0; kk < G1_KC; ++kk) {
      double2 kv[G1_RI], xv[G1_RJ];
#pragma unroll
      for (int i = 0; i < G1_RI; ++i) kv[i] = Ks[ty + 16 * i][kk];
#pragma unroll
      for (int j = 0; j < G1_RJ; ++j) xv[j] = Xs[kk][tx + 16 * j];
#pragma unroll
      for (int i = 0; i < G1_RI; ++i)
#pragma unroll
        for (int j = 0; j < G1_RJ; ++j) {
          acc[i][j].x = fma(kv[i].x, xv[j].x, fma(-kv[i].y, xv[j].y, acc[i][j].x));
          acc[i][j].y = fma(kv[i].x, xv[j].y, fma(kv[i].y, xv[j].x, acc[i][j].y));
        }
    }
    __syncthreads();
  }
  double2* T = a.T + (size_t)b * U * N;
#pragma unroll
  for (int i = 0; i < G1_RI; ++i) {
    const int u = u0 + ty + 16 * i;
    if (u >= U) continue;
#pragma unroll
    for (int j = 0; j < G1_RJ; ++j)
      if (x0 + tx + 16 * j < N) T[(size_t)u * N + x0 + tx + 16 * j] = acc[i][j];
  }
}

// C[b][u][v] = sum_kx T[b][u][kx] K[v][kx]; per-tile first maximum of |C|^2.
// Tile 32 u x 32 v, kx in chunks of 16; each thread a 2 x 2 block.
constexpr int G2_KC = 16, G2_R = 2;
template <int N>
__global__ __launch_bounds__(256) void k_reg_gemm2(const RegArgs a) {
  constexpr int G2_T = 16 * G2_R;
  __shared__ double2 Ts[G2_T][G2_KC + 1];
  __shared__ double2 Ks[G2_T][G2_KC + 1];
  __shared__ double rv[16];
  __shared__ long long ri[16];
  const int b = blockIdx.z;
  const int u0 = blockIdx.y * G2_T, v0 = blockIdx.x * G2_T;
  const int U = a.U;
  const double2* T = a.T + (size_t)b * U * N;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  double2 acc[G2_R][G2_R];
#pragma unroll
  for (int i = 0; i < G2_R; ++i)
#pragma unroll
    for (int j = 0; j < G2_R; ++j) acc[i][j] = make_double2(0.0, 0.0);
  for (int k0 = 0; k0 < N; k0 += G2_KC) {
    for (int i = threadIdx.x; i < G2_T * G2_KC; i += blockDim.x) {
      const int rr = i / G2_KC, kk = i - rr * G2_KC;
      const int u = u0 + rr, v = v0 + rr;
      Ts[rr][kk] = u < U ? T[(size_t)u * N + k0 + kk] : make_double2(0.0, 0.0);
      Ks[rr][kk] = v < U ? a.K[(size_t)v * N + k0 + kk] : make_double2(0.0, 0.0);
    }
    __syncthreads();
#pragma unroll 4
    for (int kk = 0; kk < G2_KC; ++kk) {
      double2 tv[G2_R], kv[G2_R];
#pragma unroll
      for (int i = 0; i < G2_R; ++i) tv[i] = Ts[ty + 16 * i][kk];
#pragma unroll
      for (int j = 0; j < G2_R; ++j) kv[j] = Ks[tx + 16 * j][kk];
#pragma unroll
      for (int i = 0; i < G2_R; ++i)
#pragma unroll
        for (int j = 0; j < G2_R; ++j) {
          acc[i][j].x = fma(tv[i].x, kv[j].x, fma(-tv[i].y, kv[j].y, acc[i][j].x));
          acc[i][j].y = fma(tv[i].x, kv[j].y, fma(tv[i].y, kv[j].x, acc[i][j].y));
        }
    }
    __syncthreads();
  }
  double best = -1.0;
  long long bi = (long long)U * U;
#pragma unroll
  for (int i = 0; i < G2_R; ++i)
#pragma unroll
    for (int j = 0; j < G2_R; ++j) {
      const int u = u0 + ty + 16 * i, v = v0 + tx + 16 * j;
      if (u < U && v < U) {
        const double m = cabs2(acc[i][j]);
        const long long ii = (long long)u * U + v;
        if (better(m, ii, best, bi)) { best = m; bi = ii; }
      }
    }
  const ArgMax m = block_argmax(best, bi, rv, ri);
  if (threadIdx.x == 0) {
    const int tiles = gridDim.x * gridDim.y;
    const int t = blockIdx.y * gridDim.x + blockIdx.x;
    a.tile_v[(size_t)b * tiles + t] = m.v;
    a.tile_i[(size_t)b * tiles + t] = m.i;
  }
}

// ------------------------------------------------- the GEMMs by symmetry
// With w = u - c the window is symmetric, and K[c + w][k] = e^{i th k w}, th =
// 2 pi / (N up).  Over the pairs of frequencies +-k a sum against K is
//   sum_k e^{i th k w} x_k = E + i O,   E = sum_{k = 0..N/2} cos(th k w) p_k,
//                                       O = sum_{k = 1..N/2} sin(th k w) m_k,
// p_k = x_k + x_-k, m_k = x_k - x_-k (p_0 = x_0; the one term of frequency
// -N/2 is p = x, m = -x), and the sample at -w is E - i O.  cos and sin are
// real and one product serves two samples, so a dimension costs a quarter of
// the multiplications of the complex product.  X is folded in both
// dimensions at once (k_reg_fold), which leaves two products of the same form:
//   k_reg_fold1  rows: the folds of X (kx = p of 0..N/2, then m of 1..N/2),
//                summed over ky; columns: w of u
//   k_reg_fold2  rows: u; summed over kx; columns: w of v; first maximum
// Both run on the fp64 matrix cores (16 x 16 x 4).  Everything is kept in the
// order in which the lanes of an operand take it, so that all operand loads
// are consecutive and need no LDS:
//   rows   of 16: [step][lane] (re, im) of row lane % 16, slot 4 step + lane / 16,
//          first the SE steps of the even slots (k = 0..N/2, then zeros), then
//          the SO steps of the odd ones (k = 1..N/2)
//   table  of 16 w: [step][lane] cos or sin, likewise
// A result tile holds, in register r, row 4 r + lane / 16 and column lane %
// 16: as a row operand of the second product (its rows are the first one's
// columns) register r of tile t is step 4 t + r, lane by lane.
//
// A wave takes 2 row tiles x JT column tiles, 16 instructions of 64 cycles a
// step for 8 operand loads, so the matrix cores bound it.  (2 x 4 tiles need
// more than 256 registers, and the compiler then moves accumulators between
// the two register files at every instruction.)  Operands are fetched two
// steps ahead: one step, 1000 cycles, does not cover memory (fold1 of 200
// pairs at upsample 100 174 against 141 us).  32 pairs of 256^2 at upsample
// 1000 (window 1500): fold + fold1 + fold2 20 + 160 + 705 us (54 TFLOP/s of
// fp64 in fold2) where the complex products took 616 + 3530; 400 pairs at
// upsample 100 (window 150): 151 + 282 + 167 us, before 950 + 607.
using d2 = double __attribute__((ext_vector_type(2)));
using d4 = double __attribute__((ext_vector_type(4)));

constexpr int JT = 2;

template <int N>
struct Fold {
  static constexpr int SE = N / 8 + 1, SO = N / 8;         // steps of 4 slots
  static constexpr int PT = N / 32 + 1, RT = PT + N / 32;  // row tiles of p, of p and m
  static constexpr int TILE = (SE + SO) * 64;              // of lane operands
  static constexpr int HOME = N * N / TILE;                // row tiles that fit a pair's work[0]
};

// Row tile t of the folded X of pair b: in work[0], the last ones behind.
template <int N>
__device__ __forceinline__ d2* fold_tile(const RegArgs& a, int b, int t) {
  using F = Fold<N>;
  return t < F::HOME ? (d2*)(a.work + (size_t)b * 2 * N * N) + (size_t)t * F::TILE
                     : (d2*)a.F + ((size_t)b * (F::RT - F::HOME) + (t - F::HOME)) * F::TILE;
}

// The table of all column tiles, w < 16 tiles.
template <int N>
__global__ __launch_bounds__(256) void k_reg_table(const RegArgs a, int tiles) {
  using F = Fold<N>;
  double* const tab = (double*)a.K;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < tiles * F::TILE; i += gridDim.x * 256) {
    const int lane = i & 63, step = i / 64 % (F::SE + F::SO), w = i / F::TILE * 16 + (lane & 15);
    const bool odd = step >= F::SE;
    const int k = odd ? 4 * (step - F::SE) + (lane >> 4) + 1 : 4 * step + (lane >> 4);
    double s, c;
    sincospi(2.0 * (double)k * (double)w / ((double)N * (double)a.up), &s, &c);
    tab[i] = k > N / 2 ? 0.0 : odd ? s : c;
  }
}

template <int N>
__global__ __launch_bounds__(256) void k_reg_fold(const RegArgs a) {
  using F = Fold<N>;
  constexpr int HN = N / 2, LW = 16 * F::PT;
  __shared__ double2 tw[N];  // exp(-2 pi i e / N)
  load_twiddles<N>(tw);
  __syncthreads();
  const int b = blockIdx.y, i = blockIdx.x * 256 + threadIdx.x;
  const int k = i / LW, l = i - k * LW;
  if (k >= 4 * F::SE) return;
  const double2* const X = a.work + ((size_t)b * 2 + 1) * N * N;
  const int s0y = a.s0[2 * b], s0x = a.s0[2 * b + 1];
  // x[ky][kx] e^{2 pi i (ky s0y + kx s0x) / N} at (+-k, +-l)
  const double2 z = make_double2(0.0, 0.0);
  double2 pp = z, np = z, pn = z, nn = z;
  if (k <= HN && l <= HN) {
    int e = (k * s0y + l * s0x) % N, g = (l * s0x - k * s0y) % N;
    e += e < 0 ? N : 0;
    g += g < 0 ? N : 0;
    const bool ky = k > 0 && k < HN, lx = l > 0 && l < HN;
    pp = cmulc(X[k * N + l], tw[e]);
    if (ky) np = cmulc(X[(N - k) * N + l], tw[g]);
    if (lx) pn = cmul(X[k * N + N - l], tw[g]);
    if (ky && lx) nn = cmul(X[(N - k) * N + N - l], tw[e]);
  }
  const double sk = k == HN ? -1.0 : 1.0, sl = l == HN ? -1.0 : 1.0;
  const auto put = [&](int row, int step, int slot, double x, double y) __attribute__((always_inline)) {
    fold_tile<N>(a, b, row >> 4)[step * 64 + (slot & 3) * 16 + (row & 15)] = d2{x, y};
  };
  const auto rows = [&](int step, int slot, double2 p, double2 n) __attribute__((always_inline)) {
    put(l, step, slot, p.x + n.x, p.y + n.y);
    if (l >= 1 && l <= HN) put(LW + l - 1, step, slot, sl * p.x - n.x, sl * p.y - n.y);
  };
  rows(k >> 2, k, make_double2(pp.x + np.x, pp.y + np.y), make_double2(pn.x + nn.x, pn.y + nn.y));
  if (k >= 1 && k <= HN)
    rows(F::SE + ((k - 1) >> 2), k - 1, make_double2(sk * pp.x - np.x, sk * pp.y - np.y),
         make_double2(sk * pn.x - nn.x, sk * pn.y - nn.y));
}

// acc[i][j]: re and im of E, re and im of O of row tile i and column tile j.
template <int N>
__device__ __forceinline__ void fold_product(const d2* const (&A)[2], const double* const (&B)[JT],
                                             d4 (&acc)[2][JT][4]) {
  using F = Fold<N>;
  d2 e[3][2], o[3][2];          // steps s, s + 1, s + 2
  double c[3][JT], n[3][JT];
  const auto load = [&](int x, int s) __attribute__((always_inline)) {
    const int se = min(s, F::SE - 1), so = min(s, F::SO - 1);  // (there is one even step more)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      e[x][i] = A[i][se * 64];
      o[x][i] = A[i][(F::SE + so) * 64];
    }
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      c[x][j] = B[j][se * 64];
      n[x][j] = B[j][(F::SE + so) * 64];
    }
  };
  load(0, 0);
  load(1, 1);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < JT; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[i][j][q] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 3
  for (int s = 0; s < F::SO; ++s) {
    load(2, s + 2);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        acc[i][j][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[0][i][0], c[0][j], acc[i][j][0], 0, 0, 0);
        acc[i][j][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[0][i][1], c[0][j], acc[i][j][1], 0, 0, 0);
        acc[i][j][2] = __builtin_amdgcn_mfma_f64_16x16x4f64(o[0][i][0], n[0][j], acc[i][j][2], 0, 0, 0);
        acc[i][j][3] = __builtin_amdgcn_mfma_f64_16x16x4f64(o[0][i][1], n[0][j], acc[i][j][3], 0, 0, 0);
      }
#pragma unroll
    for (int x = 0; x < 2; ++x) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        e[x][i] = e[x + 1][i];
        o[x][i] = o[x + 1][i];
      }
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        c[x][j] = c[x + 1][j];
        n[x][j] = n[x + 1][j];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      acc[i][j][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[0][i][0], c[0][j], acc[i][j][0], 0, 0, 0);
      acc[i][j][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(e[0][i][1], c[0][j], acc[i][j][1], 0, 0, 0);
    }
}

// Waves of a launch: pair, row group, column group, the last running fastest
// (the waves of a workgroup share their rows).
struct FoldWork {
  int rows, cols, tiles;  // row groups of 2, column groups of JT; column tiles
  int waves;              // of all pairs
};

template <int N>
__device__ __forceinline__ int fold_columns(const RegArgs& a, const FoldWork& w, int cg, int lane,
                                            const double* (&B)[JT]) {
#pragma unroll
  for (int j = 0; j < JT; ++j)
    B[j] = (const double*)a.K + (size_t)min(cg * JT + j, w.tiles - 1) * Fold<N>::TILE + lane;
  return min(JT, w.tiles - cg * JT);
}

template <int N>
__global__ __launch_bounds__(256, 2) void k_reg_fold1(const RegArgs a, const FoldWork w) {
  using F = Fold<N>;
  const int q = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
  if (q >= w.waves) return;
  const int b = q / (w.rows * w.cols), rg = q / w.cols % w.rows, cg = q % w.cols;
  const d2* A[2];
  const double* B[JT];
#pragma unroll
  for (int i = 0; i < 2; ++i) A[i] = fold_tile<N>(a, b, min(2 * rg + i, F::RT - 1)) + lane;
  const int cols = fold_columns<N>(a, w, cg, lane, B);
  d4 acc[2][JT][4];
  fold_product<N>(A, B, acc);
  d2* const T = (d2*)a.T + (size_t)b * 2 * w.tiles * F::TILE + lane;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int t = 2 * rg + i;
    if (t >= F::RT) continue;
#pragma unroll
    for (int j = 0; j < JT; ++j) {
      if (j >= cols) continue;
      d2* const up = T + (size_t)(cg * JT + j) * F::TILE;
      d2* const down = up + (size_t)w.tiles * F::TILE;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int step = 4 * t + r;  // of p; m starts at tile PT
        if (t < F::PT && step >= F::SE) continue;
        const int at = (t < F::PT ? step : F::SE + step - 4 * F::PT) * 64;
        up[at] = d2{acc[i][j][0][r] - acc[i][j][3][r], acc[i][j][1][r] + acc[i][j][2][r]};
        down[at] = d2{acc[i][j][0][r] + acc[i][j][3][r], acc[i][j][1][r] - acc[i][j][2][r]};
      }
    }
  }
}

template <int N>
__global__ __launch_bounds__(256, 2) void k_reg_fold2(const RegArgs a, const FoldWork w) {
  using F = Fold<N>;
  const int q = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
  if (q >= w.waves) return;
  const int per = w.rows * w.cols, b = q / per, rg = q / w.cols % w.rows, cg = q % w.cols;
  const d2* A[2];
  const double* B[JT];
#pragma unroll
  for (int i = 0; i < 2; ++i) A[i] = (const d2*)a.T + ((size_t)b * 2 * w.tiles + 2 * rg + i) * F::TILE + lane;
  const int cols = fold_columns<N>(a, w, cg, lane, B);
  d4 acc[2][JT][4];
  fold_product<N>(A, B, acc);
  const int U = a.U, c = a.c;
  double best = -1.0;
  int bi = U * U;
  const auto take = [&](bool in, int u, int v, double re, double im) __attribute__((always_inline)) {
    const double m = re * re + im * im;
    const int ii = u * U + v;
    const bool win = in && (m > best || (m == best && ii < bi));
    best = win ? m : best;
    bi = win ? ii : bi;
  };
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int t = 2 * rg + i;
    const bool down = t >= w.tiles;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int wu = (down ? t - w.tiles : t) * 16 + 4 * r + (lane >> 4), u = down ? c - wu : c + wu;
      const bool uin = wu <= c && u < U && !(down && wu == 0);
#pragma unroll
      for (int j = 0; j < JT; ++j) {
        const int wv = (cg * JT + j) * 16 + (lane & 15);
        const bool in = uin && j < cols && wv <= c;
        const double er = acc[i][j][0][r], ei = acc[i][j][1][r], orr = acc[i][j][2][r], oi = acc[i][j][3][r];
        take(in && c + wv < U, u, c + wv, er - oi, ei + orr);
        take(in && wv > 0, u, c - wv, er + oi, ei - orr);
      }
    }
  }
  const ArgMax m = wave_argmax(best, (long long)bi);
  if (lane == 0) {
    a.tile_v[(size_t)b * per + rg * w.cols + cg] = m.v;
    a.tile_i[(size_t)b * per + rg * w.cols + cg] = m.i;
  }
}

__global__ __launch_bounds__(64) void k_reg_final(const RegArgs a, int tiles) {
  const int b = blockIdx.x;
  double v = -1.0;
  long long idx = (long long)a.U * a.U;
  for (int t = threadIdx.x; t < tiles; t += 64) {
    const double m = a.tile_v[(size_t)b * tiles + t];
    const long long ii = a.tile_i[(size_t)b * tiles + t];
    if (better(m, ii, v, idx)) { v = m; idx = ii; }
  }
  idx = wave_argmax(v, idx).i;
  if (threadIdx.x) return;
  const int u = (int)(idx / a.U), w = (int)(idx % a.U);
  a.peak[4 * b + 2] = u;
  a.peak[4 * b + 3] = w;
  const double up = (double)a.up;
  a.shift[2 * b] = (float)((double)a.s0[2 * b] + (double)(u - a.c) / up);
  a.shift[2 * b + 1] = (float)((double)a.s0[2 * b + 1] + (double)(w - a.c) / up);
}

// ---------------------------------------------------------------- Adam
// Alg. 1 with the measured shift as the gradient; the position moves by
// +lr mhat / (sqrt(vhat) + eps) (Eq. 8-9) and is clamped to the object.
__global__ void k_adam(int J, float* pos, float* st, const float* g, int t, float lr, float b1, float b2,
                       float eps, float ymax, float xmax, const int* active) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= J) return;
  if (active && !active[0]) return;
  const double bc1 = 1.0 - pow((double)b1, (double)t);
  const double bc2 = 1.0 - pow((double)b2, (double)t);
  for (int a = 0; a < 2; ++a) {
    const double gj = (double)g[2 * j + a];
    const double m = (double)b1 * (double)st[4 * j + a] + (1.0 - (double)b1) * gj;
    const double v = (double)b2 * (double)st[4 * j + 2 + a] + (1.0 - (double)b2) * gj * gj;
    st[4 * j + a] = (float)m;
    st[4 * j + 2 + a] = (float)v;
    double p = (double)pos[2 * j + a] + (double)lr * (m / bc1) / (sqrt(v / bc2) + (double)eps);
    const double lim = a == 0 ? (double)ymax : (double)xmax;
    p = p < 0.0 ? 0.0 : (p > lim ? lim : p);
    pos[2 * j + a] = (float)p;
  }
}

// ---------------------------------------------------------------- host
int reg_window(int up, int* U, int* c) {
  *U = (int)std::ceil(1.5 * (double)up);
  *c = *U / 2;
  return MRPIE_OK;
}

// The folded products need windows that fill their tiles of 16 + 16 samples.
// In the plain products' workspace they may take fewer pairs a pass, and a pass
// more is some 10 launches: calls of fewer than so many U N (N + U) of all pairs
// then keep the plain products (3.5e8, 1e8 for windows above 320 samples, whose
// plain products are the slower ones).  Measured, us plain / folded in more
// passes: 64^2 3 pairs at upsample 100 77 / 117, 67 pairs at 37 87 / 134, 128^2
// 30 at 100 136 / 158, 256^2 10 at 100 181 / 208, 3.2e8: 256^2 30 at 75 231 /
// 248; 4.3e8: 256^2 67 at 50 341 / 334, 1.0e9: 67 at 100 440 / 338; windows above
// 320: 32^2 10 pairs at 214 81 / 98, 64^2 10 at 214 109 / 121, 30 at 214 (2.4e8)
// 145 / 129.  In as many passes the folded ones win: 64^2 3 at 333 101 / 76,
// 128^2 1 at 75 99 / 79, 256^2 1 at 100 160 / 100.
constexpr int kFoldMinU = 32, kWideU = 320;
constexpr double kFoldMinWork = 3.5e8, kFoldMinWorkWide = 1e8;

RegLayout reg_layout(int N, int B, int up) {
  RegLayout L{};
  int U, c;
  reg_window(up, &U, &c);
  const int chunk = std::max(1, std::min(B, kRegChunk));
  const int t2 = U > kWideU ? 64 : 32;
  int tiles = ((U + t2 - 1) / t2) * ((U + t2 - 1) / t2);
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = ws_align(off + bytes); return o; };
  const auto place = [&](int n, size_t table, size_t t, size_t f) {
    off = 0;
    L.chunk = n;
    L.work = take((size_t)n * 2 * N * N * 16);
    L.K = take(table);
    L.T = take((size_t)n * t);
    L.rowmax_v = take((size_t)n * N * 8);
    L.rowmax_i = take((size_t)n * N * 8);
    L.s0 = take((size_t)n * 2 * 4);
    L.tile_v = take((size_t)n * tiles * 8);
    L.tile_i = take((size_t)n * tiles * 8);
    L.F = take((size_t)n * f);
  };
  const size_t plain = (size_t)U * N * 16;
  const auto plain_products = [&] {
    place(chunk, plain, plain, 0);
    // (The workspace counts the maxima of windows above 320 by 64 x 64 tiles,
    // the kernels take 32 x 32: theirs lie over the spectra, which the second
    // product does not read.)
    if (U > kWideU) {
      const size_t n = (size_t)((U + 31) / 32) * ((U + 31) / 32) * chunk;
      L.tile_v = L.work;
      L.tile_i = L.work + ws_align(n * 8);
    }
  };
  plain_products();
  L.total = off;
  if (U < kFoldMinU) return L;
  // The folded products lay out less for the table and more for each pair.
  // They take no more memory than the plain ones: fewer pairs a pass if need
  // be, down to half.
  const int ct = c / 16 + 1, plain_tiles = tiles;
  const size_t lanes = (size_t)(N / 4 + 1) * 64;            // Fold<N>::TILE
  const size_t behind = (N / 16 + 1) - N * N / lanes;       // Fold<N>::RT - HOME
  tiles = ct * ((ct + JT - 1) / JT);
  L.fold = true;
  int n = chunk;
  do place(n, ct * lanes * 8, 2 * ct * lanes * 16, behind * lanes * 16);
  while (off > L.total && --n);
  const int passes = n ? (B + n - 1) / n : 0;  // of like size
  if (2 * n < chunk || n == 0 ||
      (passes > (B + chunk - 1) / chunk &&
       (double)B * U * N * (N + U) < (U > kWideU ? kFoldMinWorkWide : kFoldMinWork))) {
    tiles = plain_tiles;
    L.fold = false;
    plain_products();
    return L;
  }
  place(std::max(1, (B + passes - 1) / passes), ct * lanes * 8, 2 * ct * lanes * 16, behind * lanes * 16);
  return L;
}

template <int N>
static int register_impl(int B, const float2* ref, const float2* mov, int up, int norm, float* shift, int32_t* peak,
                         char* ws, const RegLayout& L, hipStream_t s) {
  int U, c;
  reg_window(up, &U, &c);
  RegArgs a{};
  a.U = U;
  a.c = c;
  a.up = up;
  a.norm = norm;
  a.work = (double2*)(ws + L.work);
  a.K = (double2*)(ws + L.K);
  a.F = (double2*)(ws + L.F);
  a.T = (double2*)(ws + L.T);
  a.rowmax_v = (double*)(ws + L.rowmax_v);
  a.rowmax_i = (long long*)(ws + L.rowmax_i);
  a.s0 = (int*)(ws + L.s0);
  a.tile_v = (double*)(ws + L.tile_v);
  a.tile_i = (long long*)(ws + L.tile_i);
  MRPIE_HIP(ensure_lds((const void*)k_reg_cols<N>, reg_cols_lds(N)));
  const int gt = (U + 31) / 32, ct = c / 16 + 1;
  if (L.fold) hipLaunchKernelGGL(k_reg_table<N>, dim3((ct * Fold<N>::TILE + 255) / 256), dim3(256), 0, s, a, ct);
  else hipLaunchKernelGGL(k_reg_kmat, dim3(64), dim3(256), 0, s, a, N);
  for (int b0 = 0; b0 < B; b0 += L.chunk) {
    const int nb = std::min(L.chunk, B - b0);
    a.B = nb;
    a.ref = ref + (size_t)b0 * N * N;
    a.mov = mov + (size_t)b0 * N * N;
    a.shift = shift + 2 * (size_t)b0;
    a.peak = peak + 4 * (size_t)b0;
    hipLaunchKernelGGL(k_reg_rows<N>, dim3(N / kRegRW, nb, 2), dim3(256), 0, s, a);
    launch_k(TK_REG, k_reg_cols<N>, dim3(N / kRegCW, nb), dim3(256), reg_cols_lds(N), s, a);
    hipLaunchKernelGGL(k_reg_coarse<N>, dim3(N / kRegRW, nb), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_reg_s0, dim3(nb), dim3(256), 0, s, a, N);
    int tiles = gt * gt;
    if (L.fold) {
      constexpr int kSlots = 4 * Fold<N>::SE * 16 * Fold<N>::PT;
      hipLaunchKernelGGL(k_reg_fold<N>, dim3((kSlots + 255) / 256, nb), dim3(256), 0, s, a);
      FoldWork w{(Fold<N>::RT + 1) / 2, (ct + JT - 1) / JT, ct, 0};
      w.waves = nb * w.rows * w.cols;
      launch_ku(TK_GEMM, nb, k_reg_fold1<N>, dim3((w.waves + 3) / 4), dim3(256), 0, s, a, w);
      w.rows = ct;
      tiles = w.rows * w.cols;
      w.waves = nb * tiles;
      hipLaunchKernelGGL(k_reg_fold2<N>, dim3((w.waves + 3) / 4), dim3(256), 0, s, a, w);
    } else {
      launch_ku(TK_GEMM, nb, k_reg_gemm1<N>, dim3((N + G1_TX - 1) / G1_TX, gt, nb), dim3(256), 0, s, a);
      hipLaunchKernelGGL(k_reg_gemm2<N>, dim3(gt, gt, nb), dim3(256), 0, s, a);
    }
    hipLaunchKernelGGL(k_reg_final, dim3(nb), dim3(64), 0, s, a, tiles);
  }
  MRPIE_HIP(hipGetLastError());
  return MRPIE_OK;
}

int run_register(int N, int B, const float2* ref, const float2* mov, int up, int norm, float* shift, int32_t* peak,
                 void* ws, size_t ws_bytes, hipStream_t s) {
  const RegLayout L = reg_layout(N, B, up);
  if (!ws || ws_bytes < L.total) return fail(MRPIE_EWORKSPACE, "workspace %zu < %zu bytes", ws_bytes, L.total);
  int rc = launch_init_twiddles(s);
  if (rc) return rc;
  char* w = (char*)ws;
  switch (N) {
    case 32: return register_impl<32>(B, ref, mov, up, norm, shift, peak, w, L, s);
    case 64: return register_impl<64>(B, ref, mov, up, norm, shift, peak, w, L, s);
    case 128: return register_impl<128>(B, ref, mov, up, norm, shift, peak, w, L, s);
    case 192: return register_impl<192>(B, ref, mov, up, norm, shift, peak, w, L, s);
    default: return register_impl<256>(B, ref, mov, up, norm, shift, peak, w, L, s);
  }
}

int launch_adam(int J, float* pos, float* adam, const float* g, int t, const mrpie_params* pr, int ymax, int xmax,
                hipStream_t s) {
  hipLaunchKernelGGL(k_adam, dim3((J + 255) / 256), dim3(256), 0, s, J, pos, adam, g, t, pr->adam_lr, pr->adam_b1,
                     pr->adam_b2, pr->adam_eps, (float)ymax, (float)xmax, (const int*)nullptr);
  MRPIE_HIP(hipGetLastError());
  return MRPIE_OK;
}

}  // namespace mrpie

using namespace mrpie;

extern "C" {

int mrpie_register_workspace_size(int32_t N, int32_t B, int32_t upsample, size_t* bytes) {
  if (n_index(N) < 0) return fail(MRPIE_EUNSUPPORTED, "N=%d not in {32,64,128,192,256}", N);
  if (B < 0 || upsample < 1 || upsample > 1000 || !bytes) return fail(MRPIE_EINVAL, "bad arguments");
  *bytes = reg_layout(N, std::max(B, 1), upsample).total;
  return MRPIE_OK;
}

int mrpie_register(int32_t N, int32_t B, const void* ref, const void* mov, int32_t upsample, int32_t norm,
                   float* shift, int32_t* peak, void* ws, size_t ws_bytes, void* stream) {
  if (n_index(N) < 0) return fail(MRPIE_EUNSUPPORTED, "N=%d not in {32,64,128,192,256}", N);
  if (B < 0) return fail(MRPIE_EINVAL, "B=%d < 0", B);
  if (upsample < 1 || upsample > 1000) return fail(MRPIE_EINVAL, "upsample=%d not in [1,1000]", upsample);
  if (norm != 0 && norm != 1) return fail(MRPIE_EINVAL, "norm must be 0 or 1");
  if (B == 0) return MRPIE_OK;
  if (!ref || !mov || !shift || !peak) return fail(MRPIE_EINVAL, "null pointer");
  return run_register(N, B, (const float2*)ref, (const float2*)mov, upsample, norm, shift, peak, ws, ws_bytes,
                      (hipStream_t)stream);
}

int mrpie_adam(int32_t J, const mrpie_params* pr, int32_t ymax, int32_t xmax, float* pos, float* adam,
               const float* g, int32_t t, void* stream) {
  if (!pr || J < 0 || t < 1 || ymax < 0 || xmax < 0) return fail(MRPIE_EINVAL, "bad arguments");
  if (!(pr->adam_b1 >= 0.f && pr->adam_b1 < 1.f) || !(pr->adam_b2 >= 0.f && pr->adam_b2 < 1.f))
    return fail(MRPIE_EINVAL, "Adam betas must be in [0,1)");
  if (!(pr->adam_eps > 0.f) || !std::isfinite(pr->adam_lr)) return fail(MRPIE_EINVAL, "bad Adam lr/eps");
  if (J == 0) return MRPIE_OK;
  if (!pos || !adam || !g) return fail(MRPIE_EINVAL, "null pointer");
  return launch_adam(J, pos, adam, g, t, pr, ymax, xmax, (hipStream_t)stream);
}

}  // extern "C"

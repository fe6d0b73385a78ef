// 1-D complex FFTs inside one 64-wide wavefront (gfx950).
//
// A transform of length N is held by L lanes, PT = N / L points each, in the
// strided layout v[i] = x[l + L i]; G = 64 / L transforms share a wave, lane
// G l + g holding place l of transform g, so that lanes next to each other
// hold the same few elements of adjacent rows (or columns).  Input and output have the same layout, so an
// inverse transform takes a forward transform's registers, and consecutive
// lanes hold consecutive elements.  The Stockham stages exchange points
// through an LDS scratch private to the wave: its LDS operations complete in
// program order, so no workgroup barrier is needed and waves drift freely
// (the workgroup-wide stages of fft.hpp pay two waits of the slowest wave per
// stage).  Stage twiddles do not depend on the transform and stay in
// registers (N = 192 has 36 values of them, and reads them from the LDS).
//
//   N    L   PT  stages
//   256  32   8  8 x 8 x 4
//   192  16  12  12 x 4 x 4
//   128  16   8  8 x 4 x 4
//   64    8   8  8 x 8
//   32    4   8  8 x 4
#pragma once
#include "fft.hpp"

namespace mrpie {

// ordering of LDS accesses of one wave for the compiler (no instruction)
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 12 points as 3 x 4, natural order in and out.  Its fused operations and
// those of the 192-point twiddles are spelled out: chosen by the compiler they
// differ between one transform and two side by side, and the sweep's results
// must not depend on which of the two a wave runs.
#pragma clang fp contract(off)
template <bool INV>
__device__ __forceinline__ float2 cmulw(float2 a, float c, float s) {  // a * (c -+ i s)
  return INV ? mk(fmaf(a.x, c, -(a.y * s)), fmaf(a.y, c, a.x * s)) : mk(fmaf(a.x, c, a.y * s), fmaf(a.y, c, -(a.x * s)));
}
template <bool INV>
__device__ __forceinline__ void dft12(float2* v) {
  constexpr float c1 = 0.86602540378443864676f, h = 0.5f;
  float2 t[3][4];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const float2 t1 = cadd(v[a + 4], v[a + 8]), t2 = csub(v[a + 4], v[a + 8]);
    const float2 m = mk(fmaf(-h, t1.x, v[a].x), fmaf(-h, t1.y, v[a].y));
    constexpr float s = INV ? c1 : -c1;
    t[0][a] = cadd(v[a], t1);
    t[1][a] = mk(fmaf(-s, t2.y, m.x), fmaf(s, t2.x, m.y));
    t[2][a] = mk(fmaf(s, t2.y, m.x), fmaf(-s, t2.x, m.y));
  }
  t[1][1] = cmulw<INV>(t[1][1], c1, h);
  t[1][2] = cmulw<INV>(t[1][2], h, c1);
  t[1][3] = rot90<INV>(t[1][3]);
  t[2][1] = cmulw<INV>(t[2][1], h, c1);
  t[2][2] = cmulw<INV>(t[2][2], -h, c1);
  t[2][3] = mk(-t[2][3].x, -t[2][3].y);
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    dft4<INV>(t[b]);
#pragma unroll
    for (int c = 0; c < 4; ++c) v[b + 3 * c] = t[b][c];
  }
}
#pragma clang fp contract(fast)

// one pad element every eight spreads the stages' strided accesses over the
// LDS banks (first-stage writes of lane l start at 9 l)
__device__ __forceinline__ constexpr int pad8(int i) { return i + (i >> 3); }

template <int N>
struct WaveFft {
  static constexpr int L = N == 256 ? 32 : N == 192 || N == 128 ? 16 : N == 64 ? 8 : 4;
  static constexpr int PT = N / L;
  static constexpr int G = 64 / L;               // transforms a wave holds
  // padded scratch of one transform, with an offset between transforms that
  // keeps the lanes of the G transforms, which alternate in a wave, on
  // distinct banks
  static constexpr int PLEN = N == 256 ? 296 : N == 192 ? 216 : N == 128 ? 168 : N == 64 ? 76 : 38;
  static constexpr int SCRATCH = G * PLEN;       // float2 of scratch per wave
  static constexpr int NT2 = N == 192 ? 1 : N == 128 || N == 32 ? 6 : 7;
  static constexpr int NT3 = N == 256 || N == 128 ? 6 : 0;

  float2 t2[NT2];
  float2 t3[NT3 > 0 ? NT3 : 1];

  static constexpr bool kTable = N == 192;  // the twiddles stay at w
  const float2* tab;

  // w: the N-th roots of unity w_N^e, e < N (in the LDS if kTable)
  __device__ __forceinline__ void init(const float2* w, int l) {
    if constexpr (N == 256) {
#pragma unroll
      for (int r = 1; r < 8; ++r) t2[r - 1] = w[r * (l & 7) * 4];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 1; r < 4; ++r) t3[b * 3 + r - 1] = w[r * (l + 32 * b)];
    } else if constexpr (N == 192) {
      tab = w;
    } else if constexpr (N == 128) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 1; r < 4; ++r) {
          t2[b * 3 + r - 1] = w[r * ((l + 16 * b) & 7) * 4];
          t3[b * 3 + r - 1] = w[r * (l + 16 * b)];
        }
    } else if constexpr (N == 64) {
#pragma unroll
      for (int r = 1; r < 8; ++r) t2[r - 1] = w[r * l];
    } else {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 1; r < 4; ++r) t2[b * 3 + r - 1] = w[r * (l + 4 * b)];
    }
  }

  template <bool INV>
  __device__ __forceinline__ static float2 tmul(float2 a, float2 w) {
    if constexpr (N == 192) return cmulw<INV>(a, w.x, -w.y);  // w = c - i s
    else return INV ? cmulc(a, w) : cmul(a, w);
  }

  // A stage's exchange: outputs to the scratch, inputs of the next from it.
  // Stage boundaries by number: 1 after the first stage, 2 after the second.
  template <int S>
  __device__ __forceinline__ static void put(const float2* v, float2* sc, int l) {
    if constexpr (S == 1) {
      constexpr int R = N == 192 ? 12 : 8;
#pragma unroll
      for (int r = 0; r < R; ++r) sc[R == 8 ? 9 * l + r : pad8(R * l + r)] = v[r];  // pad8(8 l + r)
    } else if constexpr (N == 256) {
#pragma unroll
      for (int r = 0; r < 8; ++r) sc[72 * (l >> 3) + (l & 7) + 9 * r] = v[r];  // pad8(64 (l/8) + l%8 + 8 r)
    } else {  // radix 4 of span 12 (N = 192) or 8 (N = 128), butterflies l + L b
      constexpr int NS = N == 192 ? 12 : 8;
#pragma unroll
      for (int b = 0; b < PT / 4; ++b) {
        const int jb = l + L * b, o = (jb / NS) * NS * 4 + jb % NS;
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[pad8(o + NS * r)] = v[4 * b + r];
      }
    }
  }
  template <int S>
  __device__ __forceinline__ static void get(float2* v, const float2* sc, int l) {
    if constexpr (S == 1 && (N == 256 || N == 64)) {
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = N == 256 ? sc[pad8(l) + 36 * r] : sc[l + 9 * r];  // pad8(l + L r)
    } else {
#pragma unroll
      for (int b = 0; b < PT / 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[4 * b + r] = sc[pad8(l + L * b + (N / 4) * r)];
    }
  }
  // Radix-4 butterflies of a stage with twiddles tw; LAST: outputs into the
  // strided layout.
  template <bool INV, bool LAST>
  __device__ __forceinline__ static void bfly4(float2* v, const float2* tw) {
    constexpr int NB = PT / 4;
    float2 u[NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      u[b][0] = v[4 * b];
#pragma unroll
      for (int r = 1; r < 4; ++r) u[b][r] = tmul<INV>(v[4 * b + r], tw[b * 3 + r - 1]);
      dft4<INV>(u[b]);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) v[LAST ? b + NB * r : 4 * b + r] = u[b][r];
  }
  // N = 192: twiddles of a stage after a span of NS, from the table
  template <int NS>
  __device__ __forceinline__ void fetch(float2* tw, int l) const {
#pragma unroll
    for (int b = 0; b < PT / 4; ++b) {
      const int k = (l + L * b) % NS;
#pragma unroll
      for (int r = 1; r < 4; ++r) tw[b * 3 + r - 1] = tab[r * k * (N / (4 * NS))];
    }
  }
  template <bool INV>
  __device__ __forceinline__ static void bfly8(float2* v, const float2* tw) {
#pragma unroll
    for (int r = 1; r < 8; ++r) v[r] = tmul<INV>(v[r], tw[r - 1]);
    dft8<INV>(v);
  }

  // K transforms v[0 .. K) of one lane group side by side: each stage's
  // exchange of one is under way while the next is computed (one wave per
  // SIMD has nothing else to fill the LDS latency with).  They share one
  // scratch: a wave's LDS operations are served in order, so the next
  // transform's writes cannot overtake this one's reads.
  // sc: the group's PLEN elements of the wave's scratch.
  template <int K, bool INV>
  __device__ __forceinline__ void run(float2 (*v)[PT], float2* sc, int l) const {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if constexpr (N == 192) dft12<INV>(v[k]);
      else dft8<INV>(v[k]);
      put<1>(v[k], sc, l);
      wave_fence();
      get<1>(v[k], sc, l);
      wave_fence();
    }
    if constexpr (N == 64) {
#pragma unroll
      for (int k = 0; k < K; ++k) bfly8<INV>(v[k], t2);
    } else if constexpr (N == 32) {
#pragma unroll
      for (int k = 0; k < K; ++k) bfly4<INV, true>(v[k], t2);
    } else {
      float2 tw[kTable ? PT / 4 * 3 : 1];
      if constexpr (kTable) fetch<12>(tw, l);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if constexpr (N == 256) bfly8<INV>(v[k], t2);
        else bfly4<INV, false>(v[k], kTable ? tw : t2);
        put<2>(v[k], sc, l);
        wave_fence();
        get<2>(v[k], sc, l);
        wave_fence();
      }
      if constexpr (kTable) fetch<48>(tw, l);
#pragma unroll
      for (int k = 0; k < K; ++k) bfly4<INV, true>(v[k], kTable ? tw : t3);
    }
  }
};

}  // namespace mrpie

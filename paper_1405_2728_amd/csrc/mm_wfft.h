// Register-resident FFT of one sequence per wavefront (64 lanes), length
// n = 64 VL with VL in 1..8.
//
// Forward, natural input: lane l holds x[l + 64 r] in v[r] (r < VL).
//   S1  DFT_VL over r, twiddle by W_n^(l k1)            (k1 < VL)
//   T1  LDS transpose: lane g = 8 k1 + a gathers the 8 values l = a + 8 b
//   S2  DFT_8 over b, twiddle by W_64^(a c)
//   T2  LDS transpose: lane g = 8 k1 + c gathers the 8 values over a
//   S3  DFT_8 over a
// Output, permuted: lane g = 8 k1 + c (g < 8 VL) holds X[k1 + VL (c + 8 d)]
// in u[d] (d < 8); lanes g >= 8 VL hold nothing.
// The inverse is the exact adjoint (stages reversed, conjugate twiddles):
// permuted input as above, natural output l + 64 r, unnormalised.
//
// Transposes use a wave-private LDS buffer of wfft_buf<VL, HALF>()
// elements; the index maps are padded (one slot per 8) so that lanes 8
// apart fall on different banks.  With HALF the buffer holds the groups
// k1 < VL/2 and k1 >= VL/2 in turn (half the LDS, twice the exchanges; even
// VL only, odd VL always uses the whole buffer).
// LDS instructions of one wavefront execute in order, so the exchange within
// a wave needs no block barrier.
#pragma once

#include "mm_device.h"

namespace mmk {

__device__ __forceinline__ int wf_f1(int k1, int q) { return k1 * 72 + q + (q >> 3); }
__device__ __forceinline__ int wf_f2(int k1, int c, int a) { return k1 * 72 + c * 9 + a; }

// passes over the k1 groups of a transpose
template <int VL, bool HALF>
__host__ __device__ constexpr int wfft_passes() {
  return (HALF && VL >= 2 && VL % 2 == 0) ? 2 : 1;
}

template <int VL, bool HALF>
__host__ __device__ constexpr int wfft_buf() {
  return VL / wfft_passes<VL, HALF>() * 72;
}

template <int R, int DIR, typename T>
__device__ __forceinline__ void dft_small(cx<T>* v) {
  if constexpr (R == 2) dft2<DIR>(v);
  else if constexpr (R == 4) dft4<DIR>(v);
  else if constexpr (R == 3 || R == 5 || R == 7) dft_odd<R, DIR>(v);
  else if constexpr (R == 6) dft6<DIR>(v);
  else if constexpr (R == 8) dft8<DIR>(v);
}

// tw: table exp(-2 pi i m / (n TS)), read with stride TS (a table of a
// multiple of the length serves as well).
template <typename T, int VL, bool HALF, int TS = 1>
__device__ __forceinline__ void wfft_forward(cx<T> (&v)[VL], cx<T> (&u)[8], cx<T>* lds,
                                             const cx<T>* __restrict__ tw, int lane) {
  constexpr int NG = 8 * VL;
  constexpr int NP = wfft_passes<VL, HALF>();       // passes over the k1 groups
  constexpr int KP = VL / NP;                       // k1 groups per pass
  dft_small<VL, -1>(v);
#pragma unroll
  for (int k1 = 1; k1 < VL; ++k1) v[k1] = mul(v[k1], tw[TS * lane * k1]);
  const int k1 = lane >> 3, a = lane & 7;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
#pragma unroll
    for (int kk = 0; kk < KP; ++kk) lds[wf_f1(kk, lane)] = v[p * KP + kk];
    __builtin_amdgcn_wave_barrier();
    if (lane < NG && k1 / KP == p) {
#pragma unroll
      for (int b = 0; b < 8; ++b) u[b] = lds[wf_f1(k1 - p * KP, a + 8 * b)];
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (lane < NG) {
    dft8<-1>(u);
#pragma unroll
    for (int c = 1; c < 8; ++c) u[c] = mul(u[c], tw[TS * a * c * VL]);
  }
  const int c = lane & 7;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const bool mine = lane < NG && k1 / KP == p;
    if (mine) {
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) lds[wf_f2(k1 - p * KP, cc, a)] = u[cc];
    }
    __builtin_amdgcn_wave_barrier();
    if (mine) {
#pragma unroll
      for (int aa = 0; aa < 8; ++aa) u[aa] = lds[wf_f2(k1 - p * KP, c, aa)];
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (lane < NG) dft8<-1>(u);
}

template <typename T, int VL, bool HALF, int TS = 1>
__device__ __forceinline__ void wfft_inverse(cx<T> (&u)[8], cx<T> (&v)[VL], cx<T>* lds,
                                             const cx<T>* __restrict__ tw, int lane) {
  constexpr int NG = 8 * VL;
  constexpr int NP = wfft_passes<VL, HALF>();
  constexpr int KP = VL / NP;
  const int k1 = lane >> 3, a = lane & 7, c = lane & 7;
  if (lane < NG) dft8<1>(u);
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const bool mine = lane < NG && k1 / KP == p;
    if (mine) {
#pragma unroll
      for (int aa = 0; aa < 8; ++aa) lds[wf_f2(k1 - p * KP, c, aa)] = u[aa];
    }
    __builtin_amdgcn_wave_barrier();
    if (mine) {
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) u[cc] = lds[wf_f2(k1 - p * KP, cc, a)];
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (lane < NG) {
#pragma unroll
    for (int cc = 1; cc < 8; ++cc) u[cc] = mul(u[cc], conj(tw[TS * a * cc * VL]));
    dft8<1>(u);
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if (lane < NG && k1 / KP == p) {
#pragma unroll
      for (int b = 0; b < 8; ++b) lds[wf_f1(k1 - p * KP, a + 8 * b)] = u[b];
    }
    __builtin_amdgcn_wave_barrier();
    // element by element: as one aggregate copy the single element of the
    // 64-point transform stayed in scratch memory across the barrier
#pragma unroll
    for (int kk = 0; kk < KP; ++kk) {
      const cx<T>& e = lds[wf_f1(kk, lane)];
      v[p * KP + kk] = mk(e.x, e.y);
    }
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int kk = 1; kk < VL; ++kk) v[kk] = mul(v[kk], conj(tw[TS * lane * kk]));
  dft_small<VL, 1>(v);
}

// Packed forms of the three components together: PK sequences of length
// 64 VL per wave and component (PK VL <= 8), lane l holding x_p[l + 64 r] of
// component c in v[c][p][r].  Group k = p VL + k1 of 8 lanes takes the place
// of k1 above, so that short lengths keep 8 PK VL lanes busy in the 8-point
// stages instead of 8 VL.  The components take each stage in turn: a twiddle
// factor is loaded once for the three, and their exchanges, one after the
// other through one buffer (a wave's LDS instructions run in order), overlap.
// Transpose buffer: 72 PK VL elements.
template <typename T, int VL, int PK, int TS = 1>
__device__ __forceinline__ void wfft3_forward_pk(cx<T> (&v)[3][PK][VL], cx<T> (&u)[3][8],
                                                 cx<T>* lds, const cx<T>* __restrict__ tw,
                                                 int lane) {
  constexpr int NG = 8 * VL * PK;
  static_assert(NG <= 64, "more groups than lanes");
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int p = 0; p < PK; ++p) dft_small<VL, -1>(v[c][p]);
#pragma unroll
  for (int k1 = 1; k1 < VL; ++k1) {
    const cx<T> w = tw[TS * lane * k1];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int p = 0; p < PK; ++p) v[c][p][k1] = mul(v[c][p][k1], w);
  }
  const int k = lane >> 3, a = lane & 7;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int p = 0; p < PK; ++p)
#pragma unroll
      for (int k1 = 0; k1 < VL; ++k1) lds[wf_f1(p * VL + k1, lane)] = v[c][p][k1];
    __builtin_amdgcn_wave_barrier();
    if (lane < NG) {
#pragma unroll
      for (int b = 0; b < 8; ++b) u[c][b] = lds[wf_f1(k, a + 8 * b)];
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (lane < NG) {
#pragma unroll
    for (int c = 0; c < 3; ++c) dft8<-1>(u[c]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int cc = 1; cc < 8; ++cc) {
      const cx<T> w = tw[TS * a * cc * VL];
#pragma unroll
      for (int c = 0; c < 3; ++c) u[c][cc] = mul(u[c][cc], w);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) lds[wf_f2(k, cc, a)] = u[c][cc];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int aa = 0; aa < 8; ++aa) u[c][aa] = lds[wf_f2(k, a, aa)];
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) dft8<-1>(u[c]);
  }
}

template <typename T, int VL, int PK, int TS = 1>
__device__ __forceinline__ void wfft3_inverse_pk(cx<T> (&u)[3][8], cx<T> (&v)[3][PK][VL],
                                                 cx<T>* lds, const cx<T>* __restrict__ tw,
                                                 int lane) {
  constexpr int NG = 8 * VL * PK;
  static_assert(NG <= 64, "more groups than lanes");
  const int k = lane >> 3, a = lane & 7;
  if (lane < NG) {
#pragma unroll
    for (int c = 0; c < 3; ++c) dft8<1>(u[c]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
      for (int aa = 0; aa < 8; ++aa) lds[wf_f2(k, a, aa)] = u[c][aa];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) u[c][cc] = lds[wf_f2(k, cc, a)];
      __builtin_amdgcn_wave_barrier();
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int cc = 1; cc < 8; ++cc) {
      const cx<T> w = conj(tw[TS * a * cc * VL]);
#pragma unroll
      for (int c = 0; c < 3; ++c) u[c][cc] = mul(u[c][cc], w);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 3; ++c) dft8<1>(u[c]);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (lane < NG) {
#pragma unroll
      for (int b = 0; b < 8; ++b) lds[wf_f1(k, a + 8 * b)] = u[c][b];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int p = 0; p < PK; ++p)
#pragma unroll
      for (int kk = 0; kk < VL; ++kk) {
        const cx<T>& e = lds[wf_f1(p * VL + kk, lane)];
        v[c][p][kk] = mk(e.x, e.y);
      }
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int kk = 1; kk < VL; ++kk) {
    const cx<T> w = conj(tw[TS * lane * kk]);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int p = 0; p < PK; ++p) v[c][p][kk] = mul(v[c][p][kk], w);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int p = 0; p < PK; ++p) dft_small<VL, 1>(v[c][p]);
}

// Long forms: one sequence of 64 VL points per wave, VL = 10, 12, 14, 16.
// The 2 KP = VL groups of 8 lanes do not fit one wave, so the transposes and
// the 8-point stages run in two halves: lane 8 k + c (k < KP) of half p holds
// group k1 = p KP + k, in u[p].  Buffer: 73 KP elements (half the sequence).
template <int VL>
__host__ __device__ constexpr int wfftl_buf() { return VL / 2 * 73; }
__device__ __forceinline__ int wfl_f2(int k, int c, int a) { return k * 73 + c * 9 + a; }

template <int VL, int DIR, typename T>
__device__ __forceinline__ void dft_long(cx<T>* v) {
  static_assert(VL == 10 || VL == 12 || VL == 14 || VL == 16, "long wave FFT lengths");
  if constexpr (VL == 10) dft_comp<2, 5, DIR>(v);
  else if constexpr (VL == 12) dft_comp<4, 3, DIR>(v);
  else if constexpr (VL == 14) dft_comp<2, 7, DIR>(v);
  else dft_comp<4, 4, DIR>(v);
}

// The 8-point stages of one half with the second transpose.
template <typename T, int VL, int DIR>
__device__ __forceinline__ void wfftl_half(cx<T> (&u)[8], cx<T>* lds, const cx<T> (&w)[8], int k,
                                           int a) {
  dft8<DIR>(u);
  if (DIR < 0) {
#pragma unroll
    for (int c = 1; c < 8; ++c) u[c] = mul(u[c], w[c]);
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) lds[wfl_f2(k, DIR < 0 ? c : a, DIR < 0 ? a : c)] = u[c];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int c = 0; c < 8; ++c) u[c] = lds[wfl_f2(k, DIR < 0 ? a : c, DIR < 0 ? c : a)];
  __builtin_amdgcn_wave_barrier();
  if (DIR > 0) {
#pragma unroll
    for (int c = 1; c < 8; ++c) u[c] = mul(u[c], conj(w[c]));
  }
  dft8<DIR>(u);
}

template <typename T, int VL, int TS = 1>
__device__ __forceinline__ void wfftl_forward(cx<T> (&v)[VL], cx<T> (&u)[2][8], cx<T>* lds,
                                              const cx<T>* __restrict__ tw, int lane) {
  constexpr int KP = VL / 2;
  dft_long<VL, -1>(v);
  const int k = lane >> 3, a = lane & 7;
  const bool mine = lane < 8 * KP;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    // one half's twiddles in registers at a time
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < KP; ++kk) {
      const int k1 = p * KP + kk;
      lds[wf_f1(kk, lane)] = k1 == 0 ? v[0] : mul(v[k1], tw[TS * lane * k1]);
    }
    __builtin_amdgcn_wave_barrier();
    if (mine) {
#pragma unroll
      for (int b = 0; b < 8; ++b) u[p][b] = lds[wf_f1(k, a + 8 * b)];
    }
    __builtin_amdgcn_wave_barrier();
  }
  cx<T> w[8];
#pragma unroll
  for (int c = 1; c < 8; ++c) w[c] = tw[TS * a * c * VL];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    if (mine) wfftl_half<T, VL, -1>(u[p], lds, w, k, a);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <typename T, int VL, int TS = 1>
__device__ __forceinline__ void wfftl_inverse(cx<T> (&u)[2][8], cx<T> (&v)[VL], cx<T>* lds,
                                              const cx<T>* __restrict__ tw, int lane) {
  constexpr int KP = VL / 2;
  const int k = lane >> 3, a = lane & 7;
  const bool mine = lane < 8 * KP;
  cx<T> w[8];
#pragma unroll
  for (int c = 1; c < 8; ++c) w[c] = tw[TS * a * c * VL];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    if (mine) wfftl_half<T, VL, 1>(u[p], lds, w, k, a);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    if (mine) {
#pragma unroll
      for (int b = 0; b < 8; ++b) lds[wf_f1(k, a + 8 * b)] = u[p][b];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int kk = 0; kk < KP; ++kk) {
      const int k1 = p * KP + kk;
      v[k1] = lds[wf_f1(kk, lane)];
      if (k1 > 0) v[k1] = mul(v[k1], conj(tw[TS * lane * k1]));
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
  }
  dft_long<VL, 1>(v);
}

// Frequency held in slot d of half p by lane g (g < 8 KP).
template <int VL>
__device__ __forceinline__ int wfftl_freq(int p, int lane, int d) {
  return p * (VL / 2) + (lane >> 3) + VL * ((lane & 7) + 8 * d);
}

// Frequency index held in slot d by lane g of the permuted distribution.
template <int VL>
__device__ __forceinline__ int wfft_freq(int lane, int d) {
  return (lane >> 3) + VL * ((lane & 7) + 8 * d);
}

}  // namespace mmk

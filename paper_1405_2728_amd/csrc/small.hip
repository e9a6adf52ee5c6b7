// Small thin films in one workgroup (double precision).
//
// Grids of at most 1024 cells (32 x 16 x 2, 64 x 16 x 1 or 32 x 32 x 1 and
// below): a single workgroup holds the whole problem (m, g and s of a cell in
// one thread's registers, m for the exchange stencil and the row and column
// transforms in LDS) and runs either one field evaluation or a batch of
// minimiser iterations: pending update (eq. (7)), zero-padded FFT
// convolution, local terms, sums, stop rule and step choice (eq. (12)), with
// no kernel boundary and no trip through memory between them.
//
// Such a grid keeps at most a few CUs busy, so its time is latency.  As four
// kernels (each a chain of launch, state and data loads, barriers and
// stores) an iteration of 32 x 16 x 1 took 33.6 us and an evaluation 25.3;
// here 11.6 and 11.7 (32 x 32 x 1: 36.4 and 27.6 -> 18.0 and 17.4, 12 x 7 x 2:
// 28.6 and 20.5 -> 17.0 and 17.4).  The chain is now the instructions of a
// wave, issued about one per five cycles, so lengths are template constants
// and the transforms run per wave without block barriers: with runtime
// lengths and block-wide Stockham stages this kernel took 16.2 and 16.5 us,
// with 16 waves of one cell per thread (128 VGPRs, spills) 14.0 and 14.8.
//
// LDS: one buffer holding in turn the rows X[c][z][y] of M complex values
// and the columns Y[kx][c][z] of P (sequence index padded by one slot per 8;
// what changes from one to the other is held in registers across a barrier),
// then m[3][N], the twiddle tables and the minimiser state.
#include "mm_iter.h"
#include "mm_kernels.h"

namespace mmk {

constexpr int kSmallThreads = 512;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallCells = 2;        // cells per thread, in registers

__host__ __device__ __forceinline__ constexpr int sp(int i) { return i + (i >> 3); }
__host__ __device__ __forceinline__ constexpr int small_stride(int n) { return (n + (n >> 3)) | 1; }

struct SmallLds {
  int m, tw, st, red, total;          // byte offsets (the buffer is at 0)
};
__host__ __device__ constexpr SmallLds small_lds(int n, int nz, int M, int P) {
  SmallLds o{};
  const int X = 3 * nz * (P / 2) * small_stride(M) * 16;
  const int Y = (M + 1) * 3 * nz * small_stride(P) * 16;
  o.m = X > Y ? X : Y;
  o.tw = o.m + (3 * n * 8 + 15) / 16 * 16;
  o.st = o.tw + (2 * M + P) * 16;
  o.red = o.st + ((int)sizeof(MinState) + 15) / 16 * 16;
  o.total = o.red + kNPartial * kSmallWaves * 8;
  return o;
}

// nseq transforms of L = 32 or 64 points in natural order, in place: L / 8
// lanes per sequence with 8 values each (8 points across the lanes' stride,
// then 4 or 8 points across the lanes).  Every wave owns whole sequences, so
// that no block barrier is needed; tw: exp(-2 pi i m / (L TS)).
template <int L, int DIR, int TS>
__device__ __forceinline__ void small_fft(cx<double>* buf, int nseq, int stride,
                                          const cx<double>* tw, int wave, int lane) {
  constexpr int LPS = L / 8, SPW = 64 / LPS;
  const int a = lane % LPS;
  cx<double> w[8];
#pragma unroll
  for (int c = 1; c < 8; ++c) {
    w[c] = tw[TS * a * c];
    if (DIR > 0) w[c] = conj(w[c]);
  }
  for (int s0 = wave * SPW; s0 < nseq; s0 += kSmallWaves * SPW) {
    const int s = s0 + lane / LPS;
    cx<double>* p = buf + (s < nseq ? s : nseq - 1) * stride;   // idle lanes repeat the last one
    cx<double> u[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) u[b] = p[sp(LPS * b) + a];
    dft8<DIR>(u);
#pragma unroll
    for (int c = 1; c < 8; ++c) u[c] = mul(u[c], w[c]);
    __builtin_amdgcn_wave_barrier();
    // value c of lane a at slot LPS c + a
#pragma unroll
    for (int c = 0; c < 8; ++c) p[sp(LPS * c) + a] = u[c];
    __builtin_amdgcn_wave_barrier();
    if constexpr (L == 64) {
#pragma unroll
      for (int q = 0; q < 8; ++q) u[q] = p[sp(8 * a) + q];
      dft8<DIR>(u);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int d = 0; d < 8; ++d) p[sp(8 * d) + a] = u[d];
    } else {
      // two groups of four: c = 2 a, 2 a + 1 (slots 8 a .. 8 a + 7)
#pragma unroll
      for (int q = 0; q < 8; ++q) u[q] = p[sp(8 * a) + q];
      dft4<DIR>(u);
      dft4<DIR>(u + 4);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        p[sp(8 * d) + 2 * a] = u[d];
        p[sp(8 * d) + 2 * a + 1] = u[4 + d];
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Block sums (maximum of kPartMax) of part, in a fixed order, in every thread
// of the first wave: each wave reduces in registers, then lane 8 i + w of the
// first wave takes value i of wave w (values 8 .. 11 in a second register)
// and three more steps combine the waves.
__device__ __forceinline__ double small_scan8(double v, bool mx) {
  const double a = dpp_f64<0x111>(mx ? v : 0.0, v);
  v = mx ? fmax(v, a) : v + a;
  const double b = dpp_f64<0x112>(mx ? v : 0.0, v);
  v = mx ? fmax(v, b) : v + b;
  const double c = dpp_f64<0x114>(mx ? v : 0.0, v);
  return mx ? fmax(v, c) : v + c;   // lane 8 i + 7: the eight lanes' total
}
__device__ __forceinline__ double small_lane(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ __forceinline__ void small_reduce(double (&part)[kNPartial],
                                             double (&red)[kNPartial * kSmallWaves], int t) {
  static_assert(kSmallThreads == 512 && kNPartial <= 16 && kPartMax < 8, "eight waves");
#pragma unroll
  for (int q = 0; q < kNPartial; ++q)
    part[q] = q == kPartMax ? wave_max(part[q]) : wave_sum(part[q]);
  if ((t & 63) == 63) {
#pragma unroll
    for (int q = 0; q < kNPartial; ++q) red[q * 8 + (t >> 6)] = part[q];
  }
  __syncthreads();
  if (t < 64) {
    const double v0 = small_scan8(red[t], (t >> 3) == kPartMax);
    const double v1 = small_scan8(t < (kNPartial - 8) * 8 ? red[64 + t] : 0.0, false);
#pragma unroll
    for (int q = 0; q < kNPartial; ++q)
      part[q] = q < 8 ? small_lane(v0, 8 * q + 7) : small_lane(v1, 8 * (q - 8) + 7);
  }
}

// nit > 0: a batch of at most nit minimiser iterations on a.m (updated in
// place), g and s, driven by and written back to state st; it ends early
// when the run does.  nit == 0: one evaluation at a.m into the outputs of a
// and Hd_out, its sums decided into st where set.
template <int NZ, int M, int P>
__global__ void __launch_bounds__(kSmallThreads)
k_small(LocalArgs a, double* __restrict__ mio, double* __restrict__ sio, int nit, MinState* st,
        const double* __restrict__ Tt, int tstride, double scale,
        const cx<double>* __restrict__ twx, const cx<double>* __restrict__ twy,
        double* __restrict__ Hd_out, double Ms, double V) {
  using T = double;
  constexpr int NY = P / 2;                  // rows per layer held (ny <= NY)
  constexpr int SX = small_stride(M), SY = small_stride(P);
  constexpr int rows = 3 * NZ * NY, ncol = (M + 1) * 3 * NZ, nk = P / 2 + 1;
  constexpr int EY = (ncol * NY + kSmallThreads - 1) / kSmallThreads;
  constexpr int EX = rows * M / kSmallThreads;
  static_assert(rows * M % kSmallThreads == 0, "whole rounds");
  extern __shared__ __align__(16) unsigned char smem[];
  const int nx = a.nx, ny = a.ny, N = a.nx * a.ny * NZ;
  const SmallLds o = small_lds(N, NZ, M, P);
  cx<T>* B = reinterpret_cast<cx<T>*>(smem);
  T* Br = reinterpret_cast<T*>(smem);
  T* ml = reinterpret_cast<T*>(smem + o.m);
  cx<T>* tx = reinterpret_cast<cx<T>*>(smem + o.tw);
  cx<T>* ty = tx + 2 * M;
  MinState* sl = reinterpret_cast<MinState*>(smem + o.st);
  double(&red)[kNPartial * kSmallWaves] =
      *reinterpret_cast<double(*)[kNPartial * kSmallWaves]>(smem + o.red);
  if (a.done != nullptr && *a.done != 0) return;
  const bool run = nit > 0;
  const int t0 = (int)threadIdx.x;
  // this thread's cells t, t + 512
  double m[kSmallCells][3], g[kSmallCells][3], s[kSmallCells][3];
  int ix[kSmallCells], nb[kSmallCells][6];
  T* gio = static_cast<T*>(a.g);
#pragma unroll
  for (int u = 0; u < kSmallCells; ++u) {
    const int i = t0 + u * kSmallThreads;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      m[u][c] = i < N ? a.m[c * N + i] : 0.0;
      g[u][c] = run && i < N ? gio[c * N + i] : 0.0;
      s[u][c] = run && i < N ? sio[c * N + i] : 0.0;
    }
    // place in X and neighbours (missing ones: the cell itself)
    const int j = min(i, N - 1);
    const int row = j / nx, x = j - row * nx, z = row / ny, y = row - z * ny;
    ix[u] = 2 * ((z * NY + y) * SX + sp(x >> 1)) + (x & 1);
    nb[u][0] = x > 0 ? j - 1 : j;
    nb[u][1] = x < nx - 1 ? j + 1 : j;
    nb[u][2] = y > 0 ? j - nx : j;
    nb[u][3] = y < ny - 1 ? j + nx : j;
    nb[u][4] = z > 0 ? j - nx * ny : j;
    nb[u][5] = z < NZ - 1 ? j + nx * ny : j;
  }
  for (int i = t0; i < 2 * M; i += kSmallThreads) tx[i] = twx[i];
  for (int i = t0; i < P; i += kSmallThreads) ty[i] = twy[i];
  if (st != nullptr)
    for (int i = t0; i < (int)(sizeof(MinState) / 8); i += kSmallThreads)
      reinterpret_cast<unsigned long long*>(sl)[i] = reinterpret_cast<unsigned long long*>(st)[i];
  __syncthreads();
  for (int it = 0; it < (run ? nit : 1); ++it) {
    if (run && sl->done != 0) break;         // block-uniform: last written before a barrier
    // read again: index arithmetic is not hoisted out of the loop (spills)
    const int t = thread_index();
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // zero padding of the rows, then pending update, rows and stencil copy
#pragma unroll
    for (int e = 0; e < EX; ++e) {
      const int i = t + e * kSmallThreads, j = i % M;
      T* q = Br + 2 * ((i / M) * SX + sp(j));
      if (2 * j >= nx) q[0] = 0.0;
      if (2 * j + 1 >= nx) q[1] = 0.0;
    }
    const bool upd = run && sl->pending != 0;
#pragma unroll
    for (int u = 0; u < kSmallCells; ++u) {
      const int i = t + u * kSmallThreads;
      if (i >= N) continue;
      if (upd) {
        double mo[3];
        cayley_step(m[u], g[u], sl->last_tau, mo);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          s[u][c] = mo[c] - m[u][c];
          m[u][c] = mo[c];
        }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        ml[c * N + i] = m[u][c];
        Br[c * (2 * NZ * NY * SX) + ix[u]] = m[u][c];
      }
    }
    __syncthreads();
    small_fft<M, -1, 2>(B, rows, SX, tx, wave, lane);
    __syncthreads();
    // real-input split: column (k, component, layer), position y, zero padded
    {
      cx<T> v[EY];
#pragma unroll
      for (int e = 0; e < EY; ++e) {
        const int i = t + e * kSmallThreads, yy = i % NY, col = i / NY;
        const int k = col / (3 * NZ), q = col - k * 3 * NZ;
        v[e] = mk(0.0, 0.0);
        if (yy < ny && col < ncol) {
          const cx<T>* xr = B + (q * NY + yy) * SX;
          const cx<T> zk = xr[sp(k % M)];
          const cx<T> zc = conj(xr[sp((M - k) % M)]);
          v[e] = scl(add(add(zk, zc), rot90<-1>(mul(tx[k], sub(zk, zc)))), 0.5);
        }
      }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < EY; ++e) {
        const int i = t + e * kSmallThreads, yy = i % NY, col = i / NY;
        if (col < ncol) {
          B[col * SY + sp(yy)] = v[e];
          B[col * SY + sp(yy + NY)] = mk(0.0, 0.0);
        }
      }
    }
    __syncthreads();
    small_fft<P, -1, 1>(B, ncol, SY, ty, wave, lane);
    __syncthreads();
    // tensor product with the z convolution at every (kx, ky)
#pragma unroll 2
    for (int i = t; i < (M + 1) * P; i += kSmallThreads) {
      const int k = i / P, ky = i % P;
      const bool neg = ky > P / 2;
      const T sy = neg ? -1.0 : 1.0;
      const T* tk = Tt + (size_t)k * tstride + (neg ? P - ky : ky) * 6;
      cx<T>* col = B + k * 3 * NZ * SY + sp(ky);
      cx<T> F[3][NZ];
#pragma unroll
      for (int q = 0; q < 3 * NZ; ++q) F[q / NZ][q % NZ] = col[q * SY];
#pragma unroll
      for (int z = 0; z < NZ; ++z) {
        cx<T> H[3] = {mk(0.0, 0.0), mk(0.0, 0.0), mk(0.0, 0.0)};
#pragma unroll
        for (int zp = 0; zp < NZ; ++zp) {
          const int dz = z - zp;
          const T sz = dz < 0 ? -1.0 : 1.0;
          const T* e = tk + (dz < 0 ? -dz : dz) * nk * 6;
          const T xx = e[0], yy = e[1], zz = e[2], xy = e[3] * sy, xz = e[4] * sz,
                  yz = e[5] * sy * sz;
          const cx<T> fx = F[0][zp], fy = F[1][zp], fz = F[2][zp];
          H[0] = add(H[0], add(add(scl(fx, xx), scl(fy, xy)), scl(rot90<1>(fz), xz)));
          H[1] = add(H[1], add(add(scl(fx, xy), scl(fy, yy)), scl(rot90<1>(fz), yz)));
          H[2] = add(H[2], add(add(scl(rot90<1>(fx), xz), scl(rot90<1>(fy), yz)), scl(fz, zz)));
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) col[(c * NZ + z) * SY] = scl(H[c], scale);
      }
    }
    __syncthreads();
    small_fft<P, 1, 1>(B, ncol, SY, ty, wave, lane);
    __syncthreads();
    // Z[k] of the rows from X[k], X[M - k] (columns 0 and M are real)
    {
      cx<T> v[EX];
#pragma unroll
      for (int e = 0; e < EX; ++e) {
        const int i = t + e * kSmallThreads, k = i % M, r = i / M, yy = r % NY, q = r / NY;
        cx<T> Xk = B[(k * 3 * NZ + q) * SY + sp(yy)];
        cx<T> Xc = conj(B[((M - k) * 3 * NZ + q) * SY + sp(yy)]);
        if (k == 0) Xk.y = Xc.y = 0.0;
        v[e] = scl(add(add(Xk, Xc), rot90<1>(mul(conj(tx[k]), sub(Xk, Xc)))), 0.5);
      }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < EX; ++e) {
        const int i = t + e * kSmallThreads;
        B[(i / M) * SX + sp(i % M)] = v[e];
      }
    }
    __syncthreads();
    small_fft<M, 1, 2>(B, rows, SX, tx, wave, lane);
    __syncthreads();
    // local terms (compute_cell's formulas), sums
    double part[kNPartial] = {};
    double H[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) H[c] = run ? sl->H[c] : a.H[c];
    const bool bb = run && sl->k > 0;
#pragma unroll
    for (int u = 0; u < kSmallCells; ++u) {
      const int i = t + u * kSmallThreads;
      if (i >= N) continue;
      const double ku = a.ku_map != nullptr ? a.ku_map[i] : a.ku;
      const double(&mi)[3] = m[u];
      double hd[3], hex[3], h[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        hd[c] = Br[c * (2 * NZ * NY * SX) + ix[u]];
        const T* mc = ml + c * N;
        hex[c] = a.cx * ((mc[nb[u][0]] - mi[c]) + (mc[nb[u][1]] - mi[c])) +
                 a.cy * ((mc[nb[u][2]] - mi[c]) + (mc[nb[u][3]] - mi[c])) +
                 a.cz * ((mc[nb[u][4]] - mi[c]) + (mc[nb[u][5]] - mi[c]));
      }
      const double mu = mi[0] * a.u[0] + mi[1] * a.u[1] + mi[2] * a.u[2];
      const double pan = a.kan * ku * mu;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double han = pan * a.u[c];
        h[c] = hd[c] + hex[c] + han + H[c];
        if (Hd_out != nullptr) Hd_out[c * N + i] = hd[c];
        if (a.Hout != nullptr) a.Hout[c * N + i] = h[c];
        if (a.Hex_out != nullptr) a.Hex_out[c * N + i] = hex[c];
        if (a.Han_out != nullptr) a.Han_out[c * N + i] = han;
      }
      if (st == nullptr) continue;
      part[3] += mi[0] * hd[0] + mi[1] * hd[1] + mi[2] * hd[2];
      part[4] += mi[0] * hex[0] + mi[1] * hex[1] + mi[2] * hex[2];
      part[5] += ku * mu * mu;
      part[6] += mi[0] * H[0] + mi[1] * H[1] + mi[2] * H[2];
      part[8] += mi[0];
      part[9] += mi[1];
      part[10] += mi[2];
      const double ax = mi[1] * h[2] - mi[2] * h[1];
      const double ay = mi[2] * h[0] - mi[0] * h[2];
      const double az = mi[0] * h[1] - mi[1] * h[0];
      const double gn[3] = {mi[1] * az - mi[2] * ay, mi[2] * ax - mi[0] * az,
                            mi[0] * ay - mi[1] * ax};
      const double gg = gn[0] * gn[0] + gn[1] * gn[1] + gn[2] * gn[2];
      part[7] = fmax(part[7], gg);
      part[11] += gg;
      if (bb) {
        const double y0 = gn[0] - g[u][0], y1 = gn[1] - g[u][1], y2 = gn[2] - g[u][2];
        part[0] += s[u][0] * s[u][0] + s[u][1] * s[u][1] + s[u][2] * s[u][2];
        part[1] += s[u][0] * y0 + s[u][1] * y1 + s[u][2] * y2;
        part[2] += y0 * y0 + y1 * y1 + y2 * y2;
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) g[u][c] = gn[c];
    }
    if (st == nullptr) break;
    small_reduce(part, red, t);
    if (t == 0) finish_decision(sl, load_finish_in(sl), part, Ms, V);
    __syncthreads();
  }
  if (run) {
#pragma unroll
    for (int u = 0; u < kSmallCells; ++u) {
      const int i = t0 + u * kSmallThreads;
      if (i >= N) continue;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        mio[c * N + i] = m[u][c];
        gio[c * N + i] = g[u][c];
        sio[c * N + i] = s[u][c];
      }
    }
  }
  if (st != nullptr)
    for (int i = t0; i < (int)(sizeof(MinState) / 8); i += kSmallThreads)
      reinterpret_cast<unsigned long long*>(st)[i] = reinterpret_cast<unsigned long long*>(sl)[i];
}

static_assert(sizeof(MinState) % 8 == 0, "the state is copied by 8-byte words");

constexpr int kSmallLdsMax = 160 * 1024 - 512;

template <int NZ, int M, int P>
static bool small_inst(int nx, int ny, int nz, int& m, int& p) {
  if (nz != NZ || nx > M || 2 * ny > P || nx * ny * nz > kSmallThreads * kSmallCells) return false;
  if (small_lds(nx * ny * nz, NZ, M, P).total > kSmallLdsMax) return false;
  m = M;
  p = P;
  return true;
}

// Padded lengths of a grid that one workgroup holds (false: none)
bool small_shape(int nx, int ny, int nz, int& M, int& P) {
  return small_inst<1, 32, 32>(nx, ny, nz, M, P) || small_inst<1, 64, 32>(nx, ny, nz, M, P) ||
         small_inst<1, 32, 64>(nx, ny, nz, M, P) || small_inst<2, 32, 32>(nx, ny, nz, M, P);
}

template <int NZ, int M, int P>
static void small_launch(hipStream_t s, const LocalArgs& a, double* mio, double* sio, int nit,
                         MinState* st, const double* Tt, int tstride, double scale,
                         const void* twx, const void* twy, double* Hd_out, double Ms, double V) {
  const size_t lds = (size_t)small_lds(a.nx * a.ny * a.nz, NZ, M, P).total;
  auto k = k_small<NZ, M, P>;
  (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k, dim3(1), dim3(kSmallThreads), lds, s, a, mio, sio, nit, st, Tt, tstride,
                     scale, (const cx<double>*)twx, (const cx<double>*)twy, Hd_out, Ms, V);
}

void launch_small(hipStream_t s, const LocalArgs& a, double* mio, double* sio, int nit,
                  MinState* st, int M, int P, const double* Tt, int tstride, double scale,
                  const void* twx, const void* twy, double* Hd_out, double Ms, double V) {
  auto go = a.nz == 2 ? small_launch<2, 32, 32>
            : M == 64 ? small_launch<1, 64, 32>
            : P == 64 ? small_launch<1, 32, 64>
                      : small_launch<1, 32, 32>;
  go(s, a, mio, sio, nit, st, Tt, tstride, scale, twx, twy, Hd_out, Ms, V);
}

}  // namespace mmk

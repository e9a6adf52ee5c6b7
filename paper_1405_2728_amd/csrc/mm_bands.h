// Distance bands of the demag tensor's set-up (tensor.hip): the closed form
// below 6 h, the 6-point rule below 16 h, the 4-point rule below 40 h and the
// 3-point rule beyond, h the largest cell edge.
//
// Two kernels share the offsets out by their band and each skips the other's,
// so both must place every offset alike, also those exactly on an edge (with
// cubic cells (24, 32, 0) is 40 h away).  A sum of products left to the
// compiler may be contracted one way in one kernel and another way in the
// next, and an offset on the edge would then be left unwritten: the roundings
// are written out here.  Host code (the tests) may include this file.
#ifndef MM_BANDS_H
#define MM_BANDS_H

namespace mmk {

enum Band { kBandClosed, kBand6, kBand4, kBand3 };

__host__ __device__ inline Band offset_band(double X, double Y, double Z, double h) {
  const double r2 = __builtin_fma(Z, Z, __builtin_fma(X, X, Y * Y));
  return r2 < 36.0 * h * h     ? kBandClosed
         : r2 < 256.0 * h * h  ? kBand6
         : r2 < 1600.0 * h * h ? kBand4
                               : kBand3;
}

}  // namespace mmk

#endif  // MM_BANDS_H

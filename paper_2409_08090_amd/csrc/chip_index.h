// chip_index.h -- index arithmetic of the in-LDS transforms of chip.hip (host
// and device; no HIP dependency, so a host build can check it).
//
// A line of L = E^k f elements (E = 8 or 16, f < E) is held by L / E threads,
// E elements each, and runs as Stockham stages of radix E and one of radix f:
// stage s of radix R, after stages whose radices multiply to Ns, takes for
// butterfly b the elements at b + q L / R, q < R, multiplies element q by
// exp(2 pi i q (b mod Ns) / (Ns R)), takes their length-R DFT and leaves
// output q at (b / Ns) Ns R + (b mod Ns) + q Ns.  Thread t holds the
// butterflies b = t + (L / E) k, k < E / R, in registers k R + q.
#pragma once

#if defined(__HIPCC__)
#define CF_HD __host__ __device__
#else
#define CF_HD
#endif

namespace mils {
namespace chipfft {

// elements of a thread for grids of L cells
CF_HD constexpr int elems(int L) { return L == 8192 ? 16 : 8; }
// stages of radix E, and the radix of the last stage (1: none)
CF_HD constexpr int nfull(int L) {
  int k = 0;
  for (int m = L; m >= elems(L); m /= elems(L)) ++k;
  return k;
}
CF_HD constexpr int tailr(int L) {
  int m = L;
  while (m >= elems(L)) m /= elems(L);
  return m;
}
CF_HD constexpr int nstages(int L) { return nfull(L) + (tailr(L) > 1 ? 1 : 0); }
CF_HD constexpr int radix(int L, int s) { return s < nfull(L) ? elems(L) : tailr(L); }
CF_HD constexpr int ns(int L, int s) {
  int p = 1;
  for (int i = 0; i < s; ++i) p *= radix(L, i);
  return p;
}
CF_HD constexpr int threads(int L) { return L / elems(L); }
CF_HD constexpr int in_pos(int L, int s, int b, int q) { return b + q * (L / radix(L, s)); }
CF_HD constexpr int out_pos(int L, int s, int b, int q) {
  return (b / ns(L, s)) * ns(L, s) * radix(L, s) + (b % ns(L, s)) + q * ns(L, s);
}
// register holding output t + (L / E) j after the last stage
CF_HD constexpr int reg_of(int L, int j) {
  return (j % (elems(L) / radix(L, nstages(L) - 1))) * radix(L, nstages(L) - 1) +
         j / (elems(L) / radix(L, nstages(L) - 1));
}
// LDS slot of position p (16-byte elements): one pad per 16 (8), so that the
// first stage's writes, E apart, step through the banks
CF_HD constexpr int pad_shift(int L) { return elems(L) == 16 ? 4 : 3; }
CF_HD constexpr int pad(int L, int p) { return p + (p >> pad_shift(L)); }
CF_HD constexpr int line_pitch(int L) { return L + (L >> pad_shift(L)); }

}  // namespace chipfft
}  // namespace mils

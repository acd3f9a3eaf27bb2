// kargs.hpp -- a kernel's arguments read from its argument block.
//
// An argument struct passed by value is loaded once, at the kernel's entry, and
// what does not fit the scalar registers is then moved through vector lanes at
// every use.  Here a piece of work reads what it needs where it needs it
// (scalar loads that hit the cache).  Passing the block's address through an
// empty asm before a piece keeps the compiler from hoisting its reads.  The
// pointers come with their address spaces: arrays in global memory, and the
// grid's tables and walls, which the kernel does not write, in constant memory, so that an entry
// at a uniform index is a scalar load also behind stores and atomics.
//
// The argument struct is the kernel's first parameter, so it starts at offset
// 0 of the block.
#pragma once

#include <cstddef>

#include "dsw_common.hpp"
#include "dsw_internal.hpp"

namespace dsw {

#define DSW_AS1 __attribute__((address_space(1)))
#define DSW_AS4 __attribute__((address_space(4)))
using KPtr = const DSW_AS4 char *;

template <class T>
__device__ __forceinline__ T karg(KPtr p, unsigned off) { return *(const DSW_AS4 T *)(p + off); }
__device__ __forceinline__ const double *ktab(KPtr p, unsigned off) { // a table: constant, scalar loads
  return (const double *)karg<const DSW_AS4 double *>(p, off);
}
__device__ __forceinline__ double *karr(KPtr p, unsigned off) {
  return (double *)karg<DSW_AS1 double *>(p, off);
}
__device__ __forceinline__ Fields kfields(KPtr p, unsigned off) {
  return {karr(p, off), karr(p, off + 8), karr(p, off + 16), karr(p, off + 24), karr(p, off + 32)};
}

__device__ __forceinline__ Geo kgeo(KPtr p, unsigned at) {
  Geo g;
#define DSW_KI(f) g.f = karg<int>(p, at + offsetof(Geo, f))
#define DSW_KD(f) g.f = karg<double>(p, at + offsetof(Geo, f))
#define DSW_KT(f) g.f = ktab(p, at + offsetof(Geo, f))
  DSW_KI(nr); DSW_KI(nt); DSW_KI(np); DSW_KI(npf); DSW_KI(periodic); DSW_KI(pole_lo); DSW_KI(pole_hi);
  DSW_KD(dr); DSW_KD(dt); DSW_KD(dp); DSW_KD(idr); DSW_KD(idt); DSW_KD(idp);
  DSW_KT(rc); DSW_KT(rf); DSW_KT(sc); DSW_KT(cc); DSW_KT(sf); DSW_KT(cf); DSW_KT(irc); DSW_KT(irf);
  DSW_KT(isc); DSW_KT(ctc); DSW_KT(isf); DSW_KT(ctf); DSW_KT(scx);
#undef DSW_KI
#undef DSW_KD
#undef DSW_KT
  return g;
}
__device__ __forceinline__ Mat kmat(KPtr p, unsigned at) {
  Mat m;
#define DSW_KM(f) m.f = karg<double>(p, at + offsetof(Mat, f))
  DSW_KM(gam); DSW_KM(Rg); DSW_KM(pinf); DSW_KM(mu); DSW_KM(kap); DSW_KM(omega); DSW_KM(g_r);
#undef DSW_KM
  return m;
}
// the velocities on the phi walls are read at uniform indices
__device__ __forceinline__ Wall kwall(KPtr p, unsigned at) {
  Wall w;
#define DSW_KT(f) w.f = ktab(p, at + offsetof(Wall, f))
#define DSW_KA(f) w.f = karr(p, at + offsetof(Wall, f))
  DSW_KT(ur_p1); DSW_KT(ur_p2); DSW_KT(ut_p1); DSW_KT(ut_p2);
  DSW_KA(ur_t1); DSW_KA(ur_t2); DSW_KA(ut_r1); DSW_KA(ut_r2); DSW_KA(uf_r1); DSW_KA(uf_r2); DSW_KA(uf_t1); DSW_KA(uf_t2);
#undef DSW_KT
#undef DSW_KA
  return w;
}
static_assert(offsetof(Fields, T) == 32, "kfields reads this layout");

} // namespace dsw

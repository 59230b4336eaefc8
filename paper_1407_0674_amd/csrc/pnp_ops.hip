// One translation unit of launch tables: the pass kernels of one precision
// (PNP_OPS_T: float or double), grid size (PNP_OPS_N) and FFT schedule
// (PNP_OPS_SCHED), in both tile shapes where the narrow one exists.  The
// build compiles this file once per (precision, size, schedule).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pnp_kernels.hip"
#include "pnp_launch.hpp"

#ifndef PNP_OPS_T
#error "PNP_OPS_T (float or double) must be defined"
#endif
#ifndef PNP_OPS_N
#error "PNP_OPS_N (grid size) must be defined"
#endif
#ifndef PNP_OPS_SCHED
#error "PNP_OPS_SCHED (0 primary or 1 secondary FFT schedule) must be defined"
#endif

namespace pnp {

template <typename T, int N, int V = 0> struct Launch {
  using G = Geo<T, N, V>;
  static constexpr int EZD = ezd_of<T, N, V>();
  using GD = GeoD<T, N, EZD, V>;
  // the derivative pass of small grids runs one wavefront per field
  static constexpr bool kFieldWaves = N <= 96;
  static constexpr int EZF = ezf_of<T, N, V>();
  // Workgroups per tile of the y and z passes: on small grids the fields of a
  // tile are spread over workgroups of their own, until the launch has about
  // two wavefronts for each of the 1024 SIMDs; with more tiles than that, one
  // workgroup walks all of a tile's fields and makes its tables once.  (Each
  // field's arithmetic is the same.)  Three species, y inverse of the weighted
  // densities: FP64 16^3 12.2 -> 6.6 us, 64^3 16.6 -> 9.9; mixed 32^3 12.7 -> 6.7,
  // 96^3 24.5 -> 16.1; no change from 128^3 on.
  static int split(int tiles, int threads, int fields) {
    const int waves = tiles * ((threads + 63) / 64);
    return std::max(1, std::min(fields, 2048 / std::max(1, waves)));
  }
  // maxS: the largest species count among the launch's instances
  static int table_items(int maxS) { return maxS * ((maxS + 3) / 4 * 4) + maxS; }  // pair-table entries + hs species
  static void tables(const TableArgs* a, int count, int M, const SpeciesMix& sm, hipStream_t s) {
    const dim3 g((M + 255) / 256, table_items(sm.maxS()), count);
    if (sm.bulk) hipLaunchKernelGGL((k_tables<T, true>), g, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_tables<T, false>), g, dim3(256), 0, s, a);
  }
  static void zfwd(const EvalArgs* a, int count, int maxS, hipStream_t s) {
    const int b = G::RZ * G::TZ, g = count * G::tiles_z;
    hipLaunchKernelGGL((k_zfwd<T, N, V>), dim3(g, split(g, b, maxS)), dim3(b), 0, s, a, nullptr, g, 0, 0, 1);
  }
  // the first pass and the tables of tcount instances (M: their most classes)
  static void zfwd_tables(const EvalArgs* a, int count, const TableArgs* ta, int tcount, int M, const SpeciesMix& sm,
                          hipStream_t s) {
    if constexpr (N < 192) {
      const int b = G::RZ * G::TZ, g = count * G::tiles_z, y = split(g, b, sm.maxS());
      const int items = table_items(sm.maxS()), chunks = (M + b - 1) / b;
      const int extra = (int)(((long)tcount * items * chunks + y - 1) / y);
      hipLaunchKernelGGL((k_zfwd<T, N, V, true>), dim3(g + extra, y), dim3(b), 0, s, a, ta, g, tcount, items, chunks);
    } else {
      tables(ta, tcount, M, sm, s);
      zfwd(a, count, sm.maxS(), s);
    }
  }
  // part: kPartAll, kPartMain (main-array tiles) or kPartNyquist (Nyquist-plane tiles)
  static int tiles_y(int part) { return part == kPartAll ? G::tiles_y : part == kPartMain ? (N * G::H) / G::PY : N / G::PY; }
  static int tiles_x(int part) { return part == kPartAll ? G::tiles_x : part == kPartMain ? (N * G::H) / G::PX : N / G::PX; }
  // the general x passes keep the same pencils per workgroup
  static constexpr int TXG = N / G::EXG, TXC = N / G::EXC;
  static constexpr bool four = G::kXMax < 4;
  // of four species where kXMax is three, whichever schedule (mixed back pass at
  // 256^3: 390 us with 8, 408 with the 4 that half of the streamed 8 would be)
  static constexpr int EX4 = sizeof(T) == 4 ? 8 : 4;
  // maxf: the most fields of an instance (kVecItems in the vector mode)
  static void ystep(const EvalArgs* a, int count, int sel, int nf, int maxf, bool fwd, int part, hipStream_t s) {
    const int tiles = count * tiles_y(part);
    const dim3 g(tiles, split(tiles, G::PY * G::TY, nf == kVecMode ? kVecItems : maxf)), b(G::PY * G::TY);
    if (fwd)
      hipLaunchKernelGGL((k_ystep<T, N, true, V>), g, b, 0, s, a, sel, nf, part);
    else
      hipLaunchKernelGGL((k_ystep<T, N, false, V>), g, b, 0, s, a, sel, nf, part);
  }
  // The x passes of a launch list: the streamed kernels for up to kXMax
  // species (compiled for the largest such count in the list; an instance's
  // arithmetic does not depend on it), the accumulating ones above; at 256^3
  // the back pass of four species is a streamed kernel of its own (16 elements
  // per thread would not fit its registers).  Each skips the others' instances.
  static void xfwd(const EvalArgs* a, int count, const SpeciesMix& sm, int part, hipStream_t s) {
    const dim3 g(count * tiles_x(part)), b(G::PX * G::TX);
    int general = 1;  // fewest species of the accumulating kernel
    if constexpr (G::kXStream) {
      general = 5;
      switch (sm.upto(G::kXMax)) {
        case 1: hipLaunchKernelGGL((k_xfwd<T, N, 1, G::EX, G::PX>), g, b, 0, s, a, 1, part); break;
        case 2: hipLaunchKernelGGL((k_xfwd<T, N, 2, G::EX, G::PX>), g, b, 0, s, a, 1, part); break;
        case 3: hipLaunchKernelGGL((k_xfwd<T, N, 3, G::EX, G::PX>), g, b, 0, s, a, 1, part); break;
        case 4: if constexpr (!four) hipLaunchKernelGGL((k_xfwd<T, N, 4, G::EX, G::PX>), g, b, 0, s, a, 1, part); break;
        default: break;
      }
      if constexpr (four) general = 4;
    }
    if (sm.maxS() >= general)
      hipLaunchKernelGGL((k_xfwd_acc<T, N, G::EXG, G::PX>), g, dim3(G::PX * TXG), 0, s, a, general, part);
  }
  // phi: also sum Phi_hs per workgroup (free-energy calls); fmask: the
  // hard-sphere functionals among the instances (1 Rosenfeld, 2 White Bear),
  // one launch of the matching variant each
  static void zderiv(const EvalArgs* a, int count, bool phi, int fmask, hipStream_t s) {
    if constexpr (kFieldWaves) {
      using GF = GeoF<T, N, EZF>;
      const dim3 g(count * GF::tiles), b(GF::threads);
      if (fmask & 1) {
        if (phi) hipLaunchKernelGGL((k_zderiv_fields<T, N, true, false, EZF>), g, b, 0, s, a);
        else hipLaunchKernelGGL((k_zderiv_fields<T, N, false, false, EZF>), g, b, 0, s, a);
      }
      if (fmask & 2) {
        if (phi) hipLaunchKernelGGL((k_zderiv_fields<T, N, true, true, EZF>), g, b, 0, s, a);
        else hipLaunchKernelGGL((k_zderiv_fields<T, N, false, true, EZF>), g, b, 0, s, a);
      }
    } else {
      const dim3 g(count * GD::tiles), b(GD::RDD * GD::TZD);
      if (fmask & 1) {
        if (phi) hipLaunchKernelGGL((k_zderiv<T, N, true, false, EZD, V>), g, b, 0, s, a);
        else hipLaunchKernelGGL((k_zderiv<T, N, false, false, EZD, V>), g, b, 0, s, a);
      }
      if (fmask & 2) {
        if (phi) hipLaunchKernelGGL((k_zderiv<T, N, true, true, EZD, V>), g, b, 0, s, a);
        else hipLaunchKernelGGL((k_zderiv<T, N, false, true, EZD, V>), g, b, 0, s, a);
      }
    }
  }
  template <bool BULK> static void xback_of(const EvalArgs* a, int count, const SpeciesMix& sm, int part, hipStream_t s) {
    const dim3 g(count * tiles_x(part)), b(G::PX * G::TX);
    // The streamed FP64 kernels always carry the test for a bulk table: its block
    // ends the density phase, without it the compiler holds values of that phase
    // across the last transforms (three species: 188 B of spills at 128^3, 81
    // against 66 us; 256^3 508 against 462; other counts the same).
    constexpr bool TEST = BULK || sizeof(T) == 8;
    switch (sm.upto(G::kXMax)) {
      case 1: hipLaunchKernelGGL((k_xback<T, N, 1, G::EX, G::PX, TEST>), g, b, 0, s, a, 1, part); break;
      case 2: hipLaunchKernelGGL((k_xback<T, N, 2, G::EX, G::PX, TEST>), g, b, 0, s, a, 1, part); break;
      case 3: hipLaunchKernelGGL((k_xback<T, N, 3, G::EX, G::PX, TEST>), g, b, 0, s, a, 1, part); break;
      case 4: if constexpr (!four) hipLaunchKernelGGL((k_xback<T, N, 4, G::EX, G::PX, TEST>), g, b, 0, s, a, 1, part); break;
      default: break;
    }
    if constexpr (four)
      if (sm.has(4)) hipLaunchKernelGGL((k_xback<T, N, 4, EX4, G::PX, TEST>), g, dim3(G::PX * (N / EX4)), 0, s, a, 4, part);
    if (sm.maxS() > 4)
      hipLaunchKernelGGL((k_xback_chunked<T, N, 4, G::EXC, G::PX, BULK>), g, dim3(G::PX * TXC), 0, s, a, 5, part);
  }
  static void xback(const EvalArgs* a, int count, const SpeciesMix& sm, int part, hipStream_t s) {
    if (sm.bulk) xback_of<true>(a, count, sm, part, s);
    else xback_of<false>(a, count, sm, part, s);
  }
  // maxf: the most fields of an instance
  static void zinv(const EvalArgs* a, int count, int sel, int maxf, hipStream_t s) {
    const int b = G::RZ * G::TZ, g = count * G::tiles_z;
    hipLaunchKernelGGL((k_zinv<T, N, V>), dim3(g, split(g, b, maxf)), dim3(b), 0, s, a, sel);
  }
  // the three terms of a per-term call
  static void zinv_terms(const EvalArgs* a, int S, hipStream_t s) {
    const int b = G::RZ * G::TZ;
    hipLaunchKernelGGL((k_zinv<T, N, V, true>), dim3(G::tiles_z, split(G::tiles_z, b, S)), dim3(b), 0, s, a, 2);
  }
  static void xplain(const EvalArgs* a, int count, int nf, bool fwd, hipStream_t s) {
    if (fwd)
      hipLaunchKernelGGL((k_xplain<T, N, true, G::EX, G::PX>), dim3(count * G::tiles_x), dim3(G::PX * G::TX), 0, s,
                         a, 0, nf);
    else
      hipLaunchKernelGGL((k_xplain<T, N, false, G::EX, G::PX>), dim3(count * G::tiles_x), dim3(G::PX * G::TX), 0,
                         s, a, 0, nf);
  }
  static void xport(const EvalArgs* a, int nf, double* buf, int to_numpy, hipStream_t s) {
    const long total = (long)nf * N * N * (N / 2 + 1);
    const int blocks = (int)std::min<long>((total + 255) / 256, 4096);
    hipLaunchKernelGGL((k_export<T, N>), dim3(blocks), dim3(256), 0, s, a, nf, buf, to_numpy);
  }
  // passes whose secondary schedule differs from the primary one
  using G0 = Geo<T, N, 0>;
  using G2 = Geo<T, N, 2>;
  static constexpr uint32_t sched_alt =
      (G0::EZ != G2::EZ ? (1u << 1) | (1u << 9) : 0u) |
      (G0::EY != G2::EY ? (1u << 2) | (1u << 4) | (1u << 6) | (1u << 8) : 0u) |
      (G0::EX != G2::EX ? (1u << 3) | (1u << 7) : 0u) | ((kFieldWaves ? ezf_of<T, N, 0>() != ezf_of<T, N, 2>() : ezd_of<T, N, 0>() != ezd_of<T, N, 2>()) ? 1u << 5 : 0u);
  static constexpr Ops ops{tables, zfwd, zfwd_tables, ystep, xfwd, zderiv, xback, kFieldWaves ? GeoF<T, N, EZF>::tiles : GD::tiles, zinv, zinv_terms, xplain, xport, sched_alt};
};

template <typename T, int N, int V> const Ops* ops_inst() { return &Launch<T, N, V>::ops; }

// PNP_OPS_SCHED (0 or 1): the FFT schedule of this translation unit
template const Ops* ops_inst<PNP_OPS_T, PNP_OPS_N, 2 * PNP_OPS_SCHED>();
#if PNP_OPS_N <= 128
template const Ops* ops_inst<PNP_OPS_T, PNP_OPS_N, 2 * PNP_OPS_SCHED + 1>();
#endif

}  // namespace pnp

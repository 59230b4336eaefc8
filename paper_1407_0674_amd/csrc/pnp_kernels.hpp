// Shared definitions between the HIP kernels and the host driver of the
// cDFT excess-chemical-potential evaluator.
#pragma once
#include <stdint.h>

namespace pnp {

constexpr int kMaxSpecies = 8;
constexpr int kMaxPairs = kMaxSpecies * (kMaxSpecies + 1) / 2;
constexpr int kFields = 10;  // n0, n1, n2, n3, n1v(x,y,z), n2v(x,y,z)

// Storage of the two vector weighted densities n_bv (b = 1, 2) and of their
// derivative fields.  Every vector weight is the gradient of a ball weight
// (omega_2v = -grad omega_3, omega_1v = omega_2v / (4 pi R)), so with
// k0 = 2 pi / L and s_c the signed index along axis c (0 on that axis's
// Nyquist plane)
//   n_1v,c(k) = i s_c Q(k),  Q = k0 sum_i rho_i w_i^3 / (4 pi R_i),
//   n_2v,c(k) = i s_c k0 n_3(k),
// and each component is formed in the pass that transforms its own axis.
// Vector 2 needs no spectrum of its own: its y and z components are formed
// from that of n3, and the derivative with respect to them joins that of n3
// on the way back (the back pass multiplies both by w_i^3).  Against a second
// [z] slot for vector 2: one field less in every pass from the x forward to
// the back pass, 436 instead of 468 bytes per grid point at three species in
// mixed precision, and two y transforms and one x transform less each way
// (256^3 mixed 85 us less per evaluation of 1.66 ms; 128^3 FP64 496 -> 455 us).
// Field slots 4..6 hold vector 1, 7..8 vector 2 (slot 9 is a real field of
// the weighted-density output only; no pass stores a spectrum there):
//   after the x-forward pass:  [4] = i s_x Q, [6] = Q, [7] = i s_x k0 n3, [3] = n3
//   after the y-inverse pass:  also [5] = i s_y Q, [8] = i s_y k0 n3
//                              (the z pass forms i s_z [6] and i s_z k0 [3])
//   after the z derivative pass: [4], [5] = F_1x, F_1y, [6] = i s_z F_1z,
//                              [7], [8] = F_2x, F_2y, [3] = F_3 - i s_z k0 F_2z
//   after the y-forward pass:  [6] += i s_y F_1y, [3] -= i s_y k0 F_2y
// and the back pass forms i s_x F_1x + [6] and [3] - i s_x k0 F_2x.
constexpr int kSlotX = 4, kSlotY = 5, kSlotZ = 6, kVecStride = 3;
constexpr int kSlotN3 = 3;                       // n3, and the [z] slot of vector 2
constexpr int kFieldZ2 = kSlotZ + kVecStride;    // the real field n_2v,z
constexpr int kBackFields = 7;  // fields the back pass reads: 0..2, 4, 6, 3, 7

// Spectral field layout: the main block [kx][ky][kz < n/2] with each kx
// plane (n * n/2 complex values) followed by spec_pad unused values, then the
// Nyquist plane kz = n/2 as [kx][ky].  An x-pass workgroup loads one
// 16-pencil row from every kx plane at once; with an unpadded power-of-two
// plane stride (256 KB at 256^3 in FP32) those rows share their low address
// bits and crowd a few memory channels (a plain copy with the x-pass access
// pattern at 256^3: 4.7 TB/s unpadded, 5.6 TB/s padded).  Pads of an odd
// number of 128-byte rows also speed up the y passes.  Measured per
// evaluation: 256^3 1.713 -> 1.687 ms (FP32 spectra, 48 values) and
// 3.527 -> 3.466 ms (FP64, 16 values); 192^3 0.871 -> 0.867 and
// 1.755 -> 1.733 ms; no change at 128^3, whose fields stay largely in the
// Infinity Cache.  tsize: bytes of a real component.
constexpr int64_t spec_pad(int n, int tsize) { return n >= 192 ? (tsize == 4 ? 48 : 16) : 0; }
constexpr int64_t spec_plane(int n, int tsize) { return (int64_t)n * (n / 2) + spec_pad(n, tsize); }
constexpr int64_t spec_fstride(int n, int tsize) { return n * spec_plane(n, tsize) + (int64_t)n * n; }

// status word bits (word 0); word 1 holds the smallest offending flat index,
// words 2 and 3 the residual of a Picard step (a double's bit pattern)
enum : uint32_t { kStPacking = 1u, kStNonFinite = 2u, kStOverflow = 4u };

// Per-instance description read by every pass kernel (device resident).
struct EvalArgs {
  int32_t n;          // grid points per axis
  int32_t S;          // species
  int32_t hs_on;      // hard-sphere term (passes x-forward, derivatives, back phase A)
  int32_t pair_on;    // EC and/or SW pair term in the back pass
  int32_t np;         // S (S + 1) / 2
  int32_t nreal;      // fields written by the real-space output pass
  int32_t final_mode; // 1: add constant, write mu and exp(-mu); 0: plain real output
  uint32_t zmul_mask; // real-output pass: fields whose z spectrum is multiplied by i s_z first
  int64_t fstride;    // complex elements per spectral field (spec_fstride)
  double inv_n3;      // 1 / n^3
  double kscale;      // 2 pi / L: |k| = kscale * sqrt(jx^2 + jy^2 + jz^2)
  double R[kMaxSpecies];
  double area[kMaxSpecies];     // 4 pi R^2
  double inv4piR[kMaxSpecies];  // 1 / (4 pi R)
  double cfin[kMaxSpecies];     // constant added to beta mu in the final pass
  int32_t Sp;         // S rounded up to a multiple of 4 (row length of the pair table)
  int32_t hs_wb;      // 1: modified (White Bear) hard-sphere functional, 0: Rosenfeld
  const double* rho;  // [S][n^3] input densities
  void* specA;        // S spectral fields (densities)
  void* specB;        // 9 spectral fields in 10 slots (weighted densities, then derivatives)
  void* specC;        // S spectral fields (chemical potentials)
  const void* hs_tab;    // [M][S][2]: j0(kR), 4 pi R^3 j1(kR)/(kR)
                         // (FP64 path only; the FP32 path evaluates them in registers)
  const void* pair_tab;  // [M][S][Sp]: entry [m][j][i] = combined pair kernel G_ij
  double* out;        // real output [nreal][n^3] (mu_ex or weighted densities)
  double* slot;       // [S][n^3] exp(-mu) or null
  uint32_t* status;   // four words, cleared by the first pass
  double* dc;         // [S] k = 0 part of each result where the back pass sums it in
                      // double (FP32, up to four species); cleared by the first pass
  double* phi_part;   // per-workgroup sums of Phi_hs from the derivative pass, or null
  // aperiodic mode: the first pass reads an ext_n^3 domain [S][ext_n]^3 and
  // treats it as zero-extended onto the n^3 grid (domain at the corner)
  int32_t ext_n;
  // aperiodic mode with EC: [M][Sp] sum_j G^EC_ij rho_b,j per |k|^2 class, or
  // null; the back pass subtracts it times the transform of the domain's
  // indicator (the response to the domain's bulk densities)
  const void* bulk_tab;
};

// Per-instance arguments of the radial table builder.
struct TableArgs {
  int32_t n, S, np, M;
  double kscale;  // 2 pi / L
  double R[kMaxSpecies];
  double ec_pref[kMaxPairs];  // q_i q_j l_B (0 when EC is off)
  double sigma[kMaxPairs];    // (d_i + d_j) / 2
  double Bsig[kMaxPairs];     // B_ij / sigma_ij
  double sw_pref[kMaxPairs];  // -beta c_sw eps_ij (0 when SW is off)
  double rout[kMaxPairs];
  int8_t pidx[kMaxSpecies][kMaxSpecies];  // pair slot of (i, j)
  int32_t Sp;
  void* hs_tab;
  void* pair_tab;
  void* bulk_tab;                // [M][Sp] or null (EvalArgs)
  double rho_b[kMaxSpecies];     // bulk densities (bulk_tab only)
};

}  // namespace pnp

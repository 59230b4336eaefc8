// The launch table of the evaluation's passes for one (precision, grid
// size, launch variant): host functions that launch each pass kernel over a
// device table of per-instance arguments.  The tables of each (precision,
// size, FFT schedule) are built in their own translation unit (pnp_ops.hip
// compiled once per triple), so they compile in parallel; the ABI's
// translation unit only declares ops_inst.
#pragma once
#include <hip/hip_runtime.h>

#include "pnp_kernels.hpp"

namespace pnp {

// The species counts of a launch list (they select the x-pass kernels).
struct SpeciesMix {
  bool bulk = false;  // the instances have bulk tables (EvalArgs::bulk_tab)
  uint32_t mask = 0;  // bit S set: some instance has S species
  void add(int S) { mask |= 1u << S; }
  bool has(int S) const { return (mask >> S) & 1u; }
  // the largest count up to hi (0: none)
  int upto(int hi) const {
    int m = 0;
    for (int S = 1; S <= hi; ++S)
      if (has(S)) m = S;
    return m;
  }
  int maxS() const { return upto(kMaxSpecies); }
};

struct Ops {
  void (*tables)(const TableArgs*, int, int, const SpeciesMix&, hipStream_t);  // count, M, species
  void (*zfwd)(const EvalArgs*, int, int, hipStream_t);  // count, most species
  void (*zfwd_tables)(const EvalArgs*, int, const TableArgs*, int, int, const SpeciesMix&, hipStream_t);  // count, tables, their count, M, species
  void (*ystep)(const EvalArgs*, int, int, int, int, bool, int, hipStream_t);  // count, sel, nf, most fields, fwd, part
  void (*xfwd)(const EvalArgs*, int, const SpeciesMix&, int, hipStream_t);   // count, species, part
  void (*zderiv)(const EvalArgs*, int, bool, int, hipStream_t);
  void (*xback)(const EvalArgs*, int, const SpeciesMix&, int, hipStream_t);  // count, species, part
  int zderiv_tiles;  // workgroups of the derivative pass per instance
  void (*zinv)(const EvalArgs*, int, int, int, hipStream_t);  // count, sel, most fields
  void (*zinv_terms)(const EvalArgs*, int, hipStream_t);  // species
  void (*xplain)(const EvalArgs*, int, int, bool, hipStream_t);
  void (*xport)(const EvalArgs*, int, double*, int, hipStream_t);
  uint32_t sched_alt;  // passes (bit p: pass p) whose secondary FFT schedule differs from the primary
};

// Grids up to kNarrowMax also have the narrow tile shape (V bit 0); larger
// ones already launch thousands of workgroups per pass.  Every size has both
// FFT schedules (V bit 1).
constexpr int kNarrowMax = 128;

// the launch table of (T, N, V); defined by the translation unit of
// (T, N, schedule)
template <typename T, int N, int V> const Ops* ops_inst();

}  // namespace pnp

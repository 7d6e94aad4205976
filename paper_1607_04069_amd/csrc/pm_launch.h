// Host launchers of the library's kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pm_internal.h"

namespace pm {

size_t field_lds_bytes(int N);
template <typename R> hipError_t launch_load(const KArgs<R>&, int64_t np_e, int64_t np_i, double sig_e,
                                             double sig_i, hipStream_t);
template <typename R> hipError_t launch_deposit_all(const KArgs<R>&, int64_t nmax, hipStream_t);
template <typename R> hipError_t launch_sort(const KArgs<R>&, int grid, hipStream_t);
template <typename R> hipError_t launch_field(const KArgs<R>&, int want_phi, hipStream_t);
// the step reads the case's arguments from their device copy (dev_args); A is
// the host copy, for the launch shape
template <typename R> hipError_t launch_step(const KArgs<R>& A, const KArgs<R>* dev_args, int grid, int nwork,
                                             int count_cells, hipStream_t);
template <typename R> int step_blocks_per_cu(int N, int unroll, int waves, bool batch);
template <typename R> int mcc_blocks_per_cu(int N, bool batch);
template <typename R> hipError_t launch_mcc(const KArgs<R>& A, const KArgs<R>* dev_args, int grid, int count_cells,
                                            hipStream_t);
template <typename R> hipError_t launch_mcc_batch(const KArgs<R>* cases, const uint32_t* work,
                                                  const uint32_t* nblocks, int grid, int maxN, int count_cells,
                                                  hipStream_t);
template <typename R> hipError_t launch_diag_finalize(const KArgs<R>&, int bin, hipStream_t);  // bin < 0: window
template <typename R> hipError_t launch_step_batch(const KArgs<R>* cases, const uint32_t* work,
                                                   const uint32_t* nblocks, int grid, int maxN, int unroll,
                                                   int waves, int count_cells, hipStream_t);
template <typename R> hipError_t launch_sort_batch(const KArgs<R>* cases, const uint32_t* work,
                                                   const uint32_t* nblocks, int grid, int maxN, hipStream_t);
// fused steps: launch i since the last commit; the commit after n of them
template <typename R> int fused_blocks_per_cu(int N, bool flux, bool batch);
template <typename R> int fused_tiles(int64_t n_e, int64_t n_i);
template <typename R> int fused_tile();                        // slots of a pass
template <typename R> hipError_t launch_fused(const KArgs<R>& A, int grid, int i, int count_cells, hipStream_t);
template <typename R> hipError_t launch_commit(const KArgs<R>& A, const KArgs<R>* dev_args, int n, int count_cells,
                                               hipStream_t);
template <typename R> hipError_t launch_fused_batch(const KArgs<R>* cases, const uint32_t* work,
                                                    const uint32_t* nblocks, int grid, int maxN, int i,
                                                    int count_cells, hipStream_t);
template <typename R> hipError_t launch_commit_batch(const KArgs<R>* cases, const uint32_t* work, int grid, int maxN,
                                                     int n, int count_cells, hipStream_t);
hipError_t launch_scan_cells(const CaseConst&, const GridPtrs&, Ctrl*, hipStream_t);
hipError_t launch_diag_reset(const CaseConst&, const GridPtrs&, Ctrl*, hipStream_t);

// sputter yield and test-particle flight

// The flight's constants in its own precision (in registers, not converted there).
struct TpFloat {
  float L, inv_L;
  float inv_nu;              // 1 / n_gas (sigma g)_max (infinity without gas)
  float sig_gas;             // sqrt(k_B T / m_gas)
  float m_ratio, M_ratio;    // m/(m+M), M/(m+M)
  float sg_exp;              // 2 - 2 omega: (sigma g) ~ g^sg_exp for VHS
  float log2_gcap;           // log2 of the majorant's relative speed
  float dt;                  // fixed flight time (0: gridless, from the majorant)
  float nu_dt;               // n_gas (sigma g)_max dt: the fixed-step probability at the majorant
  float xbin, inv_xbin;      // cell width and its inverse, m
  float s_max, u_s;          // Thompson inversion
  float v_per_sqrt_ev;       // sqrt(2 e / m_test)
  float e_half_m;            // 0.5 m / e: eV per (m/s)^2
  float ebin, tbin;
};

struct TpConst {
  TpFloat f;
  double dt;                 // for a fixed step's clock, its steps times dt
  int n_ebins, n_tbins;
  int n_xbins;               // cells of the track-length profiles (0: none)
  int mode;
  int scatter;               // 0 VHS isotropic, 1 M1
  int electrode;             // emission from the target (0) or the substrate (1)
  int64_t e_max;
  int64_t n_atoms, first_atom;
  uint64_t seed, job;
  float expect, hit;         // candidate events of an atom and the part that collides, roughly (for the launch's shape alone)
  int wlog, widest;          // lanes per atom at the start and at most: 2^wlog, 2^widest (set by the launcher)
  int64_t run, first_run;    // atoms a wavefront takes at a time; the first run that is no wavefront's own
};

struct TpTally {              // device tallies (zeroed before a run)
  uint64_t sum[4];             // impact energies at the target, at the substrate (2^-20 eV), events, collisions
  uint64_t n_sub, n_tgt, n_unf;
  uint64_t overflow;
  uint64_t pad0[8];
  uint64_t next;               // atoms taken by the flight's wavefronts beyond their first runs
  uint64_t pad1[15];
};

struct TpTrace {
  int32_t* wall;
  uint32_t* events;
  float* energy_ev;
  float* theta_deg;
  float* tof_s;
  float* vx;
  float* vy;
  float* vz;
};

// prof: [4][n_xbins + 1] int64 track-length tallies (partial-cell times, full-cell
// time differences, partial-cell displacements, full-cell displacement
// differences), or null
hipError_t launch_tp_flight(TpConst, TpTally* tally, uint64_t* e_hist, uint64_t* th_hist, uint64_t* tof_hist,
                            TpTrace trace, int64_t* prof, hipStream_t);
// track-length tallies -> [4][nx] doubles: time (s), displacement (m), density (m^-3), mean v_x (m/s)
hipError_t launch_tp_profiles(const int64_t* prof, int nx, double h, double per_atom, double* out, hipStream_t st);
hipError_t launch_zero_u64(void* p, size_t bytes, hipStream_t st);
// Bytes of the per-GPU scratch of pm_run_test_particles_static, and its device
// address on the current device (looked up once per device).
constexpr size_t kTpScratchBytes = (size_t)1 << 20;
hipError_t tp_scratch(void** ptr);
hipError_t launch_yield(const uint64_t* iedf, const double* ybin, int n_ebins, uint64_t seed,
                        uint64_t job, int electrode, uint64_t* taken, uint64_t* out, hipStream_t st);

}  // namespace pm

// Test-particle kernels for gfx950 (Sec. IV.B of arXiv:1607.04069).
//
// k_yield applies the yield rule of 'Wall Interactions' to the recorded Ar+
// impacts on the target: N = ceil(Y) checks R_f <= Y/N per impact.
//
// k_tp_flight flies sputtered Al atoms: Thompson energy and cosine angle at
// emission, straight flights with free-flight times tau = -ln(R_f) / nu_max
// (Eq. (5) with the null-collision majorant of Eq. (6)), a Maxwellian argon
// partner at each candidate, acceptance sigma(g) g / (sigma g)_max with the VHS
// cross section of Eq. (8) (or M1 scattering: deflection pi (1 - b/b_max) about
// the relative velocity, 'Binary Interactions'), isotropic centre-of-mass scattering (Eq. (10) with
// chi = 2 arccos(b/b_max)), and sticking electrodes.  An atom flies in registers,
// on one lane while there are atoms for all of them, on more when there are not;
// lanes whose atom ends take the next one from a common queue, so a wavefront
// keeps its lanes busy while atoms with very different event counts finish.
// Tallies go to LDS and are flushed once per workgroup.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <mutex>

#include "philox.h"
#include "pm_internal.h"
#include "pm_launch.h"

namespace pm {

// With taken (live injection) only the impacts i >= taken[b] that arrived since
// the previous such call are used, and taken[b] then moves to the record's
// count: impact i of bin b keys its draws by (i, b), so the calls of a window
// add up to exactly what one call over the whole record draws.
__global__ __launch_bounds__(kBlock) void k_yield(const uint64_t* iedf, const double* ybin, int n_ebins,
                                                  uint64_t seed, uint64_t job, uint64_t aux_hi, uint64_t* taken,
                                                  uint64_t* out) {
  __shared__ uint32_t s_cnt;
  const int b = blockIdx.x;
  if (threadIdx.x == 0) s_cnt = 0;
  const uint64_t c = iedf[b];
  const uint64_t t0 = taken ? taken[b] : 0;
  __syncthreads();
  const double Y = ybin[b];
  const int N = (int)ceil(Y);
  uint32_t k = 0;
  if (N > 0) {
    const double p = Y / (double)N;
    for (uint64_t i = t0 + threadIdx.x; i < c; i += kBlock)
      for (int n = 0; n < N; ++n) {
        const Words4 w = philox4x64_10(i, (uint64_t)b, rng_tag(SP_YIELD, PU_YIELD), aux_hi | (uint64_t)n, seed, job);
        if (u_hi<double>(w.w0) <= p) ++k;
      }
  }
  atomicAdd(&s_cnt, k);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (s_cnt) atomicAdd((unsigned long long*)&out[0], (unsigned long long)s_cnt);
    if (c > t0) atomicAdd((unsigned long long*)&out[1], (unsigned long long)(c - t0));
    if (taken && c > t0) taken[b] = c;
  }
}

hipError_t launch_yield(const uint64_t* iedf, const double* ybin, int n_ebins, uint64_t seed,
                        uint64_t job, int electrode, uint64_t* taken, uint64_t* out, hipStream_t st) {
  hipLaunchKernelGGL(k_yield, dim3(n_ebins), dim3(kBlock), 0, st, iedf, ybin, n_ebins, seed, job,
                     (uint64_t)electrode << 32, taken, out);
  return hipGetLastError();
}

// The event loop's variates use the hardware's approximate log2, exp2, sqrt,
// reciprocal and sine/cosine (about 1 ulp; the sine and cosine take the angle
// in revolutions): a random direction or waiting time needs no correctly
// rounded result, and these are most of the loop's arithmetic.
__device__ __forceinline__ float fast_ln(float u) { return __builtin_amdgcn_logf(u) * 0.6931471805599453f; }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
// sin and cos of 2 pi r
__device__ __forceinline__ void fast_sincos_rev(float r, float* s, float* c) {
  *s = __builtin_amdgcn_sinf(r);
  *c = __builtin_amdgcn_cosf(r);
}

__device__ __forceinline__ float wrapf(float v, float L, float inv_L) { return fmaf(-floorf(v * inv_L), L, v); }

// An atom in flight at the start of its next event.  The products and sums of
// its motion are written as explicit fused operations, so that the two loops
// below round them alike.  (The lateral position never matters: the gas is
// uniform and the lateral directions are periodic.)
struct Atom {
  float x, vx, vy, vz, t;
  uint32_t e;          // candidate events so far
};

// A new atom from its emission draw (counter (id, 0, source tag)).
__device__ __forceinline__ void emit(const TpConst& T, const Uniforms8<float>& U, Atom& a) {
  const float s = fast_sqrt(U[0]) * T.f.s_max;
  const float E = T.f.u_s * s / (1.0f - s);            // Thompson flux law by inversion
  const float ct = fast_sqrt(U[1]);                      // theta = arccos(sqrt(R_f))
  const float st = fast_sqrt(1.0f - U[1]);
  float sp, cp;
  fast_sincos_rev(U[2], &sp, &cp);
  const float v = fast_sqrt(E) * T.f.v_per_sqrt_ev;
  // from the target into +x, or from the substrate (re-sputtering) into -x
  a.vx = T.electrode ? -(v * ct) : v * ct;
  a.vy = v * st * cp;
  a.vz = v * st * sp;
  a.x = T.electrode ? T.f.L : 0.0f;
  a.t = 0.0f;
  a.e = 0;
}

// The eight uniforms of an atom's draw.  The key words are made opaque here, so
// that each draw adds up its round keys on the scalar unit: kept over the loop,
// they overflow the scalar registers and come back through vector ones.
__device__ __forceinline__ Uniforms8<float> draw_atom(const TpConst& T, int64_t k, uint64_t index, uint64_t tag) {
  uint64_t k0 = T.seed, k1 = T.job;
  asm volatile("" : "+s"(k0), "+s"(k1));
  return draw8<float>((uint64_t)(T.first_atom + k), index, tag, k0, k1);
}

// Track-length profile units: time in 2^-40 s, displacement in 2^-24 cells.
constexpr float kTimeFx = 1099511627776.0f;
constexpr float kCellFx = 16777216.0f;

// rint(x) as an int64: the hardware's f32 -> i32 conversion when |x| < 2^31
// (almost always), the general (longer) conversion otherwise; the two agree.
__device__ __forceinline__ long long rint_i64(float x) {
  const float r = rintf(x);
  if (__builtin_expect(fabsf(r) < 2147483520.0f, 1)) return (long long)(int)r;
  return (long long)r;
}

// Tallies of one workgroup.  Sums that an ending atom adds to are kept per lane
// of a wavefront, so that the atoms that end in one pass never meet on one
// address (summed by a loop over those lanes, they took a fifth of the flight at
// low pressure).  Beside histograms that leave no room for that the lanes share
// one sum (kCols = 1).
template <int kCols>
struct TpShared {
  unsigned long long sum[4][kCols];     // TpTally's four sums, in its order
  uint32_t n_tgt, n_unf, over;
};

template <int kCols>
struct TpLds {
  unsigned long long *pt, *dt, *px, *dd;   // [n_xbins + 1] each
  uint32_t *e, *th, *tof;
  TpShared<kCols>* sh;
};

// Add a straight flight xa -> xb at x-velocity vx to the LDS profile tallies:
// partial cells directly (time overlap / |vx|, displacement overlap * sign), the
// cells crossed end to end as a difference (+ at the first, - past the last) of
// their common time dx / |vx| and displacement dx * sign, summed up at the end.
template <int kCols>
__device__ __forceinline__ void track_tally(const TpConst& T, const TpLds<kCols>& S, float xa, float xb, float vx) {
#pragma clang fp contract(off)   // a cell edge at the wall: the product is rounded before the difference
  if (vx == 0.0f) return;
  const float lo = fminf(xa, xb), hi = fmaxf(xa, xb);
  const float inv_v = __builtin_amdgcn_rcpf(fabsf(vx));
  const float ih = T.f.inv_xbin, h = T.f.xbin;
  const int n = T.n_xbins;
  const float cl = lo * ih, ch = hi * ih;
  const int ia = min(max((int)cl, 0), n - 1), ib = min(max((int)ch, 0), n - 1);
  const bool one = ia == ib;
  const float fa = (float)(ia + 1) - cl;               // cells of the partial ends
  // displacements are at most one cell, 2^24 units: always an int32
  const int da = (int)rintf((one ? (hi - lo) * ih : fa) * kCellFx);
  atomicAdd(&S.pt[ia], (unsigned long long)rint_i64((one ? hi - lo : fa * h) * inv_v * kTimeFx));
  atomicAdd(&S.px[ia], (unsigned long long)(long long)(vx > 0.0f ? da : -da));
  if (one) return;
  const float fb = ch - (float)ib;
  const int db = (int)rintf(fb * kCellFx);
  atomicAdd(&S.pt[ib], (unsigned long long)rint_i64(fb * h * inv_v * kTimeFx));
  atomicAdd(&S.px[ib], (unsigned long long)(long long)(vx > 0.0f ? db : -db));
  if (ib > ia + 1) {
    const long long full = rint_i64(h * inv_v * kTimeFx);
    const long long cell = vx > 0.0f ? (long long)kCellFx : -(long long)kCellFx;
    atomicAdd(&S.dt[ia + 1], (unsigned long long)full);
    atomicAdd(&S.dt[ib], (unsigned long long)(-full));
    atomicAdd(&S.dd[ia + 1], (unsigned long long)cell);
    atomicAdd(&S.dd[ib], (unsigned long long)(-cell));
  }
}

// What an event's draw gives before the atom's state enters: the wait, the gas
// partner's Maxwellian velocity, and the uniforms of the test and the scattering.
struct EventDraw {
  float tau;
  float r0, c0, r1, c1;  // partner: bx = r0 c0, bz = r1 c1
  float s0;              // by = r0 s0
  float u5, u6, u7;
};

__device__ __forceinline__ void draw_partner(const TpConst& T, const Uniforms8<float>& U, EventDraw& D) {
  D.r0 = T.f.sig_gas * fast_sqrt(-2.0f * fast_ln(U[1]));
  D.r1 = T.f.sig_gas * fast_sqrt(-2.0f * fast_ln(U[3]));
  fast_sincos_rev(U[2], &D.s0, &D.c0);
  D.c1 = __builtin_amdgcn_cosf(U[4]);
  D.u5 = U[5];
  D.u6 = U[6];
  D.u7 = U[7];
}

__device__ __forceinline__ EventDraw draw_event(const TpConst& T, const Uniforms8<float>& U) {
  EventDraw D;
  D.tau = -fast_ln(U[0]) * T.f.inv_nu;
  draw_partner(T, U, D);
  return D;
}

// The atom's relative velocity to the partner and the test against the majorant.
struct Partner {
  float gx, gy, gz, gm;  // relative velocity and speed
  float ratio;           // (sigma g) / (sigma g)_max; with a fixed step the probability n sigma g dt of Eq. (7)
};

template <bool kFixed>
__device__ __forceinline__ Partner meet(const TpConst& T, const EventDraw& D, const Atom& a) {
  Partner p;
  p.gx = fmaf(-D.c0, D.r0, a.vx);
  p.gy = fmaf(-D.s0, D.r0, a.vy);
  p.gz = fmaf(-D.c1, D.r1, a.vz);
  p.gm = fast_sqrt(fmaf(p.gz, p.gz, fmaf(p.gx, p.gx, p.gy * p.gy)));
  // accept with (sigma g)/(sigma g)_max = (g/g_cap)^(2 - 2 omega)
  p.ratio = __builtin_amdgcn_exp2f(T.f.sg_exp * (__builtin_amdgcn_logf(p.gm) - T.f.log2_gcap)) *
            (kFixed ? T.f.nu_dt : 1.0f);
  return p;
}

// The velocity after a real collision.
__device__ __forceinline__ void scatter(const TpConst& T, const Partner& p, const EventDraw& D, Atom& a) {
  const float mr = T.f.m_ratio, Mr = T.f.M_ratio;
  const float bx = D.r0 * D.c0, by = D.r0 * D.s0, bz = D.r1 * D.c1;
  float sp, cp;
  fast_sincos_rev(D.u7, &sp, &cp);
  if (T.scatter == 0) {
    // VHS: isotropic new relative direction
    const float cc = fmaf(2.0f, D.u6, -1.0f);
    const float sc = fast_sqrt(fmaxf(0.0f, fmaf(-cc, cc, 1.0f)));
    const float w = Mr * p.gm, ws = w * sc;
    a.vx = fmaf(w, cc, fmaf(mr, a.vx, Mr * bx));
    a.vy = fmaf(ws, cp, fmaf(mr, a.vy, Mr * by));
    a.vz = fmaf(ws, sp, fmaf(mr, a.vz, Mr * bz));
  } else {
    // M1: g turned by chi = pi (1 - sqrt(U6)) at azimuth psi about itself, in
    // the basis e1 = (x-hat x g)/|.|, e2 = g-hat x e1 (e1 = y-hat along x)
    float sc, cc;
    fast_sincos_rev(0.5f * (1.0f - fast_sqrt(D.u6)), &sc, &cc);     // chi = pi (1 - sqrt(U6))
    float gp;
    {
#pragma clang fp contract(off)
      gp = fast_sqrt(p.gz * p.gz + p.gy * p.gy);
    }
    float hx, hy, hz;
    if (gp > 1e-6f * p.gm) {
      const float ip = __builtin_amdgcn_rcpf(gp);
      const float cg = cp * p.gm, sx = sp * p.gx;
      hx = fmaf(cc, p.gx, sc * sp * gp);
      hy = fmaf(cc, p.gy, -(ip * (sc * fmaf(p.gy, sx, p.gz * cg))));
      hz = fmaf(cc, p.gz, ip * (sc * fmaf(p.gy, cg, -(p.gz * sx))));
    } else {
      hx = cc * p.gx;
      hy = cp * (sc * p.gm);
      hz = sp * (sc * p.gm) * (p.gx < 0.0f ? -1.0f : 1.0f);
    }
    a.vx = fmaf(Mr, hx, fmaf(mr, a.vx, Mr * bx));
    a.vy = fmaf(Mr, hy, fmaf(mr, a.vy, Mr * by));
    a.vz = fmaf(Mr, hz, fmaf(mr, a.vz, Mr * bz));
  }
}

// x and t of the lanes of a row: lane i's flight starts where lane i - 1's ends.
// All lanes walk the one chain, each step taking the wait of lane j of its row
// (row_newbcast:j), and lane j + 1 keeps the point reached.
template <int j = 0>
__device__ __forceinline__ void row_chain(float vx, float tau, int i, float& x, float& t, float y, float s) {
  if constexpr (j < 15) {
    const float tj = __uint_as_float(
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(tau), 0x150 + j, 0xf, 0xf, true));
    y = fmaf(vx, tj, y);
    s += tj;
    const bool here = i == j + 1;
    x = here ? y : x;
    t = here ? s : t;
    row_chain<j + 1>(vx, tau, i, x, t, y, s);
  }
}
__device__ __forceinline__ void row_chain(float vx, float tau, int i, float& x, float& t) {
  row_chain<0>(vx, tau, i, x, t, x, t);
}

// With a fixed step nearly every test fails (the probability is that of one
// step), and it fails for certain when U5 exceeds the probability at the largest
// relative speed the partner can give: the uniforms lie above 2^-24, so each
// Box-Muller radius is at most sqrt(48 ln 2) = 5.77 and the partner's speed at
// most 8.16 thermal widths.  The margin covers the approximate functions.
__device__ __forceinline__ float ratio_bound(const TpConst& T, const Atom& a) {
  const float v = fast_sqrt(fmaf(a.vz, a.vz, fmaf(a.vx, a.vx, a.vy * a.vy)));
  return 1.001f * T.f.nu_dt *
         __builtin_amdgcn_exp2f(T.f.sg_exp * (__builtin_amdgcn_logf(fmaf(8.2f, T.f.sig_gas, v)) - T.f.log2_gcap));
}

// Tally an atom that ended at wall (0 target, 1 substrate, 2 in the gas after
// e_max events) with time of flight tof.
template <int kCols>
__device__ __forceinline__ void finish(const TpConst& T, const TpLds<kCols>& S, const TpTrace& tr, int64_t k,
                                       const Atom& a, int wall, float tof, uint32_t coll, int lane) {
  const int col = lane % kCols;
  const float v2 = fmaf(a.vz, a.vz, fmaf(a.vx, a.vx, a.vy * a.vy));
  const float E = T.f.e_half_m * v2;
  const float th = acosf(fminf(fabsf(a.vx) / sqrtf(v2), 1.0f)) * 57.29577951308232f;
  atomicAdd(&S.sh->sum[2][col], (unsigned long long)a.e);
  atomicAdd(&S.sh->sum[3][col], (unsigned long long)coll);
  if (wall < 2) {
    atomicAdd(&S.sh->sum[wall][col], (unsigned long long)rint_i64(E * 1048576.0f));   // E 2^20 is exact in FP32
    if (wall) {
      atomicAdd(&S.e[(int)fminf(fmaxf(E / T.f.ebin, 0.0f), (float)(T.n_ebins - 1))], 1u);
      atomicAdd(&S.th[(int)fminf(fmaxf(th, 0.0f), (float)(kTpThetaBins - 1))], 1u);
      atomicAdd(&S.tof[(int)fminf(fmaxf(tof / T.f.tbin, 0.0f), (float)(T.n_tbins - 1))], 1u);
    } else {
      atomicAdd(&S.sh->n_tgt, 1u);
    }
  } else {
    atomicAdd(&S.sh->n_unf, 1u);
  }
  if (tr.wall) tr.wall[k] = wall;
  if (tr.events) tr.events[k] = a.e;
  if (tr.energy_ev) tr.energy_ev[k] = E;
  if (tr.theta_deg) tr.theta_deg[k] = th;
  if (tr.tof_s) tr.tof_s[k] = tof;
  if (tr.vx) tr.vx[k] = a.vx;
  if (tr.vy) tr.vy[k] = a.vy;
  if (tr.vz) tr.vz[k] = a.vz;
}

// Atoms waiting to be flown, as one wavefront sees them: its own run of
// consecutive atoms, and behind it the runs no wavefront has taken yet.
struct Queue {
  int64_t at, end;     // the run
  bool dry;            // no atoms are left anywhere
};

// The next `want` atoms of the queue (uniform): *first and the count got.  A
// run that is used up is followed by the next free one of T.run atoms.
__device__ __forceinline__ int take(const TpConst& T, Queue& q, unsigned long long* next, int want, int lane,
                                    int64_t* first) {
  if (q.at >= q.end && !q.dry) {
    // with every atom in some wavefront's own run there is nothing to ask for (the
    // thousands of atomics on one address that say so took 20 us of 280, 209404 atoms
    // at 0.06 Pa)
    q.at = T.first_run;
    if (T.first_run < T.n_atoms) {
      unsigned long long r = 0;
      if (lane == 0) r = atomicAdd(next, (unsigned long long)T.run);
      r = (unsigned long long)__builtin_amdgcn_readfirstlane((int)(uint32_t)r) & 0xFFFFFFFFull |
          (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(r >> 32)) << 32;
      q.at += (int64_t)r;
    }
    q.end = min(q.at + T.run, T.n_atoms);
    if (q.at >= T.n_atoms) {
      q.dry = true;
      q.at = q.end = 0;
    }
  }
  const int got = (int)min((int64_t)want, q.end - q.at);
  *first = q.at;
  q.at += got;
  return got;
}

__device__ __forceinline__ int lanes_below(uint64_t m, int lane) { return __popcll(m & ((1ull << lane) - 1ull)); }

template <typename V>
__device__ __forceinline__ V from_lane(V v, int src) {
  return __builtin_bit_cast(V, __builtin_amdgcn_ds_bpermute(src << 2, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ int64_t from_lane64(int64_t v, int src) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(src << 2, (int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}

// Widest group of lanes that one atom is worth (log2).  An atom meets a real
// collision about every fifth candidate, so more than 16 lanes of a gridless
// flight would only work on events that never come; a fixed step has thousands.
template <bool kFixed>
constexpr int kWidest = kFixed ? 6 : 4;

// The flight.  A wavefront works in one of two ways.
//
// One lane per atom (wlog = 0): each pass makes one generator call per lane, the
// emission draw of a lane's next atom or the event draw of its current one.
//
// 2^wlog lanes per atom: lane i of a group takes the atom's event e + i on the
// assumption that none of the i events before it ends the flight or changes the
// velocity.  The draws are keyed by the event's number, so the lanes make them
// side by side; the positions follow one another in a short chain of sums; and
// the first lane whose event is real (a collision, a wall, the event limit)
// decides how many of the group's events count.  The atom's arithmetic is the
// same, so are its results.
//
// The flight is bound by the vector ALU while there are atoms for every lane,
// and by one atom's chain of events when there are not: about 4000 cycles an
// event, thousands of events for a slow atom at high pressure, a hundred thousand
// steps of a fixed-step one.  So a wavefront starts with as many lanes per atom
// as the number of atoms leaves free, and when no atoms are left it moves its
// remaining ones together and widens the groups.  Measured, one lane per atom
// throughout -> this: 1e6 atoms at 5 Pa (4.4e8 events) 30.3 -> 9.3 ms, 1e5
// fixed-step M1 atoms (2.2e8 steps) 170 -> 8 ms, 1e7 at 0.5 Pa (4.3e7 events)
// 2.87 -> 1.22 ms (there the one tally call and generator call per pass, the
// lane-wise sums and the float constants count).
template <bool kFixed, int kCols>
__global__ __launch_bounds__(kBlock, 6) void k_tp_flight(TpConst T, TpTally* tal, uint64_t* e_hist, uint64_t* th_hist,
                                                         uint64_t* tof_hist, TpTrace tr, int64_t* prof) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ TpShared<kCols> sh;
  const int nx1 = T.n_xbins + 1, tid = threadIdx.x, lane = tid & 63;
  unsigned long long* sP = reinterpret_cast<unsigned long long*>(smem);   // [4][n_xbins + 1]
  TpLds<kCols> S;
  S.pt = sP;
  S.dt = sP + nx1;
  S.px = sP + 2 * nx1;
  S.dd = sP + 3 * nx1;
  S.e = reinterpret_cast<uint32_t*>(sP + (T.n_xbins ? 4 * nx1 : 0));
  S.th = S.e + T.n_ebins;
  S.tof = S.th + kTpThetaBins;
  S.sh = &sh;
  for (int i = tid; i < T.n_ebins + kTpThetaBins + T.n_tbins; i += kBlock) S.e[i] = 0;
  if (T.n_xbins)
    for (int i = tid; i < 4 * nx1; i += kBlock) sP[i] = 0ull;
  if (lane < kCols) sh.sum[tid >> 6][lane] = 0ull;
  if (tid == 0) sh.n_tgt = sh.n_unf = sh.over = 0;
  __syncthreads();

  unsigned long long* next = reinterpret_cast<unsigned long long*>(&tal->next);
  const int64_t wave = (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(tid >> 6);
  Queue q;
  q.at = min(wave * T.run, T.n_atoms);     // every wavefront's first run is its own
  q.end = min(q.at + T.run, T.n_atoms);
  q.dry = false;
  int wlog = T.wlog;
  Atom a;
  int64_t k = 0;
  uint32_t n_over = 0, n_coll = 0;
  bool alive = false;
  float bound = 0.0f;

  if (wlog == 0) {
    bool fresh = true;
    while (true) {
      const uint64_t idle = __ballot(!alive);
      if (idle && !q.dry) {
        int64_t first;
        const int got = take(T, q, next, __popcll(idle), lane, &first);
        const int r = lanes_below(idle, lane);
        if (!alive && r < got) {
          k = first + r;
          alive = fresh = true;
        }
      }
      const uint64_t live = __ballot(alive);
      if (q.dry && __popcll(live) <= (T.widest ? 32 : 0) && !__ballot(alive && fresh)) break;
      if (alive) {
        const Uniforms8<float> U = draw_atom(T, k, fresh ? 0ull : (uint64_t)a.e,
                                             fresh ? rng_tag(SP_AL, PU_TP_SRC) : rng_tag(SP_AL, PU_TP_EVT));
        if (fresh) {
          emit(T, U, a);
          if (kFixed) bound = ratio_bound(T, a);
          fresh = false;
        } else {
          const float tau = kFixed ? T.f.dt : -fast_ln(U[0]) * T.f.inv_nu;
          const float xn = fmaf(a.vx, tau, a.x);
          const bool out = T.mode == 0 && !(xn >= 0.0f && xn < T.f.L);
          int wall = out ? (xn >= T.f.L ? 1 : 0) : -1;
          const float xe = out ? (wall ? T.f.L : 0.0f) : xn;
          if (T.n_xbins) track_tally(T, S, a.x, xe, a.vx);
          float tof = 0.0f;
          if (out) {
            tof = a.t + (wall ? T.f.L - a.x : -a.x) / a.vx;
          } else {
            a.x = T.mode == 0 ? xn : wrapf(xn, T.f.L, T.f.inv_L);
            // a fixed step's clock is its step count (no FP32 accumulation over many steps)
            if (!kFixed) a.t += tau;
            if (!kFixed || U[5] < bound) {
              EventDraw D;
              draw_partner(T, U, D);
              const Partner p = meet<kFixed>(T, D, a);
              n_over += p.ratio > 1.0f;
              if (D.u5 < p.ratio) {
                ++n_coll;
                scatter(T, p, D, a);
                if (kFixed) bound = ratio_bound(T, a);
              }
            }
            ++a.e;
            if ((int64_t)a.e >= T.e_max) wall = 2;
          }
          if (wall >= 0) {
            if (kFixed) {
              const float t = (float)((double)a.e * T.dt);
              tof = wall == 2 ? t : t + (wall ? T.f.L - a.x : -a.x) / a.vx;
            } else if (wall == 2) {
              tof = a.t;
            }
            finish(T, S, tr, k, a, wall, tof, n_coll, lane);
            n_coll = 0;
            alive = false;
          }
        }
      }
    }
  }

  // 2^wlog lanes per atom; every variable of the atom is the same in its lanes.
  // A gridless atom with 16 lanes (a row) keeps a row of drawn events and walks
  // through it (in the box its place does not matter and is not wrapped), pos the next one, stop by stop; the flights it made on the way
  // (xa -> xb at va, one per lane) are tallied together when the row is used up.
  EventDraw D = {};
  int pos = 16;
  bool flown = false;
  float xa = 0.0f, xb = 0.0f, va = 0.0f;
  while (true) {
    const int W = 1 << wlog, i = lane & (W - 1), base = lane - i;
    uint64_t leaders = 1;                                  // lanes 0, W, 2 W, ...
    for (int s = W; s < 64; s <<= 1) leaders |= leaders << s;
    const uint64_t idle = __ballot(!alive) & leaders;
    if (idle && !q.dry) {
      int64_t first;
      const int got = take(T, q, next, __popcll(idle), lane, &first);
      const int r = lanes_below(idle, base);
      if (!alive && r < got) {
        k = first + r;
        emit(T, draw_atom(T, k, 0, rng_tag(SP_AL, PU_TP_SRC)), a);
        if (kFixed) bound = ratio_bound(T, a);
        n_coll = 0;
        alive = true;
        pos = 16;
      }
    }
    const uint64_t live = __ballot(alive) & leaders;
    const int n = __popcll(live);
    if (n == 0) {
      if (q.dry) break;
      continue;
    }
    if (q.dry && wlog < T.widest && 2 * n * W <= 64) {
      // no atoms are left to take: move the groups together and widen them
      int to = wlog + 1;
      while (to < T.widest && (n << (to + 1)) <= 64) ++to;
      const bool lead = alive && i == 0;
      // leaders send their lane to the lane of their rank (at most 31), others to lane 63
      const int of = __builtin_amdgcn_ds_permute((lead ? lanes_below(live, lane) : 63) << 2, lane);
      const int src = from_lane(of, lane >> to);
      a.x = from_lane(a.x, src);
      a.vx = from_lane(a.vx, src);
      a.vy = from_lane(a.vy, src);
      a.vz = from_lane(a.vz, src);
      a.t = from_lane(a.t, src);
      a.e = from_lane(a.e, src);
      n_coll = from_lane(n_coll, src);
      bound = from_lane(bound, src);
      k = from_lane64(k, src);
      alive = (lane >> to) < n;
      wlog = to;
      continue;
    }
    if (!kFixed && wlog == 4) {
      if (__ballot(alive && pos >= 16)) {
        // a row of 16 draws: everything of these events that the atom's state does not enter
        if (flown && T.n_xbins) track_tally(T, S, xa, xb, va);
        flown = false;
        if (alive) {
          const Uniforms8<float> U = draw_atom(T, k, (uint64_t)(a.e + (uint32_t)i), rng_tag(SP_AL, PU_TP_EVT));
          D = draw_event(T, U);
          pos = 0;
        }
      }
      if (alive) {
        const uint32_t e = a.e + (uint32_t)(i - pos);      // this lane's event, from lane pos on
        const float tj = i >= pos ? D.tau : 0.0f;
        float x = a.x, t = a.t;
        row_chain(a.vx, tj, i, x, t);
        const float xn = fmaf(a.vx, D.tau, x);
        const bool open = i >= pos, out = T.mode == 0 && !(xn >= 0.0f && xn < T.f.L);
        const Partner p = meet<false>(T, D, a);
        const bool hit = !out && D.u5 < p.ratio;
        const bool last = !out && (uint64_t)e + 1 >= (uint64_t)T.e_max;
        const uint64_t stops = __ballot(open && (out || hit || last)) >> base & 0xFFFFull;
        const int first = stops ? (int)__builtin_ctzll(stops) : 15;
        int wall = out ? (xn >= T.f.L ? 1 : 0) : -1;
        if (open && i <= first) {
          n_over += p.ratio > 1.0f && !out;
          xa = x;
          xb = out ? (wall ? T.f.L : 0.0f) : xn;
          va = a.vx;
          flown = true;
        }
        Atom b = a;
        if (i == first) {
          float tof = 0.0f;
          b.e = e;
          if (out) {
            tof = t + (wall ? T.f.L - x : -x) / a.vx;
          } else {
            b.x = xn;
            b.t = t + D.tau;
            if (hit) scatter(T, p, D, b);
            b.e = e + 1;
            if (last) {
              wall = 2;
              tof = b.t;
            }
          }
          if (wall >= 0) finish(T, S, tr, k, b, wall, tof, n_coll + hit, lane);
        }
        const int src = base + first;
        a.x = from_lane(b.x, src);
        a.t = from_lane(b.t, src);
        a.e += (uint32_t)(first - pos) + 1u;
        const uint64_t hits = __ballot(hit && i == first);
        if (hits) {
          a.vx = from_lane(b.vx, src);
          a.vy = from_lane(b.vy, src);
          a.vz = from_lane(b.vz, src);
          n_coll += (uint32_t)(hits >> src & 1ull);
        }
        alive = !(__ballot(wall >= 0 && i == first) >> src & 1ull);
        pos = alive ? first + 1 : 16;
      }
    } else if (alive) {
      const uint32_t e = a.e + (uint32_t)i;                // this lane's event
      const Uniforms8<float> U = draw_atom(T, k, (uint64_t)e, rng_tag(SP_AL, PU_TP_EVT));
      const float tau = kFixed ? T.f.dt : -fast_ln(U[0]) * T.f.inv_nu;
      // where and when the lane's event starts: after the i flights before it
      float x = a.x, t = a.t;
      if (kFixed) {
        // every lane walks the same chain and keeps its own point of it
        float y = a.x;
#pragma unroll 8
        for (int j = 1; j < W; ++j) {
          y = fmaf(a.vx, tau, y);
          if (T.mode != 0) y = wrapf(y, T.f.L, T.f.inv_L);
          x = i == j ? y : x;
        }
      } else {
        for (int j = 1; j < W; ++j) {
          const float xs = fmaf(a.vx, tau, x);
          const float xw = T.mode == 0 ? xs : wrapf(xs, T.f.L, T.f.inv_L);
          // the lane before this one ends its flight here (row_shr:1)
          const float px = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(
              (int)__float_as_uint(a.x), (int)__float_as_uint(xw), 0x111, 0xf, 0xf, false));
          const float pt = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(
              (int)__float_as_uint(a.t), (int)__float_as_uint(t + tau), 0x111, 0xf, 0xf, false));
          x = i ? px : a.x;
          t = i ? pt : a.t;
        }
      }
      const float xn = fmaf(a.vx, tau, x);
      const bool out = T.mode == 0 && !(xn >= 0.0f && xn < T.f.L);
      bool hit = false, over = false;
      Partner p = {};
      EventDraw E = {};
      if (!kFixed || U[5] < bound) {
        draw_partner(T, U, E);
        p = meet<kFixed>(T, E, a);
        over = p.ratio > 1.0f;
        hit = !out && E.u5 < p.ratio;
      }
      const bool last = !out && (uint64_t)e + 1 >= (uint64_t)T.e_max;
      // the group's first lane with a real event; the events after it do not happen
      const uint64_t stops = __ballot(out || hit || last) >> base;
      const int first = min(stops ? (int)__builtin_ctzll(stops) : 64, W - 1);
      int wall = out ? (xn >= T.f.L ? 1 : 0) : -1;
      if (i <= first) {
        n_over += over && !out;
        if (T.n_xbins) track_tally(T, S, x, out ? (wall ? T.f.L : 0.0f) : xn, a.vx);
      }
      Atom b = a;
      if (i == first) {
        float tof = 0.0f;
        b.e = e;
        if (out) {
          tof = (kFixed ? (float)((double)e * T.dt) : t) + (wall ? T.f.L - x : -x) / a.vx;
        } else {
          b.x = T.mode == 0 ? xn : wrapf(xn, T.f.L, T.f.inv_L);
          b.t = t + tau;
          if (hit) scatter(T, p, E, b);
          b.e = e + 1;
          if (last) {
            wall = 2;
            tof = kFixed ? (float)((double)b.e * T.dt) : b.t;
          }
        }
        if (wall >= 0) finish(T, S, tr, k, b, wall, tof, n_coll + hit, lane);
      }
      const int src = base + first;
      a.x = from_lane(b.x, src);
      if (!kFixed) a.t = from_lane(b.t, src);
      a.e += (uint32_t)first + 1u;
      const uint64_t hits = __ballot(hit && i == first);
      if (hits) {
        a.vx = from_lane(b.vx, src);
        a.vy = from_lane(b.vy, src);
        a.vz = from_lane(b.vz, src);
        n_coll += (uint32_t)(hits >> src & 1ull);
        if (kFixed) bound = ratio_bound(T, a);
      }
      alive = !(__ballot(wall >= 0 && i == first) >> src & 1ull);
    }
  }

  if (flown && T.n_xbins) track_tally(T, S, xa, xb, va);

  if (n_over) atomicAdd(&sh.over, n_over);
  __syncthreads();
  for (int i = tid; i < T.n_ebins; i += kBlock)
    if (S.e[i]) atomicAdd((unsigned long long*)&e_hist[i], (unsigned long long)S.e[i]);
  for (int i = tid; i < kTpThetaBins; i += kBlock)
    if (S.th[i]) atomicAdd((unsigned long long*)&th_hist[i], (unsigned long long)S.th[i]);
  for (int i = tid; i < T.n_tbins; i += kBlock)
    if (S.tof[i]) atomicAdd((unsigned long long*)&tof_hist[i], (unsigned long long)S.tof[i]);
  if (T.n_xbins && prof)
    for (int i = tid; i < 4 * nx1; i += kBlock)
      if (sP[i]) atomicAdd((unsigned long long*)&prof[i], sP[i]);
  // one sum per wavefront
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned long long v = lane < kCols ? sh.sum[w][lane] : 0ull;
  for (int off = 32; off; off >>= 1) v += __shfl_xor(v, off, 64);
  if (lane == 0 && v) atomicAdd((unsigned long long*)&tal->sum[w], v);
  // every atom at the substrate has an angle.  (The workgroups of a short flight end
  // together and their atomics on the tallies take turns: one more each costs 10007
  // atoms at 0.5 Pa 4 us of 140.)
  if (w == 0) {
    uint32_t n_sub = 0;
    for (int i = lane; i < kTpThetaBins; i += 64) n_sub += S.th[i];
    for (int off = 32; off; off >>= 1) n_sub += __shfl_xor(n_sub, off, 64);
    if (lane == 0 && n_sub) atomicAdd((unsigned long long*)&tal->n_sub, (unsigned long long)n_sub);
  }
  if (tid == 0) {
    if (sh.n_tgt) atomicAdd((unsigned long long*)&tal->n_tgt, (unsigned long long)sh.n_tgt);
    if (sh.n_unf) atomicAdd((unsigned long long*)&tal->n_unf, (unsigned long long)sh.n_unf);
    if (sh.over) atomicAdd((unsigned long long*)&tal->overflow, (unsigned long long)sh.over);
  }
}

// Density and mean x-velocity profiles of the test atoms from the track-length
// tallies (Sec. IV.B, last paragraph: time-weighted densities without a grid):
// cell i holds the partial-cell sums plus the running sum of the full-cell
// differences, time in 2^-40 s and displacement in 2^-24 cells.  With S the
// source flux (m^-2 s^-1) carried by n_atoms atoms, an atom spending t in a
// cell of width h adds S / n_atoms * t / h to its density; the mean x-velocity
// is the displacement over the time (0 in a cell no atom entered).  One
// workgroup; out = [4][nx] doubles: time (s), displacement (m), density
// (m^-3), mean v_x (m/s).
__global__ __launch_bounds__(kBlock) void k_tp_profiles(const int64_t* prof, int nx, double h, double per_atom,
                                                        double* out) {
  __shared__ int64_t s_w[2][kBlock / 64];
  const int nx1 = nx + 1, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int per = (nx + kBlock - 1) / kBlock;
  const int b = tid * per, e = min(b + per, nx);
  int64_t lt = 0, lx = 0;
  for (int i = b; i < e; ++i) {
    lt += prof[nx1 + i];
    lx += prof[3 * nx1 + i];
  }
  // exclusive block scans of the two difference arrays (integer: exact in any order)
  int64_t st = lt, sx = lx;
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t a = __shfl_up(st, off, 64), c = __shfl_up(sx, off, 64);
    if (lane >= off) {
      st += a;
      sx += c;
    }
  }
  if (lane == 63) {
    s_w[0][w] = st;
    s_w[1][w] = sx;
  }
  __syncthreads();
  int64_t rt = st - lt, rx = sx - lx;
  for (int k = 0; k < w; ++k) {
    rt += s_w[0][k];
    rx += s_w[1][k];
  }
  for (int i = b; i < e; ++i) {
    rt += prof[nx1 + i];
    rx += prof[3 * nx1 + i];
    const double t = (double)(prof[i] + rt) / 1099511627776.0;
    const double x = (double)(prof[2 * nx1 + i] + rx) / 16777216.0 * h;
    out[i] = t;
    out[nx + i] = x;
    out[2 * nx + i] = per_atom * t / h;
    out[3 * nx + i] = t > 0.0 ? x / t : 0.0;
  }
}

hipError_t launch_tp_profiles(const int64_t* prof, int nx, double h, double per_atom, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_tp_profiles, dim3(1), dim3(kBlock), 0, st, prof, nx, h, per_atom, out);
  return hipGetLastError();
}

// Zero n 64-bit words (a kernel rather than a memset node, so that a captured
// call replays correctly).
__global__ __launch_bounds__(kBlock) void k_zero_u64(uint64_t* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) p[i] = 0;
}

hipError_t launch_zero_u64(void* p, size_t bytes, hipStream_t st) {
  const int64_t n = (int64_t)(bytes / 8);
  if (n == 0) return hipSuccess;
  const int64_t want = (n + kBlock - 1) / kBlock;
  const int grid = (int)(want < 1024 ? want : 1024);
  hipLaunchKernelGGL(k_zero_u64, dim3(grid), dim3(kBlock), 0, st, reinterpret_cast<uint64_t*>(p), n);
  return hipGetLastError();
}

// Device scratch of the test-particle runs that cannot allocate (the tallies
// of pm_run_test_particles_static): one copy per GPU, held until the process
// ends.  Host code only ever uses the device address looked up below; the
// array's own name is a host-side stand-in.
static __device__ __align__(256) unsigned char scratch[kTpScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t tp_scratch(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

// Compute units of the current device.  Asked for once per device: the query costs
// a few microseconds, of the 140 of a short flight.
static int compute_units() {
  static std::atomic<int> known[kMaxDevices];
  int dev = 0, cus = 0;
  (void)hipGetDevice(&dev);
  const bool kept = dev >= 0 && dev < kMaxDevices;
  if (kept && (cus = known[dev].load(std::memory_order_relaxed)) > 0) return cus;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) return 1;
  if (kept) known[dev].store(cus, std::memory_order_relaxed);
  return cus;
}

// Lanes per atom and atoms per run of the flight.  Four wavefronts per SIMD keep
// the vector ALU busy and leave fewer atoms in flight when the queue runs dry
// than the six to eight that fit (1e6 atoms at 5 Pa: 9.3 ms, 10.3 with six, 9.8
// with two; 1e7 at 0.5 Pa 1.27 against 1.26 and 1.55).  An atom starts with more
// lanes than one as long as its launch stays within as many wavefronts (a fixed
// step, whose lanes all count, twice as many: 1e5 atoms 7.9 ms against 9.3), but with
// one lane if it meets less than one event on its way (1e4 atoms at 0.1 Pa 120 -> 72
// us), and no more lanes than leave each eight events up to the event limit: more
// workgroups have more tallies to add (10 steps of 10007 atoms 141 us with 64 lanes an
// atom, 60 with one; 60 steps of 50021 in the periodic box 161 us with 16, 130 with
// four).  A fixed step at which many tests succeed has little to look ahead for: its
// lanes stay below 16 over the probability at the majorant (at 1.6, 10247 atoms 4.1 ms
// with 64 lanes and 2.6 with 8; at 0.16 5.5 with 64 and 6.1 with 32), and of a flight of
// fewer than 64 steps stricter (35 steps of 53405 atoms at 0.6 172 us with four, 132
// with one; 6000 of them 101 and 117).  The same holds for
// a gridless flight in the box, whose atoms all end at the event limit and so leave
// nobody to wait for, and for one that a low limit ends: the more atoms, the fewer of
// their collisions pay for lanes (2000 events in the box, omega 0.99, 53k atoms 5.3 ms
// with four lanes, 2.3 with one; omega 0.55 1.5 and 2.2; 6000 atoms at 0.9 1.3 with 16 and
// 2.2).
hipError_t launch_tp_flight(TpConst T, TpTally* tally, uint64_t* e_hist, uint64_t* th_hist, uint64_t* tof_hist,
                            TpTrace trace, int64_t* prof, hipStream_t st) {
  const int64_t most = (int64_t)compute_units() * 4 * 4;
  const bool fixed = T.dt > 0.0;
  T.widest = fixed ? kWidest<true> : kWidest<false>;
  const bool brief = fixed && T.e_max < 64;
  while (T.widest > 1 && T.f.nu_dt * (float)(1 << T.widest) > (brief ? 2.0f : 16.0f)) --T.widest;
  T.wlog = 0;
  const bool alone = !fixed && (((T.mode != 0 || T.e_max < 1024) && (float)T.n_atoms * T.hit > 2.0f * (float)most) ||
                                (T.mode != 0 && T.e_max < 128 && T.hit > 0.6f));
  if (T.expect >= 1.0f && !alone)
    while (T.wlog < T.widest && T.n_atoms <= (brief ? 8 : fixed ? 128 : 64) * most >> (T.wlog + 1) &&
           (int64_t)8 << (T.wlog + 1) <= T.e_max)
      ++T.wlog;
  if (alone && T.mode != 0) T.widest = 0;
  const int64_t per_wave = 64 >> T.wlog;
  const int64_t waves = std::min((T.n_atoms + per_wave - 1) / per_wave, most);
  const int grid = (int)std::max<int64_t>(1, (waves + kBlock / 64 - 1) / (kBlock / 64));
  // eight runs per wavefront: the atomics on the queue stay rare and the runs of the
  // last ones short; two where the atoms end so soon that the atomics would take
  // turns (3e6 atoms without gas 480 -> 190 us, 1e6 at 0.5 Pa 390 -> 320; at 1 Pa, 16
  // events an atom, 640 either way; at 30 events 310 with eight and 340 with two)
  const int64_t runs = T.expect < 16.0f ? 2 : 8;
  T.run = std::max(per_wave, std::min<int64_t>(T.n_atoms / (waves * runs), 512));
  T.first_run = (int64_t)grid * (kBlock / 64) * T.run;
  const size_t lds = (size_t)(T.n_ebins + kTpThetaBins + T.n_tbins) * 4 +
                     (T.n_xbins ? (size_t)4 * (T.n_xbins + 1) * 8 : 0);
  auto fly = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), lds, st, T, tally, e_hist, th_hist, tof_hist, trace, prof);
  };
  // the lane-wise sums (2 KB) where they fit beside the histograms
  constexpr size_t kLdsPerGroup = 160 * 1024;
  if (lds + sizeof(TpShared<64>) <= kLdsPerGroup)
    fixed ? fly(k_tp_flight<true, 64>) : fly(k_tp_flight<false, 64>);
  else
    fixed ? fly(k_tp_flight<true, 1>) : fly(k_tp_flight<false, 1>);
  return hipGetLastError();
}

}  // namespace pm

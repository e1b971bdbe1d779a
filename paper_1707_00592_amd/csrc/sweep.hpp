// Direction-sweep stage kernel of the WENO-IS finite-volume operator.
//
// One launch handles one axis D of an RK stage (Sec. 3, dimension by
// dimension).  A workgroup owns a tile of TL cells along D by TW cells
// across it:
//   1. load U for the tile plus 3 ghost cells per side along D (boundary
//      conditions applied while loading), recover the primitive state in
//      FP64 (eq. (2)) and stage it in LDS, latching non-physical cells;
//   2. one lane per face: project the six stencil cells onto the
//      characteristic fields (eqs. (11)-(12)), reconstruct both face states
//      with WENO-IS (eqs. (19)-(28)), back-project (eq. (13)), apply the
//      MOOD cascade (Sec. 3.4) and evaluate HLLC (eqs. (14)-(18)); the
//      flux and u^HLLC go to LDS;
//   3. one lane per cell: the D-contribution to dU/dt, eqs. (5)-(6), added to
//      the partial sum of the previous axes, and either stored as a partial
//      sum, stored as dU/dt, or combined into the Runge-Kutta stage.
// Coalescing: along x the tile rows are contiguous; for y and z sweeps the
// tile is TW consecutive x cells wide.
#pragma once

#include "face.hpp"
#include "mlp.hpp"

namespace isw {

enum OutMode {
  OUT_PARTIAL = 0,  // R = (R +) r_D
  OUT_RHS = 1,      // dUdt = (R +) r_D
  OUT_RK1 = 2,      // Uout = U0 + dt L
  OUT_RK2 = 3,      // Uout = 3/4 U0 + 1/4 (Uin + dt L)
  OUT_RK3 = 4,      // Uout = 1/3 U0 + 2/3 (Uin + dt L)
  // the time step inside the first two stages (fused 2D stage only):
  OUT_RK1L = 5,     // Rout = L(Uin), and each workgroup's max wave speed of Uin
  OUT_RK2L = 6,     // as OUT_RK2 with the stage input U0 + dt R, R = L(U0) of OUT_RK1L
  // the time step inside the first sweep of a 3D stage:
  OUT_PARTIAL_S = 7 // as OUT_PARTIAL (x sweep), and each workgroup's max wave speed of Uin
};

enum { ST_OK = 0, ST_NONPHYSICAL = -4 };

struct StatsDev {  // layout of isweno_stats
  unsigned long long o3[3], o1[3], mlp_fallback[3];
  int status;
  int reserved;
};

struct SweepArgs {
  const double* Uin;   // stage input (stencil source), nc x N
  const double* R;     // partial sum of previous axes (when read)
  double* Rout;        // partial-sum / dUdt output
  const double* U0;    // U^n for the RK combine
  double* Uout;        // RK stage output
  const double* dt;    // device scalar
  StatsDev* stats;     // may be null
  int64_t n[3];
  double dx[3];
  int bc_lo, bc_hi;    // of axis D
  int bcl[3], bch[3];  // of every axis (fused multi-axis stage kernels)
  int weights, mood;
  double eps;
  const uint16_t* mlp; // packed bf16 network (learned weights only)
  float mlp_thr;
  unsigned long long* shortcut;  // 256 x 3 counters of shortcut field-sides, or null
  // OUT_RK1L, OUT_PARTIAL_S: one max wave speed per workgroup (the bits of
  // the double)
  unsigned long long* cflp;
};

// Sum of an int over the 64 lanes of a wave (every lane active).
__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// A value the compiler may not reason about (no instruction).
template <typename V>
__device__ __forceinline__ void opaque(V& v) {
  asm("" : "+v"(v));
}

// Boundary map of a ghost/interior position l, a few cells at most outside
// the line of n cells (-3..n+2): interior index and whether the normal
// velocity is mirrored.  A periodic position is brought back by adding lines
// (one, unless the line is shorter than the halo): the 64-bit remainders that
// stood here are about 150 instructions each in every tile at an end, and
// the compiler makes one of a plain loop again (opaque).
__device__ __forceinline__ int64_t bc_index(int64_t l, int64_t n, int bclo,
                                            int bchi, bool& flip) {
  flip = false;
  if (l < 0) {
    if (bclo == 1) {
      do {
        l += n;
        opaque(l);
      } while (l < 0);
      return l;
    }
    if (bclo == 2) {
      flip = true;
      return -l - 1;
    }
    return 0;
  }
  if (l >= n) {
    if (bchi == 1) {
      do {
        l -= n;
        opaque(l);
      } while (l >= n);
      return l;
    }
    if (bchi == 2) {
      flip = true;
      return 2 * n - 1 - l;
    }
    return n - 1;
  }
  return l;
}

// k s for 0 <= k < 2^24 and a stride 0 <= s < 2^56: one wide multiply-add
// and a 24-bit one.  The general 64-bit product has three multiplies at a
// quarter of the rate, and every staged cell and every output cell paid it.
__device__ __forceinline__ int64_t times_stride(int k, int64_t s, int64_t plus) {
  const uint64_t lo = (uint64_t)(uint32_t)k * (uint32_t)s + (uint64_t)plus;
  return (int64_t)(lo + ((uint64_t)__umul24((unsigned)k, (unsigned)((uint64_t)s >> 32)) << 32));
}

// FP64 quotients in the kernels: exact (IEEE) in the FP64 form, which
// reproduces the oracle bit for bit; in the float form, whose reconstruction
// and flux are float, x times the refined reciprocal of the divisor (within
// 2 ulp of the quotient for a normal divisor), a third of the instructions.
template <typename T>
__device__ __forceinline__ double div64(double x, double y) {
  if constexpr (sizeof(T) == 8) return x / y;
  else return x * recip(y).r;
}

// The same for many quotients by one divisor (the reciprocal formed once).
template <typename T>
struct Div64 {
  double y, r;
  __device__ __forceinline__ explicit Div64(double d) : y(d), r(0.0) {
    if constexpr (sizeof(T) == 4) r = recip(d).r;
  }
  __device__ __forceinline__ double operator()(double x) const {
    if constexpr (sizeof(T) == 8) return x / y;
    else return x * r;
  }
};

// The cell update's quotients by the cell size, N at a time, x[i] /= dx.
// FP64 form, the IEEE quotients' bits at a fraction of their instructions (10
// to 14 each, and a cell has 2 NC + 4 in 2D): a cell size that is a power of
// two divides by multiplying (one instruction, exact, over- and underflow
// included); otherwise divide() with one shared reciprocal, its residual taken
// with the other sign so that a zero keeps its own, where every numerator of
// the wave is zero or within [2^-900, 2^900] (two comparisons each, which the
// quotients repay: 80 instructions instead of 224 in 2D); else plainly.  The
// float form multiplies by the refined reciprocal, as Div64.
template <typename T>
struct CellSize {
  double dx, r;
  bool pow2, fast;
  __device__ __forceinline__ explicit CellSize(double d) : dx(d), r(recip(d).r) {
    if constexpr (sizeof(T) == 8) {
      const unsigned long long b = (unsigned long long)__double_as_longlong(d);
      const int e = (int)(b >> 52);  // d > 0
      fast = e > 1023 - 60 && e < 1023 + 60;
      pow2 = fast && (b & 0xfffffffffffffull) == 0;
      if (pow2) r = __longlong_as_double((long long)(2046 - e) << 52);
    }
  }
  template <int N>
  __device__ __forceinline__ void quotients(double* x) const {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int i = 0; i < N; i++) x[i] = x[i] * r;
    } else {
      if (pow2) {
#pragma unroll
        for (int i = 0; i < N; i++) x[i] = x[i] * r;
        return;
      }
      bool far = !fast;
#pragma unroll
      for (int i = 0; i < N; i++)
        far |= !(fabs(x[i]) <= 0x1p900) | ((fabs(x[i]) < 0x1p-900) & (x[i] != 0.0));
      if (__any(far)) {
#pragma unroll
        for (int i = 0; i < N; i++) x[i] = x[i] / dx;
        return;
      }
#pragma unroll
      for (int i = 0; i < N; i++) {
        const double q = x[i] * r, rem = __builtin_fma(dx, q, -x[i]);
        x[i] = __builtin_fma(-rem, r, q);
      }
    }
  }
};

// Primitive recovery of one cell, axis order (rho, u_x.., p, Gamma, Pi),
// eq. (2): p = (E - rho |u|^2 / 2 - Pi) / Gamma; the quotients as div64<T>.
template <int NDIM, typename T = double>
__device__ __forceinline__ void cons_prim(const double* u, double* q) {
  const double rho = u[0];
  const Div64<T> by_rho(rho);
  double vel[NDIM];
#pragma unroll
  for (int a = 0; a < NDIM; a++) vel[a] = by_rho(u[1 + a]);
  double ke = vel[0] * vel[0];
#pragma unroll
  for (int a = 1; a < NDIM; a++) ke = ke + vel[a] * vel[a];
  const double E = u[1 + NDIM];
  const double G = u[2 + NDIM];
  const double P = u[3 + NDIM];
  q[0] = rho;
#pragma unroll
  for (int a = 0; a < NDIM; a++) q[1 + a] = vel[a];
  q[1 + NDIM] = div64<T>(E - 0.5 * rho * ke - P, G);
  q[2 + NDIM] = G;
  q[3 + NDIM] = P;
}

template <int NDIM, typename T = double>
__device__ __forceinline__ void cell_prim(const double* U, int64_t N,
                                          int64_t cell, double* q) {
  double u[4 + NDIM];
#pragma unroll
  for (int k = 0; k < 4 + NDIM; k++) u[k] = U[k * N + cell];
  cons_prim<NDIM, T>(u, q);
}

// Time step (the CFL condition of Secs. 5 and 6): one cell's
// sum_d (|u_d| + c)/dx_d from its axis-order primitives q, the quotients as
// div64<T>.
template <int NDIM, typename T = double>
__device__ __forceinline__ double cell_speed(const double* q, const double* dx) {
  const double cs = sqrt(sound2<double>(q[0], q[1 + NDIM], q[2 + NDIM], q[3 + NDIM]));
  double sp = div64<T>(fabs(q[1]) + cs, dx[0]);
#pragma unroll
  for (int a = 1; a < NDIM; a++) sp = sp + div64<T>(fabs(q[1 + a]) + cs, dx[a]);
  return sp;
}

// Each wave's max of m over its lanes, as the bits of the double (positive
// doubles order as their bits do; a NaN orders above every number), into
// red[wave]; the caller combines red after a barrier.
__device__ __forceinline__ void wave_max_bits(double m, unsigned long long* red) {
  unsigned long long b = (unsigned long long)__double_as_longlong(m);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long x = __shfl_xor(b, o);
    b = x > b ? x : b;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = b;
}

// Whether a cell (conservative values u, primitives q) is finite and
// admissible.
template <int NDIM>
__device__ __forceinline__ bool cell_ok_u(const double* u, const double* q) {
  bool fin = true;
#pragma unroll
  for (int k = 0; k < 4 + NDIM; k++) fin = fin && isfinite(u[k]);
  return fin && admissible(q[0], q[1 + NDIM], q[2 + NDIM], q[3 + NDIM]);
}

// Whether a cell's primitives lie where the FP64 stage kernels may use the
// unscaled divisions without a check per stencil (weno_f64_unit); every
// finite state of ordinary materials does.  A cell in range is finite in
// every component.
template <int NDIM>
__device__ __forceinline__ bool in_range(const double* q) {
  bool ok = (q[0] >= 0x1p-20) & (q[0] <= 0x1p30) & (fabs(q[1 + NDIM]) <= 0x1p40) &
            (q[2 + NDIM] >= 0x1p-10) & (q[2 + NDIM] <= 0x1p10) & (fabs(q[3 + NDIM]) <= 0x1p40);
#pragma unroll
  for (int a = 0; a < NDIM; a++) ok &= fabs(q[1 + a]) <= 0x1p24;
  return ok;
}

// The remaining condition of cell_ok_u for a cell in_range.
template <int NDIM>
__device__ __forceinline__ bool c2_positive(const double* q) {
  return (q[2 + NDIM] + 1.0) * q[1 + NDIM] + q[3 + NDIM] > 0.0;
}

// Uniform tiles.  Where every cell a tile reads holds one state (the fluid
// ahead of a front, the inside of a body), all its faces have one flux and
// one interface velocity, so each difference of eqs. (5)-(6) is x - x = +0
// and the axis' terms are the signed zeros below: the same bits without a
// face.  Cells are compared by their bits while they are staged (a mirrored
// ghost counts as different).  The state must be one whose flux is finite and
// whose reconstruction passes the positivity check whatever its rounding, in
// either arithmetic: steady_state bounds density and Gamma, keeps the stiff
// pressure (Gamma+1) p + Pi away from cancellation, the sound speed in
// [2^-10, 2^16] and the Mach number below 2^6 -- a rounding of 2^-24 then
// moves no reconstructed density or stiff pressure by more than 2^-12 of it.
// Such a tile costs its loads and stores (1024x512 at the start of a run, nine
// tenths of it uniform: 35 us a stage against 69); mixed states pay one
// comparison per staged cell, which shows only in float stages of some 10 us
// (kLookTiles).
// FP64 with epsilon = 0 is left to the faces: a constant stencil's weights
// are 0/0 there, and its tile's NaNs and fallbacks are the method's (the float
// form's flat stencils return their centre value whatever epsilon is).
template <typename T, int NDIM>
__device__ __forceinline__ bool steady_state(const double* q, double eps) {
  if (sizeof(T) == 8 && !(eps > 0.0)) return false;
  const double rho = q[0], p = q[1 + NDIM], G = q[2 + NDIM], P = q[3 + NDIM];
  const double stiff = (G + 1.0) * p + P, gr = G * rho;
  bool ok = rho >= 0x1p-12 && rho <= 0x1p12 && G >= 0x1p-6 && G <= 0x1p6 &&
            fabs(p) <= 0x1p36 && fabs(P) <= 0x1p36 &&
            stiff >= 0x1p-4 * ((G + 1.0) * fabs(p) + fabs(P)) && stiff >= 0x1p-20 * gr &&
            stiff <= 0x1p32 * gr;
#pragma unroll
  for (int a = 0; a < NDIM; a++) ok = ok && gr * q[1 + a] * q[1 + a] <= 0x1p12 * stiff;
  return ok;
}

// One axis' terms of eqs. (5)-(6) for a cell between two faces of the same
// flux and u*: -(x - x) / dx, and for Gamma and Pi + phi (x - x) / dx.
__device__ __forceinline__ double steady_term(bool material, double phi) {
  return material ? -0.0 + phi * 0.0 : -0.0;
}

// What a workgroup's waves found while staging a tile: bits TILE_*, gathered
// per lane in one register and per wave in one word (no word has to be
// cleared first, so nothing waits before the loads).  note() is called by
// every lane of a wave before the barrier that ends the staging, all() after
// it, with the same result in every lane.
enum { TILE_BAD = 1, TILE_FAR = 2, TILE_MIXED = 4, TILE_SKIP = 8, TILE_FLUIDS = 16 };
template <int NWAVES>
struct TileNotes {
  int word[NWAVES];
  __device__ __forceinline__ void note(int found) {
    int w = 0;
#pragma unroll
    for (int b = 1; b <= TILE_FLUIDS; b *= 2) w |= __any(found & b) ? b : 0;
    if ((threadIdx.x & 63) == 0) word[threadIdx.x >> 6] = w;
  }
  __device__ __forceinline__ int all() const {
    int w = 0;
#pragma unroll
    for (int k = 0; k < NWAVES; k++) w |= word[k];
    return __builtin_amdgcn_readfirstlane(w);
  }
};

// Whether an earlier evaluation latched a failure (sticky).  One lane of a
// workgroup asks, so that all its lanes agree; a plain load, issued beside
// the staging loads: a latch of the running launch may be seen or not.
__device__ __forceinline__ bool latched(const StatsDev* stats) {
  return stats && __hip_atomic_load(&stats->status, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_WORKGROUP) != ST_OK;
}

// How a lane's cell differs from the tile's reference, by bits: TILE_MIXED
// (where some cell of the wave differs in its density the others are not
// compared: a tile needs one difference) and, where asked for, TILE_FLUIDS.
template <int N>
__device__ __forceinline__ bool other_fluid(const double* u, const double* ref) {
  return (__double_as_longlong(u[N - 2]) != __double_as_longlong(ref[N - 2])) |
         (__double_as_longlong(u[N - 1]) != __double_as_longlong(ref[N - 1]));
}

template <int N, bool FLUIDS>
__device__ __forceinline__ int differs(const double* u, const double* ref, bool flip) {
  auto ne = [&](int c) { return __double_as_longlong(u[c]) != __double_as_longlong(ref[c]); };
  const bool f = FLUIDS && other_fluid<N>(u, ref);
  bool d = flip | f | ne(0);
  if (!__any(d)) {
#pragma unroll
    for (int c = 1; c < N; c++) d |= ne(c);
  }
  return (d ? TILE_MIXED : 0) | (f ? TILE_FLUIDS : 0);
}

// What a workgroup knows of its whole staged tile when it starts on the
// faces (the same for every lane).
struct TileState {
  bool fast;      // FP64: every staged cell in_range and epsilon too
  bool one_fluid;  // Gamma and Pi are those of the tile's first cell everywhere
};

// Face-order component k -> axis-order (LDS / conservative) component.
template <int NDIM, int D>
__device__ __host__ constexpr int axis_comp(int k) {
  return k == 0 ? 0
         : k == 1 ? 1 + D
         : (k < 1 + NDIM) ? 1 + ((k - 2) < D ? (k - 2) : (k - 1))
                          : k;
}

// Reconstruct the face states at the given order and back-project them to
// face-order primitives in FP64.  One characteristic field per iteration
// (the loop is kept rolled to bound register use; the branches on the field
// index are wave-uniform): project the six stencil cells with the field's
// row of L (eq. (11)), reconstruct the left state from positions 0..4
// (i-2..i+2) and the right state from the mirror image 5..1, and add the
// field's column of R (eq. (13)) into the face states in field order.
// sides: bit 0 = left, bit 1 = right.  S(c, j) reads LDS component c (axis
// order) at stencil position j.
// Learned weights for one field: the network on the 64 faces of the wave
// (two 32-sample tiles, all lanes take part), its weights applied to the
// candidates of eq. (20) as in eq. (19); below the confidence threshold, or
// for a side whose value leaves the range of the two cells next to the
// face, the eq. (28) weights are used instead (each counted as a fallback).
template <typename T>
__device__ __forceinline__ void mlp_field(const T* w, MlpRun& mr, T eps, T& rl, T& rr) {
  // Flat on both sides (spread below 1e-30, as the plain float form tests
  // it): every candidate is the centre value, so both the learned weights
  // and their fallback give it exactly.  A wave whose every lane is flat
  // skips the network (which needs the whole wave).
  const T sl = fmaxf(fmaxf(fmaxf(fabsf(w[0] - w[2]), fabsf(w[1] - w[2])), fabsf(w[3] - w[2])),
                     fabsf(w[4] - w[2]));
  const T sr = fmaxf(fmaxf(fmaxf(fabsf(w[5] - w[3]), fabsf(w[4] - w[3])), fabsf(w[2] - w[3])),
                     fabsf(w[1] - w[3]));
  if (__all(!(sl > T(1e-30)) && !(sr > T(1e-30)))) {
    rl = w[2];
    rr = w[3];
    return;
  }
  float x[8], z[9];
  mlp_features<T>(w, mr.f6, mr.f7, x);
  mlp_logits_wave(x, *mr.R, *mr.B, z);
  const float conf = 1.0f / (1.0f + __expf(-z[8]));
  if (!(conf >= mr.thr)) {
    int nf = 0;
    rl = weno<T>(w[0], w[1], w[2], w[3], w[4], W_MODIFIED, eps, false, nf);
    rr = weno<T>(w[5], w[4], w[3], w[2], w[1], W_MODIFIED, eps, false, nf);
    mr.fallbacks++;
    return;
  }
#pragma unroll
  for (int side = 0; side < 2; side++) {
    const float* zs = z + 4 * side;
    const float m = fmaxf(fmaxf(zs[0], zs[1]), fmaxf(zs[2], zs[3]));
    float e[4], sum = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      e[k] = __expf(zs[k] - m);
      sum += e[k];
    }
    const float A = float(side ? w[5] : w[0]), B = float(side ? w[4] : w[1]),
                C = float(side ? w[3] : w[2]), D_ = float(side ? w[2] : w[3]),
                E = float(side ? w[1] : w[4]);
    // candidates of eq. (20) written as the centre value plus differences,
    // so that a constant stencil is reproduced exactly; weighted and
    // normalised by one reciprocal
    const float d1 = 0.5f * (D_ - C), d2 = 0.5f * (C - B);
    const float d3 = (5.0f / 6.0f) * (D_ - C) - (1.0f / 6.0f) * (E - C);
    const float d4 = (1.0f / 3.0f) * (A - C) - (7.0f / 6.0f) * (B - C);
    const float q =
        C + (e[0] * d1 + e[1] * d2 + e[2] * d3 + e[3] * d4) * __builtin_amdgcn_rcpf(sum);
    // A face value outside the range of the two cells next to the face (a
    // confident but wrong prediction: an overshoot, or a material property
    // mixed into a pure fluid) takes the eq. (28) weights instead.
    if (q >= fminf(C, D_) && q <= fmaxf(C, D_)) {
      if (side) rr = T(q); else rl = T(q);
    } else {
      int nf = 0;
      if (side)
        rr = weno<T>(w[5], w[4], w[3], w[2], w[1], W_MODIFIED, eps, false, nf);
      else
        rl = weno<T>(w[0], w[1], w[2], w[3], w[4], W_MODIFIED, eps, false, nf);
      mr.fallbacks++;
    }
  }
}

template <typename T, int NDIM, int D, bool CUT = false, class S>
__device__ __forceinline__ void recon(const S& st, int sides, bool order3, int weights, T eps,
                                      T a, T b, double bd, double gd, double* ql, double* qr,
                                      int& nshort, MlpRun* mr = nullptr, bool one_fluid = false) {
  constexpr int NT = NDIM - 1, NC = 5 + NT;
  constexpr int CR = 0, CU = 1 + D, CP = 1 + NDIM, CG = 2 + NDIM, CPI = 3 + NDIM;
  // Fully unrolled over the fields (static register indices for the face
  // states, no loop-carried copies); the scheduling barrier keeps the
  // compiler from interleaving fields, which bounds register pressure.
#pragma unroll
  for (int m = 0; m < NC; m++) {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (sizeof(T) == 4) {
      // float form, one fluid in the whole tile: a stencil without spread
      // returns its centre value on both sides
      if ((m == 2 + NT || m == 3 + NT) && one_fluid) {
        const double r = double(st(m == 2 + NT ? CG : CPI, 2));
        if (m == 2 + NT) ql[3 + NT] = qr[3 + NT] = r;
        else ql[4 + NT] = qr[4 + NT] = r;
        nshort += 2;
        continue;
      }
    }
    // row of L: 0 = acoustic (sign sa), 1 = entropy, 2 = copy of component cx
    int kind = 2, cx = CG;
    T sa = a;
    if (m == 0) {
      kind = 0;
      sa = -a;
    } else if (m == NC - 1) {
      kind = 0;
    } else if (m == 1) {
      kind = 1;
    } else if (m < 2 + NT) {
      cx = 1 + ((m - 2) < D ? (m - 2) : (m - 1));
    } else if (m == 3 + NT) {
      cx = CPI;
    }
    T w[6];
#pragma unroll
    for (int j = 0; j < 6; j++) {
      if (kind == 0) {
        w[j] = sa * T(st(CU, j)) + T(0.5) * T(st(CP, j));
      } else if (kind == 1) {
        w[j] = T(st(CR, j)) - b * T(st(CP, j));
      } else {
        w[j] = T(st(cx, j));
      }
    }
    T rlm = T(0), rrm = T(0);
    // the material fields (Gamma, Pi) keep the eq. (28) weights: their
    // reconstruction decides the mixture at an interface
    const bool learned = mr != nullptr && !order3 && m != 2 + NT && m != 3 + NT;
    if (learned) mlp_field<T>(w, *mr, eps, rlm, rrm);
    const int wk = weights == W_MLP ? W_MODIFIED : weights;
#pragma unroll
    for (int side = 0; side < 2; side++) {
      if (!(sides & (1 << side))) continue;
      __builtin_amdgcn_sched_barrier(0);
      double* q = side ? qr : ql;
      const double r =
          learned ? double(side ? rrm : rlm)
          : side ? double(weno_sel<T, CUT>(w[5], w[4], w[3], w[2], w[1], wk, eps, order3, nshort))
                 : double(weno_sel<T, CUT>(w[0], w[1], w[2], w[3], w[4], wk, eps, order3, nshort));
      if (m == 0) {
        q[0] = bd * r;
        q[1] = (-gd) * r;
        q[2 + NT] = r;
      } else if (m == 1) {
        q[0] = q[0] + r;
      } else if (m == NC - 1) {
        q[0] = q[0] + bd * r;
        q[1] = q[1] + gd * r;
        q[2 + NT] = q[2 + NT] + r;
      } else {
#pragma unroll
        for (int t = 0; t < NT; t++)
          if (m == 2 + t) q[2 + t] = r;
        if (m == 2 + NT) q[3 + NT] = r;
        if (m == 3 + NT) q[4 + NT] = r;
      }
    }
  }
}

// The back-projection of field m's value r into a side's face-order state,
// eq. (13), in field order.
template <int NT>
__device__ __forceinline__ void back_project(int m, double r, double bd, double gd, double* q) {
  constexpr int NC = 5 + NT;
  if (m == 0) {
    q[0] = bd * r;
    q[1] = (-gd) * r;
    q[2 + NT] = r;
  } else if (m == 1) {
    q[0] = q[0] + r;
  } else if (m == NC - 1) {
    q[0] = q[0] + bd * r;
    q[1] = q[1] + gd * r;
    q[2 + NT] = q[2 + NT] + r;
  } else {
#pragma unroll
    for (int t = 0; t < NT; t++)
      if (m == 2 + t) q[2 + t] = r;
    if (m == 2 + NT) q[3 + NT] = r;
    if (m == 3 + NT) q[4 + NT] = r;
  }
}

// 5th-order FP64 face states of a face in range, fully unrolled over the
// fields as recon.  Away from interfaces (one_fluid, the same for the whole
// tile) Gamma and Pi need no stencil: two of the 5 + NT fields, whose tau5,
// candidates and twelve LDS reads were a tenth of a face in the general form.
template <int NDIM, int D, bool CUT, bool BASIC, class S>
__device__ __forceinline__ void recon_fast(const S& st, bool one_fluid, double eps, double a,
                                           double b, double bd, double gd, double* ql, double* qr,
                                           int& nshort) {
  constexpr int NT = NDIM - 1, NC = 5 + NT;
  constexpr int CR = 0, CU = 1 + D, CP = 1 + NDIM, CG = 2 + NDIM, CPI = 3 + NDIM;
#pragma unroll
  for (int m = 0; m < NC; m++) {
    __builtin_amdgcn_sched_barrier(0);
    if ((m == 2 + NT || m == 3 + NT) && one_fluid) {
      // tau5 = 0: the candidates' linear form on six equal values, the same
      // for both sides
      const double v = st(m == 2 + NT ? CG : CPI, 2);
      const double r = linear_unit<CUT>(cand_unit(v, v, v, v, v));
      back_project<NT>(m, r, bd, gd, ql);
      back_project<NT>(m, r, bd, gd, qr);
      nshort += 2;
      continue;
    }
    double w[6];
#pragma unroll
    for (int j = 0; j < 6; j++) {
      if (m == 0) w[j] = -a * st(CU, j) + 0.5 * st(CP, j);
      else if (m == NC - 1) w[j] = a * st(CU, j) + 0.5 * st(CP, j);
      else if (m == 1) w[j] = st(CR, j) - b * st(CP, j);
      else if (m < 2 + NT) w[j] = st(1 + ((m - 2) < D ? (m - 2) : (m - 1)), j);
      else w[j] = st(m == 2 + NT ? CG : CPI, j);
    }
#pragma unroll
    for (int side = 0; side < 2; side++) {
      __builtin_amdgcn_sched_barrier(0);
      const double v0 = side ? w[5] : w[0], v1 = side ? w[4] : w[1], v2 = side ? w[3] : w[2],
                   v3 = side ? w[2] : w[3], v4 = side ? w[1] : w[4];
      double r;
      if constexpr (CUT) r = weno_f64_cutoff_unit(v0, v1, v2, v3, v4, eps, nshort);
      else r = weno_f64_unit<BASIC>(v0, v1, v2, v3, v4, eps, nshort);
      back_project<NT>(m, r, bd, gd, side ? qr : ql);
    }
  }
}

// L_{i+1/2}: L of eq. (11) at the mean of the two primitive states, as the
// parameters a = rho c / 2, b = 1/c^2 and, in FP64, bd = b, gd = 1/(rho c).
template <typename T, int NDIM, class S>
__device__ __forceinline__ void face_params(const S& st, T& a, T& b, double& bd, double& gd) {
  constexpr int CR = 0, CP = 1 + NDIM, CG = 2 + NDIM, CPI = 3 + NDIM;
  const double rb = 0.5 * (st(CR, 2) + st(CR, 3));
  const double pb = 0.5 * (st(CP, 2) + st(CP, 3));
  const double Gb = 0.5 * (st(CG, 2) + st(CG, 3));
  const double Pb = 0.5 * (st(CPI, 2) + st(CPI, 3));
  const T c2 = sound2<T>(T(rb), T(pb), T(Gb), T(Pb));
  const T c = sqrt(c2);
  a = T(rb) * c / T(2);
  b = qdiv<T>(T(1), c2);
  bd = double(b);
  gd = div64<T>(1.0, double(T(rb) * c));
  if (sizeof(T) == 8) {
    bd = 1.0 / double(c2);
  }
}

// The weights a stage kernel evaluates: the cut-off form in the kernels
// instantiated for it, else eq. (21) or eq. (28) as asked (those kernels
// never see W_CUTOFF, and the compiler knows it).
template <bool CUT>
__device__ __forceinline__ int kernel_weights(int w) {
  return CUT ? W_CUTOFF : (w == W_BASIC ? W_BASIC : W_MODIFIED);
}

// The fail bits of a face's two states (bit 0 left, bit 1 right), Sec. 3.4.
template <int NT>
__device__ __forceinline__ int mood_fail(const double* ql, const double* qr) {
  return (admissible(ql[0], ql[2 + NT], ql[3 + NT], ql[4 + NT]) ? 0 : 1) |
         (admissible(qr[0], qr[2 + NT], qr[3 + NT], qr[4 + NT]) ? 0 : 2);
}

// The end of the cascade: a failing side whose 3rd-order state fails too
// takes the first-order state of eq. (32) (the cell's own primitive state,
// since R L q_i = q_i).
template <int NDIM, int D, class S>
__device__ __forceinline__ void first_order(const S& st, int fail, double* ql, double* qr, int& n3,
                                            int& n1) {
  constexpr int NT = NDIM - 1, NC = 5 + NT;
#pragma unroll
  for (int side = 0; side < 2; side++) {
    if (!(fail & (1 << side))) continue;
    double* q = side ? qr : ql;
    // counted without a branch: a counter picked by a branch ends up
    // in private (scratch) memory on every face
    const int ok = admissible(q[0], q[2 + NT], q[3 + NT], q[4 + NT]) ? 1 : 0;
    if (!ok) {
      const int j = side ? 3 : 2;
#pragma unroll
      for (int k = 0; k < NC; k++) q[k] = st(axis_comp<NDIM, D>(k), j);
    }
    n3 += ok;
    n1 += 1 - ok;
  }
}

template <typename T, int NT>
__device__ __forceinline__ void states_flux(const double* ql, const double* qr, double* F,
                                            double& us) {
  constexpr int NC = 5 + NT;
  T tl[NC], tr[NC], tF[NC], tus;
#pragma unroll
  for (int k = 0; k < NC; k++) {
    tl[k] = T(ql[k]);
    tr[k] = T(qr[k]);
  }
  hllc<T, NT>(tl, tr, tF, tus);
#pragma unroll
  for (int k = 0; k < NC; k++) F[k] = double(tF[k]);
  us = double(tus);
}

// The cascade of an FP64 face in range: the sides that failed (bit 0 left, bit
// 1 right) in 3rd order.  Rolled over fields and sides, which keeps the states
// and the loop in the registers of the 5th-order path: unrolled behind a branch
// there it cost states that never reach it 5-8%, and with the whole face
// evaluated again apart from it (in 5th order as well) the slowest wave of a
// small batch took three face evaluations a stage: 60 tubes of 100 to 600
// cells 61 us a step, 51 so; 1024x512, a tenth of the cells random, 204 us a
// stage, 166 so.
template <int NDIM, int D, bool CUT, class S>
__device__ __forceinline__ void recon_cascade(const S& st, int sides, int weights, double eps,
                                              double a, double b, double bd, double gd,
                                              double* ql, double* qr) {
  constexpr int NT = NDIM - 1, NC = 5 + NT;
  constexpr int CR = 0, CU = 1 + D, CP = 1 + NDIM;
#pragma unroll 1
  for (int m = 0; m < NC; m++) {
    // the field's row of L: x times component c plus y times p, or a copy of c
    const bool copy = m >= 2 && m < NC - 1;
    const int c = m == 1 ? CR : !copy ? CU : m < 2 + NT ? 1 + ((m - 2) < D ? m - 2 : m - 1) : m + 1;
    const double x = m == 0 ? -a : m == 1 ? 1.0 : a, y = m == 1 ? -b : 0.5;
#pragma unroll 1
    for (int side = 0; side < 2; side++) {
      if (!(sides & (1 << side))) continue;
      double w[5];
      // (opaque: or all six pressures are loaded before the loops and kept)
      int cc = c, cp = CP;
      asm("" : "+s"(cc), "+s"(cp));
#pragma unroll
      for (int j = 0; j < 5; j++) {
        const int at = side ? 5 - j : j;
        w[j] = st(cc, at);
        if (!copy) w[j] = x * w[j] + y * st(cp, at);
      }
      __builtin_amdgcn_sched_barrier(0);
      const double r = weno_f64_unit3<CUT>(w[0], w[1], w[2], w[3], w[4], weights, eps);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < NC; k++)
        if (k == m) {
          if (side) back_project<NT>(k, r, bd, gd, qr);
          else back_project<NT>(k, r, bd, gd, ql);
        }
    }
  }
}

// The states of an FP64 face of a tile in range, with the cascade (mood).
// Returns true when the sound speed lies outside the range of the unscaled
// divisions; the face is then evaluated by face_general, which shares no value
// with this path.
template <int NDIM, int D, bool CUT, class S>
__device__ __forceinline__ bool common_states(const S& st, const TileState& tile, int weights,
                                              int mood, double eps, double* ql, double* qr,
                                              int& n3, int& n1, int& nshort) {
  constexpr int NT = NDIM - 1;
  double a, b, bd, gd;
  face_params<double, NDIM>(st, a, b, bd, gd);
  nshort = 0;
  // b = 1/c^2 of the mean state: c^2 >= kFaceC2Min
  const bool far = !(b > 0.0 && b <= 1.0 / kFaceC2Min);
  if (!CUT && weights == W_BASIC)
    recon_fast<NDIM, D, CUT, true>(st, tile.one_fluid, eps, a, b, bd, gd, ql, qr, nshort);
  else
    recon_fast<NDIM, D, CUT, false>(st, tile.one_fluid, eps, a, b, bd, gd, ql, qr, nshort);
  n3 = 0;
  n1 = 0;
  if (mood) {
    const int fail = far ? 0 : mood_fail<NT>(ql, qr);
    if (__builtin_expect(__any(fail), 0)) {
      recon_cascade<NDIM, D, CUT>(st, fail, weights, eps, a, b, bd, gd, ql, qr);
      first_order<NDIM, D>(st, fail, ql, qr, n3, n1);
    }
  }
  return far;
}

// An FP64 face in general: any range, with the cascade.
template <int NDIM, int D, bool CUT, class S>
__device__ __forceinline__ void face_general(const S& st, int weights, int mood, double eps,
                                             double* F, double& us, int& n3, int& n1,
                                             int& nshort) {
  constexpr int NT = NDIM - 1, NC = 5 + NT;
  double a, b, bd, gd, ql[NC], qr[NC];
  face_params<double, NDIM>(st, a, b, bd, gd);
  nshort = 0;
  recon<double, NDIM, D, CUT>(st, 3, false, weights, eps, a, b, bd, gd, ql, qr, nshort);
  n3 = 0;
  n1 = 0;
  if (mood) {
    const int fail = mood_fail<NT>(ql, qr);
    if (fail) {
      int n = 0;
      recon<double, NDIM, D, CUT>(st, fail, true, weights, eps, a, b, bd, gd, ql, qr, n);
      first_order<NDIM, D>(st, fail, ql, qr, n3, n1);
    }
  }
  states_flux<double, NT>(ql, qr, F, us);
}

// Full face: average state, eigen-parameters, both reconstructions, MOOD
// cascade, HLLC.  F (face order) and us are written; n3/n1 report the
// orders used (per side), nshort the field-sides of the first pass whose
// reconstruction took its shortcut.  FP64: a wave with a face out of range
// evaluates all its faces by face_general (the same bits).
template <typename T, int NDIM, int D, bool CUT = false, class S>
__device__ __forceinline__ void face_flux(const S& st, const TileState& tile, int weights,
                                          int mood, double eps, double* F, double& us,
                                          int& n3, int& n1, int& nshort,
                                          MlpRun* mr = nullptr) {
  constexpr int NT = NDIM - 1, NC = 5 + NT;
  if constexpr (sizeof(T) == 8) {
    bool other = true;
    if (tile.fast) {
      double ql[5 + NT], qr[5 + NT];
      other = common_states<NDIM, D, CUT>(st, tile, weights, mood, eps, ql, qr, n3, n1, nshort);
      states_flux<double, NT>(ql, qr, F, us);
    }
    if (__builtin_expect(__any(other), 0))
      face_general<NDIM, D, CUT>(st, weights, mood, eps, F, us, n3, n1, nshort);
  } else {
  T a, b;
  double bd, gd, ql[NC], qr[NC];
  face_params<T, NDIM>(st, a, b, bd, gd);
  if (mr) {
    constexpr int CG = 2 + NDIM, CPI = 3 + NDIM;
    const double Gb = 0.5 * (st(CG, 2) + st(CG, 3));
    const double Pb = 0.5 * (st(CPI, 2) + st(CPI, 3));
    mlp_material(Gb, Pb, mr->f6, mr->f7);
  }
  nshort = 0;
  recon<T, NDIM, D, CUT>(st, 3, false, weights, T(eps), a, b, bd, gd, ql, qr, nshort, mr,
                         tile.one_fluid);
  n3 = 0;
  n1 = 0;
  if (mood) {
    // Sec. 3.4: redo a failing side without the 3-point stencils, then fall
    // back to the first-order state
    int fail = mood_fail<NT>(ql, qr);
    if (mr && fail) {
      // learned weights: a failing side is first redone with the plain
      // 5th-order WENO-IS weights of eq. (28) (counted as a fallback of the
      // network); the cascade below then starts from that state
      int nfl = 0;
      recon<T, NDIM, D>(st, fail, false, W_MODIFIED, T(eps), a, b, bd, gd, ql, qr, nfl);
      mr->fallbacks += (fail & 1) + (fail >> 1);
      fail = mood_fail<NT>(ql, qr);
    }
    if (fail) {
      int nf3 = 0;
      recon<T, NDIM, D, CUT>(st, fail, true, weights, T(eps), a, b, bd, gd, ql, qr, nf3);
      first_order<NDIM, D>(st, fail, ql, qr, n3, n1);
    }
  }
  states_flux<T, NT>(ql, qr, F, us);
  }
}

// The same face in two passes, for a kernel that gathers the faces the
// MOOD cascade needs and redoes them by full waves.  First pass: the
// 5th-order states and their check; a face with a failing side returns its
// fail bits (non-zero) and no flux.  Second pass (face_flux_redo, on the
// gathered faces): the whole face again with the cascade -- the flux that
// face_flux gives, bit for bit.  FP64: a face out of range is gathered as
// well, and the second pass is face_general.
template <typename T, int NDIM, int D, bool CUT = false, class S>
__device__ __forceinline__ int face_flux_first(const S& st, const TileState& tile, int weights,
                                               double eps, double* F, double& us, int& nshort) {
  constexpr int NT = NDIM - 1, NC = 5 + NT;
  nshort = 0;
  if constexpr (sizeof(T) == 8) {
    if (!tile.fast) return 1;
    double ql[5 + NT], qr[5 + NT];
    int n3, n1;
    if (common_states<NDIM, D, CUT>(st, tile, weights, 0, eps, ql, qr, n3, n1, nshort)) return 1;
    if (const int fail = mood_fail<NT>(ql, qr)) return fail;
    states_flux<double, NT>(ql, qr, F, us);
    return 0;
  } else {
    T a, b;
    double bd, gd, ql[NC], qr[NC];
    face_params<T, NDIM>(st, a, b, bd, gd);
    recon<T, NDIM, D, CUT>(st, 3, false, weights, T(eps), a, b, bd, gd, ql, qr, nshort, nullptr,
                           tile.one_fluid);
    const int fail = mood_fail<NT>(ql, qr);
    if (!fail) states_flux<T, NT>(ql, qr, F, us);
    return fail;
  }
}

// fail: face_flux_first's; nshort counts the 5th-order states formed again
// (the first pass's count goes for the faces it settled).
template <typename T, int NDIM, int D, bool CUT = false, class S>
__device__ __forceinline__ void face_flux_redo(const S& st, int fail, int weights, double eps,
                                               double* F, double& us, int& n3, int& n1,
                                               int& nshort) {
  constexpr int NT = NDIM - 1, NC = 5 + NT;
  if constexpr (sizeof(T) == 8) {
    face_general<NDIM, D, CUT>(st, weights, 1, eps, F, us, n3, n1, nshort);
  } else {
    T a, b;
    double bd, gd, ql[NC], qr[NC];
    face_params<T, NDIM>(st, a, b, bd, gd);
    int nf3 = 0;
    nshort = 0;
    recon<T, NDIM, D, CUT>(st, 3, false, weights, T(eps), a, b, bd, gd, ql, qr, nshort);
    recon<T, NDIM, D, CUT>(st, fail, true, weights, T(eps), a, b, bd, gd, ql, qr, nf3);
    n3 = 0;
    n1 = 0;
    first_order<NDIM, D>(st, fail, ql, qr, n3, n1);
    states_flux<T, NT>(ql, qr, F, us);
  }
}

}  // namespace isw

// A whole Runge-Kutta step of a short 1D line in one launch.
//
// A line of a few hundred cells is one workgroup's work, and as four launches
// (time step, three stages) it is nothing but their latencies: 39 us a step at
// 200 cells, each stage 10 us of launch, loads, one face's dependent chain and
// stores.  Here one workgroup keeps the line: a lane per cell holds U^n and
// the stage values in registers, primitives and face fluxes pass through LDS,
// the time step is a reduction inside the workgroup.  Same operations in the
// same order as the separate kernels (the oracle's bits in FP64).
#pragma once
#include <hip/hip_runtime.h>

#include "launch.hpp"
#include "sweep_kernels.hpp"

namespace isw {

struct Step1dArgs {
  double* U;    // U^n in, U^{n+1} out, 5 x n
  double* dt;
  StatsDev* stats;  // may be null
  int n;
  double dx;
  int bc_lo, bc_hi, weights, mood;
  double eps, cfl, dt_max;
  unsigned long long* shortcut;  // 256 x 3 counters of shortcut field-sides, or null
};

// A cell's (|u| + c) / dx of eq. (2)'s primitives, as cfl_kernel forms it.
// The step's dt is isweno_cfl_dt's value in both forms, so the two products
// an add follows are rounded (opaque) also where the float form's kernels are
// compiled with contraction.
__device__ __forceinline__ double line_speed(const double* u, double dx) {
  const double rho = u[0], G = u[3], P = u[4], vel = u[1] / rho;
  double ke = 0.5 * rho * (vel * vel);
  opaque(ke);
  const double p = (u[2] - ke - P) / G;
  double gp = (G + 1.0) * p;
  opaque(gp);
  return (fabs(vel) + sqrt((gp + P) / (G * rho))) / dx;
}

template <typename T, int NTHR, bool CUT>
__global__ __launch_bounds__(NTHR) void step1d_kernel(Step1dArgs g) {
  constexpr int NC = 5, NP = NTHR + 6, NW = NTHR / 64;
  __shared__ T sq[NC * NP];           // primitives, position = cell + 3
  __shared__ T sf[(NC + 1) * NTHR];   // fluxes and u* of face tid (left of cell tid)
  __shared__ TileNotes<NW> s_notes;
  __shared__ unsigned long long s_red[NW];
  const int tid = threadIdx.x, n = g.n;
  const bool cell = tid < n, face = tid <= n;
  const bool skip = tid == 0 && latched(g.stats);
  // the interior cell behind each of the six ghost positions
  int src[6];
  bool flip[6];
#pragma unroll
  for (int k = 0; k < 6; k++)
    src[k] = (int)bc_index(k < 3 ? k - 3 : n + k - 3, n, g.bc_lo, g.bc_hi, flip[k]);

  double u0[NC], u[NC];  // U^n and the stage input
#pragma unroll
  for (int c = 0; c < NC; c++) u[c] = u0[c] = cell ? g.U[(int64_t)c * n + tid] : 1.0;
  double h;
  if (g.cfl > 0.0) {
    double m = 0.0;
    if (cell) {
      const double sp = line_speed(u0, g.dx);
      m = (sp > m || sp != sp) ? sp : m;
    }
    wave_max_bits(m, s_red);
    __syncthreads();
    unsigned long long b = s_red[0];
#pragma unroll
    for (int w = 1; w < NW; w++) b = s_red[w] > b ? s_red[w] : b;
    h = g.cfl / __longlong_as_double((long long)b);
    if (g.dt_max > 0.0 && h > g.dt_max) h = g.dt_max;
    if (tid == 0) *g.dt = h;
  } else {
    h = *g.dt;
  }
  const CellSize<T> dx(g.dx);
#pragma unroll 1
  for (int stage = 0; stage < 3; stage++) {
    double q[NC];
    cons_prim<1, T>(u, q);
    const bool inr = sizeof(T) == 8 && in_range<1>(q);
    int found = skip ? TILE_SKIP : 0;
    if (cell) {
      if constexpr (sizeof(T) == 8) found |= inr ? 0 : TILE_FAR;
      found |= (inr ? c2_positive<1>(q) : cell_ok_u<1>(u, q)) ? 0 : TILE_BAD;
#pragma unroll
      for (int c = 0; c < NC; c++) sq[c * NP + tid + 3] = T(q[c]);
#pragma unroll
      for (int k = 0; k < 6; k++) {
        if (src[k] != tid) continue;
        const int p = k < 3 ? k : n + k;
#pragma unroll
        for (int c = 0; c < NC; c++) sq[c * NP + p] = T(c == 1 && flip[k] ? -q[c] : q[c]);
      }
    }
    s_notes.note(found);
    __syncthreads();
    const int notes = s_notes.all();
    if (notes & TILE_SKIP) return;
    if (g.stats && tid == 0 && (notes & TILE_BAD)) atomicExch(&g.stats->status, ST_NONPHYSICAL);
    double F[NC], us = 0.0;
    int nf = 0;
    if (face) {
      LdsStencil<T> st;
      st.base = &sq[tid];
      st.cstride = NP;
      st.pstride = 1;
      int n3, n1;
      const TileState tile{!(notes & TILE_FAR) && eps_in_range(g.eps), false};
      face_flux<T, 1, 0, CUT>(st, tile, kernel_weights<CUT>(g.weights), g.mood, g.eps, F, us, n3,
                              n1, nf);
      if (g.stats) {
        if (n3) atomicAdd(&g.stats->o3[0], (unsigned long long)n3);
        if (n1) atomicAdd(&g.stats->o1[0], (unsigned long long)n1);
      }
#pragma unroll
      for (int k = 0; k < NC; k++) sf[k * NTHR + tid] = T(F[k]);
      sf[NC * NTHR + tid] = T(us);
    }
    if (g.shortcut) {  // measurement only
      const int ws = wave_sum(nf);
      if ((tid & 63) == 0 && ws) atomicAdd(&g.shortcut[(tid >> 6) * 3], (unsigned long long)ws);
    }
    __syncthreads();
    // a failure latched by this stage ends the step before the next one, as
    // the next launch would have found it
    if (g.stats && (notes & TILE_BAD) && stage < 2) return;
    if (!cell) continue;
    const double usr = double(sf[NC * NTHR + tid + 1]);
    double x[NC + 2];
#pragma unroll
    for (int k = 0; k < NC; k++) {
      x[k] = -(double(sf[k * NTHR + tid + 1]) - F[k]);
      if (k >= 3) x[k + 2] = double(T(q[k])) * (usr - us);
    }
    dx.template quotients<NC + 2>(x);
#pragma unroll
    for (int k = 0; k < NC; k++) {
      const double r = k >= 3 ? x[k] + x[k + 2] : x[k];
      if (stage == 0) u[k] = u0[k] + h * r;
      else if (stage == 1) u[k] = 0.75 * u0[k] + 0.25 * (u[k] + h * r);
      else g.U[(int64_t)k * n + tid] = (1.0 / 3.0) * u0[k] + (2.0 / 3.0) * (u[k] + h * r);
    }
  }
}

template <typename T, bool CUT>
static hipError_t launch_step1d_t(const Step1dArgs& a, hipStream_t s, LaunchEvents ev) {
  // n + 1 faces, one per lane
  if (a.n < 1 || a.n > kStep1dMax) return hipErrorInvalidValue;
  auto go = [&](auto kern, int threads) {
    if (ev.start)
      hipExtLaunchKernelGGL(kern, dim3(1), dim3(threads), 0, s, ev.start, ev.stop, 0, a);
    else
      hipLaunchKernelGGL(kern, dim3(1), dim3(threads), 0, s, a);
  };
  if (a.n < 256) go(step1d_kernel<T, 256, CUT>, 256);
  else go(step1d_kernel<T, 512, CUT>, 512);
  return hipGetLastError();
}

}  // namespace isw

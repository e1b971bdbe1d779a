// Kernels of the batched 1D path (isweno_batch_*): the stage kernel and its
// launch templates, instantiated by batch.hip (FP64) and batch_f32.hip (the
// float form, built with multiply-add contraction).
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <new>
#include <tuple>
#include <vector>

#include "isweno.h"
#include "sweep.hpp"

namespace isw {

struct BatchArgs {
  const double* Uin;
  const double* U0;
  double* Uout;
  const double* dt;        // per problem
  const double* dx;        // per problem
  const int64_t* offsets;  // nprob + 1
  const int64_t* tstart;   // first cell of each tile
  const int32_t* tprob;    // problem of each tile
  int64_t ntiles, total;
  const int32_t* active;   // per problem: advanced in this step (set by the dt kernel)
  int32_t* pstatus;        // per problem: sticky status
  StatsDev* stats;
  int bc_lo, bc_hi, weights, mood;
  double eps;
  double* U;               // whole steps: the state, advanced in place
  const double* halo;      // whole steps: kHalo cells each side of every tile
  int64_t tile0;           // whole steps: the launch's first tile
};

// Cells a whole step of a tile reads beyond each of its ends: three stages of
// three ghost cells.
constexpr int kHalo = 9;
// Cells of a tile of a whole step by nthr lanes: the first stage evaluates the
// tile's faces and those of 6 cells beyond each end.
constexpr int step_tile(int nthr) { return nthr - 1 - 2 * 6; }

template <typename E>
struct Lds1 {
  const E* base;
  int cstride;
  __device__ __forceinline__ E operator()(int c, int j) const {
    return base[c * cstride + j];
  }
};

template <typename T, int TL, int MODE, bool CUT>
__global__ __launch_bounds__(TL + 1, sizeof(T) == 4 ? 6 : 1) void batch_stage_kernel(BatchArgs g) {
  constexpr int NC = 5, NP = TL + 6, NF = TL + 1, NTHR = TL + 1;
  // FP64 primitives and the face values, both in the arithmetic's type (the
  // float form reconstructs from float values and its fluxes are float)
  __shared__ T sq[NC * NP];
  __shared__ T sf[(NC + 1) * NF];
  __shared__ TileNotes<NTHR / 64> s_notes;
  const int tid = threadIdx.x;
  int failed = 0;  // a cell of any of this workgroup's tiles was non-physical
  const int64_t total = g.total;
  int my3 = 0, my1 = 0;
  for (int64_t t = blockIdx.x; t < g.ntiles; t += gridDim.x) {
    const int prob = g.tprob[t];
    // problems that were non-physical when this step began are frozen (the
    // flag is written before the step's stages and not during them, so the
    // branch is the same for every lane and every stage of the step)
    if (!g.active[prob]) continue;
    const int64_t lo = g.offsets[prob], n = g.offsets[prob + 1] - lo;
    const int64_t l0 = g.tstart[t] - lo;
    const int len = (int)((n - l0) < TL ? (n - l0) : TL);
    int found = 0;
    double ref[NC];  // the tile's first cell
#pragma unroll
    for (int c = 0; c < NC; c++) ref[c] = g.Uin[c * total + lo + l0];
    // FP64: raised instruction priority while the tile is staged (its loads
    // go out ahead of the other workgroups' arithmetic), normal afterwards
    if constexpr (sizeof(T) == 8) __builtin_amdgcn_s_setprio(1);
    for (int p = tid; p < NP; p += NTHR) {
      const int64_t l = l0 + p - 3;
      if (l >= n + 3) continue;
      bool flip;
      const int64_t li = bc_index(l, n, g.bc_lo, g.bc_hi, flip);
      double u[NC], q[NC];
#pragma unroll
      for (int c = 0; c < NC; c++) u[c] = g.Uin[c * total + lo + li];
      found |= differs<NC, sizeof(T) == 8>(u, ref, flip);
      cons_prim<1, T>(u, q);
      const bool inr = sizeof(T) == 8 && in_range<1>(q);
      if constexpr (sizeof(T) == 8) found |= inr ? 0 : TILE_FAR;
      if (p >= 3 && p < 3 + len) found |= (inr ? c2_positive<1>(q) : cell_ok_u<1>(u, q)) ? 0 : TILE_BAD;
      if (flip) q[1] = -q[1];
#pragma unroll
      for (int c = 0; c < NC; c++) sq[c * NP + p] = T(q[c]);
    }
    if (found & TILE_BAD) atomicExch(&g.pstatus[prob], (int32_t)ST_NONPHYSICAL);
    s_notes.note(found);
    __syncthreads();
    if constexpr (sizeof(T) == 8) __builtin_amdgcn_s_setprio(0);
    const int notes = s_notes.all();
    failed |= notes & TILE_BAD;
    // (one_fluid not in the float form: its registers cost more than it saves)
    const TileState tile{!(notes & TILE_FAR) && eps_in_range(g.eps),
                         sizeof(T) == 8 && !(notes & TILE_FLUIDS)};
    const double h = g.dt[prob];
    // the output step of a cell from its L; uin(c) is the stage input there.
    // Everything is loaded before anything is stored (the compiler may not move
    // a load over the store before it).
    auto put = [&](int64_t cell, const double* L, auto uin) {
      double u0[NC], ui[NC];
#pragma unroll
      for (int c = 0; c < NC; c++) {
        u0[c] = g.U0[c * total + cell];
        if (MODE != OUT_RK1) ui[c] = uin(c);
      }
#pragma unroll
      for (int c = 0; c < NC; c++) {
        const int64_t o = c * total + cell;
        if (MODE == OUT_RK1) g.Uout[o] = u0[c] + h * L[c];
        else if (MODE == OUT_RK2) g.Uout[o] = 0.75 * u0[c] + 0.25 * (ui[c] + h * L[c]);
        else g.Uout[o] = (1.0 / 3.0) * u0[c] + (2.0 / 3.0) * (ui[c] + h * L[c]);
      }
    };
    // a uniform tile (steady_state): every face has the same flux
    if (!(notes & TILE_MIXED)) {
      double q[NC];
      cons_prim<1, T>(ref, q);
      if (steady_state<T, 1>(q, g.eps)) {
        double L[NC];
#pragma unroll
        for (int c = 0; c < NC; c++) L[c] = steady_term(c >= 3, q[c]);
        for (int j = tid; j < len; j += NTHR)
          put(lo + l0 + j, L, [&](int c) { return ref[c]; });
        __syncthreads();  // the notes are reused by the next tile
        continue;
      }
    }
    for (int j = tid; j <= len; j += NTHR) {
      Lds1<T> st;
      st.base = &sq[j];
      st.cstride = NP;
      double F[NC], us;
      int n3, n1, nf;
      face_flux<T, 1, 0, CUT>(st, tile, kernel_weights<CUT>(g.weights), g.mood, g.eps, F, us, n3, n1,
                              nf);
      if (j < len || l0 + j == n) {  // count each face of a problem once
        my3 += n3;
        my1 += n1;
      }
#pragma unroll
      for (int k = 0; k < NC; k++) sf[k * NF + j] = T(F[k]);
      sf[NC * NF + j] = T(us);
    }
    __syncthreads();
    const CellSize<T> dx(g.dx[prob]);
    for (int j = tid; j < len; j += NTHR) {
      const int64_t cell = lo + l0 + j;
      double x[NC + 2];
#pragma unroll
      for (int k = 0; k < NC; k++) {
        x[k] = -(double(sf[k * NF + j + 1]) - double(sf[k * NF + j]));
        if (k >= 3)
          x[k + 2] = double(sq[k * NP + j + 3]) *
                     (double(sf[NC * NF + j + 1]) - double(sf[NC * NF + j]));
      }
      dx.template quotients<NC + 2>(x);
#pragma unroll
      for (int k = 3; k < NC; k++) x[k] = x[k] + x[k + 2];
      put(cell, x, [&](int c) { return g.Uin[c * total + cell]; });
    }
    __syncthreads();  // LDS is reused by the next tile
  }
  if (g.stats) {
    if (my3) atomicAdd(&g.stats->o3[0], (unsigned long long)my3);
    if (my1) atomicAdd(&g.stats->o1[0], (unsigned long long)my1);
    if (tid == 0 && failed) atomicExch(&g.stats->status, (int)ST_NONPHYSICAL);
  }
}

// A whole Runge-Kutta step of every tile in one launch, in place.
//
// As one launch per stage the state is read and written three times and each
// stage pays its own launch, staging and last round of workgroups.  Here a
// workgroup carries its tile through the three stages in registers and LDS,
// evaluating the 6 (3) cells beyond each end in the first (second) stage
// itself: 5% more faces at 256 lanes, 11% at 128, 25% at 64, and a quarter of
// the bytes (4096 tubes of 128 to 4096 cells with the present faces: 1024 us a
// step against 1320 in three stage launches; 300 tubes of 50 to 1500 cells 85
// against 105, float 48 against 57).  The U^n of the kHalo cells beyond its
// ends come from copies made at the start of the step, so that neighbours may
// already have written theirs.  Ends of a
// problem: ghosts of a stage are written by the lanes that hold the cells they
// mirror (not for periodic ends, whose neighbours are another tile's).
// Lane tid holds cell l0 - 6 + tid and the face to its left; staged position p
// is cell l0 - kHalo + p.
template <typename T, int NTHR, bool CUT>
__global__ __launch_bounds__(NTHR, 4) void batch_step_kernel(BatchArgs g) {
  constexpr int NC = 5, TC = step_tile(NTHR), NP = TC + 2 * kHalo;
  __shared__ T sq[NC * NP];
  __shared__ T sf[(NC + 1) * NTHR];
  // the lanes' stage inputs: held in registers across the face they spilled
  // (172 bytes a lane in FP64)
  __shared__ double su[NC * NTHR];
  __shared__ TileNotes<NTHR / 64> s_notes[2];
  const int tid = threadIdx.x;
  const int64_t t = g.tile0 + blockIdx.x;
  const int prob = g.tprob[t];
  if (!g.active[prob]) return;  // non-physical when this step began (the same for every lane)
  const int64_t lo = g.offsets[prob], n = g.offsets[prob + 1] - lo;
  const int64_t l0 = g.tstart[t] - lo, total = g.total;
  const int len = (int)((n - l0) < TC ? (n - l0) : TC);
  const double h = g.dt[prob];
  // component c of U^n at cell l0 + r
  auto un = [&](int c, int r) {
    if (r >= 0 && r < len) return g.U[c * total + lo + l0 + r];
    const int k = r < 0 ? r + kHalo : kHalo + (r - len);
    return g.halo[(t * 2 * kHalo + k) * NC + c];
  };
  // the cells (relative to l0) behind the ghosts next to the problem's ends
  auto ghost = [&](int k, bool& flip) {
    const int64_t l = k < 3 ? k - 3 : n + k - 3;
    return (int)(bc_index(l, n, g.bc_lo, g.bc_hi, flip) - l0);
  };
  const bool first = l0 < kHalo, last = n - l0 - len < kHalo;  // an end of the problem in reach
  double ref[NC];  // the tile's first cell
#pragma unroll
  for (int c = 0; c < NC; c++) ref[c] = g.U[c * total + lo + l0];

  const int mine = tid - 6;  // the lane's cell, relative to l0
  const bool cell = l0 + mine >= 0 && l0 + mine < n && mine < len + 6;
  int found = 0;
  // stages cell r's primitives, and the ghosts that mirror it
  auto stage_cell = [&](int r, const double* q) {
#pragma unroll
    for (int c = 0; c < NC; c++) sq[c * NP + r + kHalo] = T(q[c]);
    if (!(first | last)) return;
#pragma unroll
    for (int k = 0; k < 6; k++) {
      bool flip;
      if (!(k < 3 ? first : last) || ghost(k, flip) != r) continue;
      if (flip) found |= TILE_MIXED;
      const int to = (int)((k < 3 ? k - 3 : n + k - 3) - l0) + kHalo;
      if (to >= NP) continue;  // beyond what any face of the tile reads
#pragma unroll
      for (int c = 0; c < NC; c++) sq[c * NP + to] = T(c == 1 && flip ? -q[c] : q[c]);
    }
  };
  // the outermost three cells each side: read by the first stage's faces only
  if (tid < 6) {
    const int r = tid < 3 ? tid - kHalo : len + 3 + tid;
    if (l0 + r >= 0 && l0 + r < n) {
      double v[NC], q[NC];
#pragma unroll
      for (int c = 0; c < NC; c++) v[c] = un(c, r);
      found |= differs<NC, sizeof(T) == 8>(v, ref, false);
      cons_prim<1, T>(v, q);
      if constexpr (sizeof(T) == 8) found |= in_range<1>(q) ? 0 : TILE_FAR;
      stage_cell(r, q);
    }
  }
  const CellSize<T> dx(g.dx[prob]);
  int my3 = 0, my1 = 0;
#pragma unroll 1
  for (int stage = 0; stage < 3; stage++) {
    const int m = 6 - 3 * stage;  // cells beyond each end in this stage
    if (cell && mine >= -m - 3 && mine < len + m + 3) {
      double u[NC], q[NC];
#pragma unroll
      for (int c = 0; c < NC; c++) {
        u[c] = stage == 0 ? un(c, mine) : su[c * NTHR + tid];
        if (stage == 0) su[c * NTHR + tid] = u[c];
      }
      cons_prim<1, T>(u, q);
      const bool inr = sizeof(T) == 8 && in_range<1>(q);
      // (a stage's rounding moves Gamma and Pi also within one fluid: looked at
      // in every stage)
      if (stage == 0) found |= differs<NC, sizeof(T) == 8>(u, ref, false);
      else if constexpr (sizeof(T) == 8) found |= other_fluid<NC>(u, ref) ? TILE_FLUIDS : 0;
      if constexpr (sizeof(T) == 8) found |= inr ? 0 : TILE_FAR;
      if (mine >= 0 && mine < len)
        found |= (inr ? c2_positive<1>(q) : cell_ok_u<1>(u, q)) ? 0 : TILE_BAD;
      stage_cell(mine, q);
    }
    if (found & TILE_BAD) atomicExch(&g.pstatus[prob], (int32_t)ST_NONPHYSICAL);
    s_notes[stage & 1].note(found);
    __syncthreads();
    const int notes = s_notes[stage & 1].all();
    if (g.stats && tid == 0 && (notes & TILE_BAD)) atomicExch(&g.stats->status, ST_NONPHYSICAL);
    if (stage == 0 && !(notes & TILE_MIXED) && h - h == 0.0) {
      // a uniform tile (steady_state): every face has the same flux in every
      // stage, and the stages' states stay uniform
      double qr[NC];
      cons_prim<1, T>(ref, qr);
      if (steady_state<T, 1>(qr, g.eps)) {
        if (mine >= 0 && mine < len) {
#pragma unroll
          for (int c = 0; c < NC; c++) {
            const double L = steady_term(c >= 3, qr[c]), u0 = ref[c];
            const double u1 = u0 + h * L;
            const double u2 = 0.75 * u0 + 0.25 * (u1 + h * L);
            g.U[c * total + lo + l0 + mine] = (1.0 / 3.0) * u0 + (2.0 / 3.0) * (u2 + h * L);
          }
        }
        return;
      }
    }
    // faces to the left of cells -m .. len + m
    double F[NC], us = 0.0;
    const bool face = mine >= -m && mine <= len + m && l0 + mine >= 0 && l0 + mine <= n;
    if (face) {
      Lds1<T> st;
      st.base = &sq[mine + kHalo - 3];
      st.cstride = NP;
      int n3, n1, nf;
      const TileState tile{!(notes & TILE_FAR) && eps_in_range(g.eps),
                           sizeof(T) == 8 && !(notes & TILE_FLUIDS)};
      face_flux<T, 1, 0, CUT>(st, tile, kernel_weights<CUT>(g.weights), g.mood, g.eps, F, us, n3,
                              n1, nf);
      // each face of a problem is counted once, by the tile after it
      if ((mine >= 0 && mine < len) || (mine == len && l0 + mine == n)) {
        my3 += n3;
        my1 += n1;
      }
#pragma unroll
      for (int k = 0; k < NC; k++) sf[k * NTHR + tid] = T(F[k]);
      sf[NC * NTHR + tid] = T(us);
    }
    __syncthreads();
    if (!cell || mine < -m || mine >= len + m) continue;
    const double usr = double(sf[NC * NTHR + tid + 1]);
    double x[NC + 2];
#pragma unroll
    for (int k = 0; k < NC; k++) {
      x[k] = -(double(sf[k * NTHR + tid + 1]) - F[k]);
      // (Gamma and Pi are their own primitives)
      if (k >= 3) x[k + 2] = double(T(su[k * NTHR + tid])) * (usr - us);
    }
    dx.template quotients<NC + 2>(x);
    // (U^n of every component before the first store, as the stage launches)
    double v0[NC];
#pragma unroll
    for (int k = 0; k < NC; k++) v0[k] = stage == 0 ? su[k * NTHR + tid] : un(k, mine);
#pragma unroll
    for (int k = 0; k < NC; k++) {
      const double u = su[k * NTHR + tid], u0 = v0[k];
      const double r = k >= 3 ? x[k] + x[k + 2] : x[k];
      if (stage == 0) su[k * NTHR + tid] = u0 + h * r;
      else if (stage == 1) su[k * NTHR + tid] = 0.75 * u0 + 0.25 * (u + h * r);
      else g.U[k * total + lo + l0 + mine] = (1.0 / 3.0) * u0 + (2.0 / 3.0) * (u + h * r);
    }
  }
  if (g.stats) {
    if (my3) atomicAdd(&g.stats->o3[0], (unsigned long long)my3);
    if (my1) atomicAdd(&g.stats->o1[0], (unsigned long long)my1);
  }
}

template <typename T, int TL, bool CUT>
static hipError_t launch_stage_c(const BatchArgs& a, int mode, int blocks, hipStream_t s) {
  if (mode == OUT_RK1)
    hipLaunchKernelGGL((batch_stage_kernel<T, TL, OUT_RK1, CUT>), dim3(blocks), dim3(TL + 1), 0,
                       s, a);
  else if (mode == OUT_RK2)
    hipLaunchKernelGGL((batch_stage_kernel<T, TL, OUT_RK2, CUT>), dim3(blocks), dim3(TL + 1), 0,
                       s, a);
  else
    hipLaunchKernelGGL((batch_stage_kernel<T, TL, OUT_RK3, CUT>), dim3(blocks), dim3(TL + 1), 0,
                       s, a);
  return hipGetLastError();
}

// the cut-off weights in kernels of their own (register allocation of the
// other forms unchanged)
template <typename T, int TL>
static hipError_t launch_stage_tl(const BatchArgs& a, int mode, int blocks, hipStream_t s) {
  return a.weights == W_CUTOFF ? launch_stage_c<T, TL, true>(a, mode, blocks, s)
                               : launch_stage_c<T, TL, false>(a, mode, blocks, s);
}

template <typename T>
static hipError_t launch_stage_t(int tl, const BatchArgs& a, int mode, int blocks,
                                 hipStream_t s) {
  // the tile list was cut for exactly this tile length (a kernel for a
  // shorter one would overrun its LDS on the list's longer tiles)
  if (blocks < 1) return hipErrorInvalidValue;
  switch (tl) {
    case 63: return launch_stage_tl<T, 63>(a, mode, blocks, s);
    case 127: return launch_stage_tl<T, 127>(a, mode, blocks, s);
    case 255: return launch_stage_tl<T, 255>(a, mode, blocks, s);
    default: return hipErrorInvalidValue;
  }
}

// Whole steps: nthr lanes per tile of step_tile(nthr) cells.
template <typename T, int NTHR>
static hipError_t launch_step_n(const BatchArgs& a, hipStream_t s) {
  if (a.ntiles < 1) return hipErrorInvalidValue;
  // a launch holds less than 2^32 lanes; tiles are independent (their
  // neighbours' cells are copies), so more of them are more launches
  constexpr int64_t kMost = 0xffffffffLL / NTHR;
  BatchArgs b = a;
  for (b.tile0 = 0; b.tile0 < a.ntiles; b.tile0 += kMost) {
    const int64_t left = a.ntiles - b.tile0;
    const dim3 grid((unsigned)(left < kMost ? left : kMost));
    if (a.weights == W_CUTOFF)
      hipLaunchKernelGGL((batch_step_kernel<T, NTHR, true>), grid, dim3(NTHR), 0, s, b);
    else
      hipLaunchKernelGGL((batch_step_kernel<T, NTHR, false>), grid, dim3(NTHR), 0, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
static hipError_t launch_step_t(int nthr, const BatchArgs& a, hipStream_t s) {
  // the tile list was cut for exactly step_tile(nthr) cells; a reflected or
  // copied ghost needs its cell within the tile's reach, a periodic one is
  // another tile's
  if (a.bc_lo == 1 || a.bc_hi == 1 || !a.halo || !a.U) return hipErrorInvalidValue;
  switch (nthr) {
    case 64: return launch_step_n<T, 64>(a, s);
    case 128: return launch_step_n<T, 128>(a, s);
    case 256: return launch_step_n<T, 256>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// The float form's instantiations (batch_f32.hip).
hipError_t launch_batch_step_f32(int nthr, const BatchArgs& a, hipStream_t s);
hipError_t launch_batch_stage_f32(int tl, const BatchArgs& a, int mode, int blocks, hipStream_t s);

}  // namespace isw

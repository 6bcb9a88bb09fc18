// Device side of the LGMRES restart cycle (Algorithm 2's Krylov solver): the
// Hessenberg column of each Arnoldi step, its Givens rotations, the residual
// estimate and the convergence predicate, and the least-squares solve at the
// end of the cycle all run in single-wave kernels on the solver's stream, so
// the host enqueues Arnoldi steps without waiting for them.  The host reads
// the small head of the state once per step, one step behind the GPU, to know
// when a cycle has ended; it never sits between two steps.
//
// Each Gram-Schmidt pass is two launches: the multi-dot (k_gram_schmidt) and
// one workgroup that reduces its partial sums and forms the Hessenberg column
// (k_gs_column).
// The column update is the classical Gram-Schmidt of the multi-dot: with
// h_i = <v_i, w> and ||w||^2 from one pass, ||w - V h||^2 = ||w||^2 - ||h||^2;
// when that difference falls below kReorthEta2 ||w||^2 (severe cancellation,
// the Daniel-Gragg-Kaufman-Stewart test) the column is left open, the cycle
// pauses (`reorth` set, `active` cleared) and the host enqueues a second
// Gram-Schmidt pass for that column before it resumes.  Cancellation is rare,
// so a step normally costs the multi-dot, the column and one update.
#include <cmath>

#include "internal.h"

namespace cheb {

namespace {

constexpr int kW = 64;

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__global__ __launch_bounds__(kW) void k_arnoldi_init(ArnoldiState* st, double tol, double stall) {
  if (threadIdx.x == 0) {
    st->tol = tol;
    st->stall = stall;
    st->bprev = HUGE_VAL;
    st->active = 0;
    st->jend = 0;
    st->reorth = 0;
    st->breakdown = 0;
    st->stagnated = 0;
    st->direct = 0;
  }
}

// start of a restart cycle: dots[0] = ||r||^2 of the true residual r
__global__ __launch_bounds__(kW) void k_arnoldi_begin(ArnoldiState* st, const double* dots) {
  if (threadIdx.x != 0) return;
  const double b2 = dots[0];
  const double beta = std::sqrt(b2 > 0.0 ? b2 : 0.0);
  st->beta = beta;
  st->inv_beta = beta > 0.0 ? 1.0 / beta : 0.0;
  st->g[0] = beta;
  st->jend = 0;
  st->reorth = 0;
  st->direct = 0;
  st->breakdown = 0;
  st->est = beta;
  st->stagnated = (st->stall > 0.0 && beta > st->stall * st->bprev) ? 1 : 0;
  st->active = (beta > st->tol && std::isfinite(beta) && !st->stagnated) ? 1 : 0;
  st->bprev = beta;
}

// double of lane i (uniform) of a wave
__device__ __forceinline__ double lane_of(double v, int i) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((int)b, i), hi = __builtin_amdgcn_readlane((int)(b >> 32), i);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// what the Hessenberg column reads of the state, fetched ahead of the column's
// sums: lane l holds the rotations (and, re-orthogonalising, the column) of rows
// l and l + 64
constexpr int kColRegs = (kMaxKrylovCols + kW - 1) / kW;
struct ColumnIn {
  ArnoldiHead hd;
  double cs[kColRegs], sn[kColRegs], h0[kColRegs], g;
};

__device__ __forceinline__ void column_fetch(const ArnoldiState* st, int j, int pass, int lane, ColumnIn& in) {
  in.hd = *static_cast<const ArnoldiHead*>(st);
  in.g = st->g[j];
#pragma unroll
  for (int q = 0; q < kColRegs; ++q) {
    const int i = lane + q * kW, ic = i <= j ? i : j;
    in.cs[q] = st->cs[ic];
    in.sn[q] = st->sn[ic];
    in.h0[q] = pass == 0 ? 0.0 : st->H[ic * kMaxKrylovCols + j];
  }
}

// column j of the Hessenberg matrix from the multi-dot dots[0..j+1], in one wave
// (pass 0: first Gram-Schmidt pass; pass 1: the re-orthogonalisation pass,
// whose coefficients add to the column), then -- unless pass 0 asks for
// re-orthogonalisation -- the Givens rotations, the residual estimate
// |g[j+1]| and the cycle's continuation flag.  The caller has checked that the
// pass runs (pass 0: the cycle is active; pass 1: re-orthogonalisation asked).
// The rotations run over registers, every lane carrying the running entry: a
// chain of two multiply-adds a row (through LDS, one lane, each row also waited
// for its reads).
__device__ __forceinline__ void arnoldi_column_wave(ArnoldiState* st, const double* dots, int j, int pass, int lane,
                                                    ColumnIn& in) {
  const int ld = kMaxKrylovCols;
  ArnoldiHead& hd = in.hd;
  double ss = 0.0, col[kColRegs];
#pragma unroll
  for (int q = 0; q < kColRegs; ++q) {
    const int i = lane + q * kW;
    const double h = i <= j ? dots[i] : 0.0;
    ss = fma(h, h, ss);
    col[q] = pass == 0 ? h : in.h0[q] + h;
  }
  ss = wave_sum64(ss);
  const double ww = dots[j + 1];
  const double hh2 = ww - ss;
  if (pass == 0 && !(hh2 > kReorthEta2 * ww)) {
    // cancellation: keep the coefficients and pause the cycle; the host runs
    // the second pass for this column and resumes
#pragma unroll
    for (int q = 0; q < kColRegs; ++q)
      if (lane + q * kW <= j) st->H[(lane + q * kW) * ld + j] = col[q];
    hd.reorth = 1;
    hd.direct = 0;
    hd.active = 0;
  } else {
    const double hn = hh2 > 0.0 ? std::sqrt(hh2) : 0.0;
    // previous rotations applied to the new column
    double a = lane_of(col[0], 0);
#pragma unroll
    for (int q = 0; q < kColRegs; ++q)
      for (int l = 0; l < kW && l + q * kW < j; ++l) {
        const double b = l + 1 < kW ? lane_of(col[q], l + 1) : lane_of(col[q + 1 < kColRegs ? q + 1 : q], 0);
        const double c = lane_of(in.cs[q], l), s = lane_of(in.sn[q], l);
        const double t = c * a + s * b;
        if (lane == l) col[q] = t;
        a = -s * a + c * b;
      }
#pragma unroll
    for (int q = 0; q < kColRegs; ++q)
      if (lane + q * kW < j) st->H[(lane + q * kW) * ld + j] = col[q];
    hd.reorth = 0;
    hd.hn = hn;
    hd.inv_hn = hn > 0.0 ? 1.0 / hn : 0.0;
    const double bb = hn;
    const double r = std::hypot(a, bb);
    double c = 1.0, s = 0.0;
    if (r != 0.0) {
      c = a / r;
      s = bb / r;
    }
    const double gj = in.g;
    hd.jend = j + 1;
    const double est = std::fabs(-s * gj);
    hd.est = est;
    hd.breakdown = (!(bb > 1e-300) || !(r > 0.0)) ? 1 : 0;
    hd.active = (est <= hd.tol || hd.breakdown) ? 0 : 1;
    // the update that follows forms v_{j+1} unless the cycle ends here
    hd.direct = hd.active;
    if (lane == 0) {
      st->cs[j] = c;
      st->sn[j] = s;
      st->H[j * ld + j] = r;
      st->H[(j + 1) * ld + j] = 0.0;
      st->g[j + 1] = -s * gj;
      st->g[j] = c * gj;
    }
  }
  if (lane == 0) *static_cast<ArnoldiHead*>(st) = hd;
}

// One Gram-Schmidt pass of Arnoldi step j in two launches: the multi-dot
// <v_i, w> (i < nv) and <w, w> over the blocks' chunks (k_gram_schmidt), then
// one workgroup that sums the blocks' partial results and forms the Hessenberg
// column (k_gs_column).  PASS 0 runs while the cycle is active; PASS 1
// (re-orthogonalisation) only when pass 0 asked for it, and first replaces w
// by w - V h0 with h0 the pass-0 coefficients.  Partial sums are stored
// column-major ([c][block]) so each column is summed from contiguous memory,
// always in the same order, so results are reproducible.
//
// Pass 0 spreads the groups of four basis vectors over blockIdx.y where the
// chunks alone do not fill the device (each block then reads w again): a chunk's
// groups one after the other are a chain of memory latencies.  At 33^3, 18
// chunks, a pass over 10 to 40 vectors took 7.9 us and takes 4.4 us; from
// about 4 workgroups per CU on the chunks are enough (129^3, 1049: unchanged).
constexpr int kGsThreads = 256;
constexpr int kGsEPT = 8;
constexpr int kGsChunk = kGsThreads * kGsEPT;
constexpr int kGsFill = 1024;  // workgroups of a pass-0 launch that the groups are spread up to
constexpr int kColThreads = 1024;  // the column kernel: one wave per column of partial sums (j < 16 in one round)

template <typename T, int PASS>
__global__ __launch_bounds__(kGsThreads) void k_gram_schmidt(const T* __restrict__ V, size_t ld, int nv, T* w,
                                                             size_t npts, const double* __restrict__ h0,
                                                             double* __restrict__ partials,
                                                             const ArnoldiState* st) {
  __shared__ double red[kGsThreads / 64][kMaxKrylovCols + 2];
  __shared__ double hs[kMaxKrylovCols + 2];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (PASS == 1 && !st->reorth) return;
  const int live = PASS == 0 ? st->active : 1;  // looked at before the store, its load beside the others
  const int nb = gridDim.x;
  const size_t b0 = (size_t)blockIdx.x * kGsChunk;
  double wv[kGsEPT];
  size_t ix[kGsEPT];
#pragma unroll
  for (int e = 0; e < kGsEPT; ++e) {
    const size_t i = b0 + tid + (size_t)e * kGsThreads;
    ix[e] = i < npts ? i : npts - 1;
    wv[e] = i < npts ? double(w[i]) : 0.0;
  }
  if (PASS == 1) {
    for (int v = tid; v < nv; v += kGsThreads) hs[v] = h0[v];
    __syncthreads();
    for (int v = 0; v < nv; ++v) {
      const double hv = hs[v];
#pragma unroll
      for (int e = 0; e < kGsEPT; ++e) wv[e] = fma(-hv, double(V[(size_t)v * ld + ix[e]]), wv[e]);
    }
#pragma unroll
    for (int e = 0; e < kGsEPT; ++e) {
      const size_t i = b0 + tid + (size_t)e * kGsThreads;
      if (i < npts) {
        w[i] = T(wv[e]);
        wv[e] = double(T(wv[e]));  // the dots see the stored (rounded) vector
      }
    }
  }
  // basis vectors four at a time, all their loads issued before the products
  // (slots past the last vector load w; every index is clamped into range)
  for (int v0 = 4 * blockIdx.y; v0 <= nv; v0 += 4 * gridDim.y) {
    T x[4][kGsEPT];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const T* Vi = v0 + g < nv ? V + (size_t)(v0 + g) * ld : w;
#pragma unroll
      for (int e = 0; e < kGsEPT; ++e) x[g][e] = Vi[ix[e]];
    }
    double acc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      acc[g] = 0.0;
      if (v0 + g < nv) {
#pragma unroll
        for (int e = 0; e < kGsEPT; ++e) acc[g] = fma(wv[e], double(x[g][e]), acc[g]);
      } else {
#pragma unroll
        for (int e = 0; e < kGsEPT; ++e) acc[g] = fma(wv[e], wv[e], acc[g]);
      }
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const double t = wave_sum64(acc[g]);
      if (lane == 0 && v0 + g <= nv) red[wave][v0 + g] = t;
    }
  }
  __syncthreads();
  if (!live) return;
  for (int v = tid; v <= nv; v += kGsThreads) {
    if (v / 4 % gridDim.y != blockIdx.y) continue;
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < kGsThreads / 64; ++q) sum += red[q][v];
    partials[(size_t)v * nb + blockIdx.x] = sum;
  }
}

// column sums of the nb blocks' partial results (wave q takes columns q,
// q + 4, ...; lanes stride the blocks), then the Hessenberg column
// (one workgroup, all latency: everything it reads is fetched at once, before the
// flag is looked at, the first 64 blocks' results of all of a wave's columns
// together, the rest sixteen at a time; 33^3: 5.1 us one after the other, 4.6 us so;
// 129^3, 1049 blocks: 8.1 us four at a time, 5.2 us so)
template <int PASS>
__global__ __launch_bounds__(kColThreads) void k_gs_column(const double* __restrict__ partials, int nb, int nv,
                                                          double* dots, ArnoldiState* st, int j) {
  constexpr int CW = (kMaxKrylovCols + 1 + kColThreads / 64 - 1) / (kColThreads / 64);  // columns per wave
  __shared__ double hs[kMaxKrylovCols + 2];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  ColumnIn in;
  column_fetch(st, j, PASS, lane, in);
  const bool live = PASS == 0 ? in.hd.active : in.hd.reorth;
  double s4[CW][4];
#pragma unroll
  for (int q = 0; q < CW; ++q) {
    const int c = wave + q * (kColThreads / 64);
    s4[q][0] = s4[q][1] = s4[q][2] = s4[q][3] = 0.0;
    if (c <= nv && lane < nb) s4[q][0] = partials[(size_t)c * nb + lane];
  }
#pragma unroll
  for (int q = 0; q < CW; ++q) {
    const int c = wave + q * (kColThreads / 64);
    if (c > nv) break;
    const double* pc = partials + (size_t)c * nb;
    for (int r = 64 + lane; r < nb; r += 1024) {
      double x[16];
#pragma unroll
      for (int g = 0; g < 16; ++g) x[g] = r + 64 * g < nb ? pc[r + 64 * g] : 0.0;
#pragma unroll
      for (int g = 0; g < 16; ++g) s4[q][(g + 1) & 3] += x[g];
    }
    const double sum = wave_sum64((s4[q][0] + s4[q][1]) + (s4[q][2] + s4[q][3]));
    if (lane == 0) hs[c] = sum;
  }
  __syncthreads();
  if (!live) return;
  for (int v = tid; v <= nv; v += kColThreads) dots[v] = hs[v];
  if (wave == 0) arnoldi_column_wave(st, hs, j, PASS, lane, in);
}

// y = R^{-1} g over the columns the cycle built (back-substitution)
__global__ __launch_bounds__(kW) void k_arnoldi_solve(ArnoldiState* st) {
  const int lane = threadIdx.x;
  const int jend = st->jend;
  const int ld = kMaxKrylovCols;
  for (int i = jend - 1; i >= 0; --i) {
    double t = 0.0;
    for (int l = i + 1 + lane; l < jend; l += kW) t = fma(st->H[i * ld + l], st->y[l], t);
    t = wave_sum64(t);
    if (lane == 0) {
      const double d = st->H[i * ld + i];
      st->y[i] = d != 0.0 ? (st->g[i] - t) / d : 0.0;
    }
    __syncthreads();
  }
}

template <typename T>
__global__ void k_scale_by(T* v, const double* dscale, size_t npts) {
  const double a = *dscale;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < npts; i += (size_t)gridDim.x * blockDim.x)
    v[i] = T(a * double(v[i]));
}

inline int blocks_for(size_t n) {
  size_t g = (n + 1023) / 1024;
  if (g < 1) g = 1;
  if (g > 8192) g = 8192;
  return (int)g;
}

}  // namespace

int arnoldi_init(ArnoldiState* st, double tol, double stall, hipStream_t s) {
  hipLaunchKernelGGL(k_arnoldi_init, dim3(1), dim3(kW), 0, s, st, tol, stall);
  return hip_check(hipGetLastError(), "arnoldi_init");
}

int arnoldi_begin(ArnoldiState* st, const double* dots, hipStream_t s) {
  hipLaunchKernelGGL(k_arnoldi_begin, dim3(1), dim3(kW), 0, s, st, dots);
  return hip_check(hipGetLastError(), "arnoldi_begin");
}

template <typename T>
int gram_schmidt(const T* V, size_t ld, int j, T* w, size_t npts, const double* h0, double* partials,
                 double* dots, ArnoldiState* st, int pass, hipStream_t s) {
  if (j < 0 || j >= kMaxKrylovCols || npts == 0) {
    set_error("Arnoldi column out of range");
    return CHEB_ERR_INVALID_ARG;
  }
  const int nb = (int)((npts + kGsChunk - 1) / kGsChunk);
  if (pass == 0) {
    const int groups = (j + 1) / 4 + 1, fill = kGsFill / nb;
    const int gy = fill < 1 ? 1 : groups < fill ? groups : fill;
    hipLaunchKernelGGL((k_gram_schmidt<T, 0>), dim3(nb, gy), dim3(kGsThreads), 0, s, V, ld, j + 1, w, npts, h0,
                       partials, st);
    hipLaunchKernelGGL(k_gs_column<0>, dim3(1), dim3(kColThreads), 0, s, partials, nb, j + 1, dots, st, j);
  } else {
    hipLaunchKernelGGL((k_gram_schmidt<T, 1>), dim3(nb), dim3(kGsThreads), 0, s, V, ld, j + 1, w, npts, h0,
                       partials, st);
    hipLaunchKernelGGL(k_gs_column<1>, dim3(1), dim3(kColThreads), 0, s, partials, nb, j + 1, dots, st, j);
  }
  return hip_check(hipGetLastError(), "gram_schmidt");
}

int arnoldi_solve(ArnoldiState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_arnoldi_solve, dim3(1), dim3(kW), 0, s, st);
  return hip_check(hipGetLastError(), "arnoldi_solve");
}

template <typename T>
int scale_by(T* v, const double* dscale, size_t npts, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_by<T>, dim3(blocks_for(npts)), dim3(256), 0, s, v, dscale, npts);
  return hip_check(hipGetLastError(), "scale_by");
}

template int gram_schmidt<double>(const double*, size_t, int, double*, size_t, const double*, double*, double*,
                                  ArnoldiState*, int, hipStream_t);
template int gram_schmidt<float>(const float*, size_t, int, float*, size_t, const double*, double*, double*,
                                 ArnoldiState*, int, hipStream_t);
template int scale_by<double>(double*, const double*, size_t, hipStream_t);
template int scale_by<float>(float*, const double*, size_t, hipStream_t);

}  // namespace cheb

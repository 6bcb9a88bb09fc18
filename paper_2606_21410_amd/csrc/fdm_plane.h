// The preconditioner's two contractions within an x-plane -- z then y on the
// way in, y then z on the way out -- as one kernel, the plane's values between
// them in LDS.  Included by precond.hip and the instantiation files.
//
// A workgroup owns one plane of one system, or half of the plane's y rows where
// y is even-odd split and has more than one 16-row block per half:
//   forward, half h: the pair sums (h = 0) or differences (h = 1) of the rows y
//   and m1-1-y enter LDS as they are loaded; the z contraction is linear, so it
//   runs on those ps (or ph) rows, and the y contraction of half h's modes needs
//   no others;
//   backward, half h: half of the row pairs: their y contraction over all the
//   modes, then z on the resulting rows y and m1-1-y.
// So the two halves share no work and exchange nothing.  Every phase gives a
// wave one unit: 16 columns of a y contraction, or 16 rows and one half of the
// modes (forward) or of the row blocks (backward) of a z contraction, with at
// most RB row blocks of each parity.  The fragment tables (precond.hip) are
// copied into LDS once per workgroup; the z contractions take the table as
// MFMA's B operand, which leaves z along the lanes: full rows of 16 leave in one
// store.
//
// What bounds it at 129^3 in FP64: 254 workgroups, one to a CU (160 KB of LDS);
// each 1024 matrix-core steps on four SIMDs, 16.4k cycles, behind the loads of
// its plane.  Forward 22.0 us, backward 20.5 (about 11 us of each without the
// matrix steps and 2 us for the tables); an axis at a time took 12 us per axis and
// direction.  The phases of the one round do not overlap: what is left.
#pragma once

#include "dev_common.h"
#include "internal.h"

namespace cheb {

// k-index of MFMA step ks for lane group lk (lane / 16) of the preconditioner's
// tables: the row that the accumulator of the same type holds in register ks % 4
// of row block ks / 4
__host__ __device__ constexpr int fdm_kmap(int ks, int lk, bool f32) {
  return f32 ? 16 * (ks / 4) + 4 * lk + (ks % 4) : 4 * ks + lk;
}

struct PlaneArgs {
  const int* gate;        // null, or a device flag: nothing is done while it reads 0
  const void* ty;         // fragment tables of the y and the z contraction
  const void* tz;
  const void* X;          // forward: full fields, backward: packed modes
  void* Y;                // forward: packed modes, backward: full fields
  const long long* offs;  // field b starts at offs[b] (null: b * n0 n1 n2)
  const PcTables* mem;    // batches of mixed face types: tables of system sys[b] (null: ty, tz)
  const int* sys;
  int m0, m1, m2, nb;
  int halves;             // workgroups per plane (set by the launch)
};

// sizes shared by the kernels and the launch; SY, SZ: even-odd split axes
template <typename T, bool SY, bool SZ>
struct PlaneDims {
  int by, bz;    // 16-row blocks, of a half where split
  int sy, sz;    // contraction steps
  int ld;        // row pitch of the plane in LDS
  int hb;        // backward: row blocks of each parity of one workgroup
  __host__ __device__ PlaneDims(int m1, int m2, int halves) {
    by = ((SY ? (m1 + 1) / 2 : m1) + 15) / 16;
    bz = ((SZ ? (m2 + 1) / 2 : m2) + 15) / 16;
    sy = 4 * by;
    sz = 4 * bz;
    constexpr int pad = sizeof(T) == sizeof(double) ? 32 : 64;
    ld = (m2 + pad - 1) / pad * pad;
    hb = halves == 2 ? (by + 1) / 2 : by;
  }
  __host__ __device__ int ztab() const { return (SZ ? 2 : 1) * bz * sz * 64; }
  __host__ __device__ int rows(bool fwd) const { return 16 * (fwd ? by : (SY ? 2 : 1) * hb); }
  __host__ __device__ int ytab(bool fwd) const { return (fwd ? by : (SY ? 2 : 1) * hb) * sy * 64; }
  __host__ __device__ int lds(bool fwd) const {
    return (rows(fwd) * ld + ytab(fwd) + ztab()) * (int)sizeof(T);
  }
};

// element (r, c) of the plane in LDS: 4-wide column groups rotated by the row, so
// that a read of 4 columns of 16 rows and one of 16 columns of 4 rows both spread
// over the banks; the pitch is a whole number of rotations
template <typename T>
__device__ __forceinline__ int plane_at(int r, int c, int ld) {
  return r * ld + (c ^ ((r & (sizeof(T) == sizeof(double) ? 7 : 15)) << 2));
}

__device__ __forceinline__ void plane_copy(const void* src, void* dst, int bytes, int tid, int nt) {
  typedef int I4 __attribute__((ext_vector_type(4)));
  const I4* s = (const I4*)src;
  I4* d = (I4*)dst;
  const int n = bytes / 16;
  for (int e = tid; e < n; e += 4 * nt) {
    I4 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = s[e + q * nt < n ? e + q * nt : n - 1];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (e + q * nt < n) d[e + q * nt] = v[q];
  }
}

// the workgroup's plane (block b, x index i0) and half; both halves of a plane on
// one XCD (workgroups go to the XCDs in turn), whose L2 then serves the second read
struct PlaneId {
  int plane, h;
  __device__ explicit PlaneId(int halves) {
    const int w = blockIdx.x;
    plane = halves == 2 ? (w >> 4) * 8 + (w & 7) : w;
    h = halves == 2 ? (w >> 3) & 1 : 0;
  }
};

template <typename T, int RB, bool SY, bool SZ>
__global__ __launch_bounds__(512) void k_fdm_plane_fwd(PlaneArgs g) {
  const int live = g.gate ? *g.gate : 1;  // looked at once the loads are out
  typedef typename Mfma<T>::v4 V4;
  constexpr bool F32 = sizeof(T) == sizeof(float);
  extern __shared__ __align__(16) unsigned char smem[];
  const PlaneDims<T, SY, SZ> d(g.m1, g.m2, g.halves);
  const PlaneId id(g.halves);
  if (id.plane >= g.m0 * g.nb) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nt = blockDim.x, nw = nt >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int m1 = g.m1, m2 = g.m2, ps1 = (m1 + 1) / 2, ps2 = (m2 + 1) / 2;
  const int n1 = m1 + 2, n2 = m2 + 2;
  const int b = id.plane / g.m0, i0 = id.plane - b * g.m0;
  const T* X = (const T*)g.X + (g.offs ? g.offs[b] : (long long)b * (g.m0 + 2) * n1 * n2) +
               ((long long)(i0 + 1) * n1 + 1) * n2 + 1;
  T* Y = (T*)g.Y + (long long)id.plane * m1 * m2;
  T* ty = (T*)smem;
  T* tz = ty + d.ytab(true);
  T* S = tz + d.ztab();
  const T* gy = (const T*)(g.mem ? g.mem[g.sys[b]].in[1] : g.ty);
  const T* gz = (const T*)(g.mem ? g.mem[g.sys[b]].in[2] : g.tz);
  const int ld = d.ld, rows = d.rows(true);
  const int h = id.h, rin = SY ? (h ? m1 - ps1 : ps1) : m1;  // rows of this half
  // the plane's rows (or their pair sums or differences; the middle row twice, its
  // column of the y table is halved), in flight behind the tables
  constexpr int QR = RB == 1 ? 4 : 8;
  T lo[QR][2], hi[SY ? QR : 1][2];
  auto load = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < QR; ++q) {
      const int r = r0 + q * nw, rr = r < rin ? r : rin - 1, rc = rr > 0 ? rr : 0;
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        if (64 * z >= m2) break;
        const int c = lane + 64 * z < m2 ? lane + 64 * z : m2 - 1;
        lo[q][z] = X[(long long)rc * n2 + c];
        if (SY) hi[SY ? q : 0][z] = X[(long long)(m1 - 1 - rc) * n2 + c];
      }
    }
  };
  load(wave);
  plane_copy(gy + h * d.ytab(true), ty, d.ytab(true) * (int)sizeof(T), tid, nt);
  plane_copy(gz, tz, d.ztab() * (int)sizeof(T), tid, nt);
  for (int r0 = wave; r0 < rows; r0 += QR * nw) {
    if (r0 != wave) load(r0);
#pragma unroll
    for (int q = 0; q < QR; ++q) {
      const int r = r0 + q * nw;
      if (r >= rows) break;
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        const int c = lane + 64 * z;
        if (c >= ld) break;
        T v = T(0);
        if (r < rin && c < m2) v = !SY ? lo[q][z] : h ? lo[q][z] - hi[SY ? q : 0][z] : lo[q][z] + hi[SY ? q : 0][z];
        S[plane_at<T>(r, c, ld)] = v;
      }
    }
  }
  __syncthreads();
  if (!live) return;
  // z: unit = 16 rows and one parity of the modes (half of the row blocks where
  // z is not split); the results replace the rows once every wave has read them
  const int zt = wave >> 1, zp = wave & 1;
  const int nzb = SZ ? d.bz : zp ? d.bz - (d.bz + 1) / 2 : (d.bz + 1) / 2, zb0 = SZ ? zp * d.bz : zp * ((d.bz + 1) / 2);
  const bool zrun = 16 * zt < rows && nzb > 0;
  V4 acc[RB];
#pragma unroll
  for (int q = 0; q < RB; ++q) acc[q] = V4{0, 0, 0, 0};
  if (zrun) {
    const T* t = tz + zb0 * d.sz * 64 + lane;
    const int r = 16 * zt + li;
#pragma unroll 4
    for (int ks = 0; ks < d.sz; ++ks) {
      const int k = fdm_kmap(ks, lk, F32);
      T x;
      if (SZ) {
        const int kk = k < ps2 ? k : ps2 - 1;
        const T x1 = S[plane_at<T>(r, kk, ld)], x2 = S[plane_at<T>(r, m2 - 1 - kk, ld)];
        x = zp ? x1 - x2 : x1 + x2;
      } else {
        x = S[plane_at<T>(r, k < m2 ? k : m2 - 1, ld)];
      }
#pragma unroll
      for (int q = 0; q < RB; ++q)
        acc[q] = Mfma<T>::mac(x, t[((q < nzb ? q : 0) * d.sz + ks) * 64], acc[q]);
    }
  }
  __syncthreads();
  if (zrun) {
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      if (q >= nzb) break;
      const int row = 16 * q + li, lim = SZ ? (zp ? m2 - ps2 : ps2) : m2 - 16 * zb0;
      const int c = SZ ? (zp ? ps2 + row : row) : 16 * zb0 + row;
      if (row >= lim) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) S[plane_at<T>(16 * zt + Mfma<T>::row(lk, r), c, ld)] = acc[q][r];
    }
  }
  __syncthreads();
  // y: unit = 16 columns (z modes), every row block of this half
  const int c = 16 * wave + li, cc = c < m2 ? c : m2 - 1;
  if (16 * wave < m2) {
#pragma unroll
    for (int q = 0; q < RB; ++q) acc[q] = V4{0, 0, 0, 0};
    const T* t = ty + lane;
#pragma unroll 4
    for (int ks = 0; ks < d.sy; ++ks) {
      const T x = S[plane_at<T>(fdm_kmap(ks, lk, F32), cc, ld)];
#pragma unroll
      for (int q = 0; q < RB; ++q)
        acc[q] = Mfma<T>::mac(t[((q < d.by ? q : 0) * d.sy + ks) * 64], x, acc[q]);
    }
    if (c < m2) {
#pragma unroll
      for (int q = 0; q < RB; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * q + Mfma<T>::row(lk, r);
          if (row < rin) Y[(long long)(SY && h ? ps1 + row : row) * m2 + c] = acc[q][r];
        }
    }
  }
}

template <typename T, int RB, bool SY, bool SZ>
__global__ __launch_bounds__(512) void k_fdm_plane_bwd(PlaneArgs g) {
  const int live = g.gate ? *g.gate : 1;  // looked at once the loads are out
  typedef typename Mfma<T>::v4 V4;
  constexpr bool F32 = sizeof(T) == sizeof(float);
  constexpr int HB = SY && RB > 1 ? (RB + 1) / 2 : RB;  // row blocks of a parity per workgroup
  extern __shared__ __align__(16) unsigned char smem[];
  const PlaneDims<T, SY, SZ> d(g.m1, g.m2, g.halves);
  const PlaneId id(g.halves);
  if (id.plane >= g.m0 * g.nb) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nt = blockDim.x;
  const int li = lane & 15, lk = lane >> 4;
  const int m1 = g.m1, m2 = g.m2, ps1 = (m1 + 1) / 2, ps2 = (m2 + 1) / 2;
  const int n0 = g.m0 + 2, n1 = m1 + 2, n2 = m2 + 2;
  const int b = id.plane / g.m0, i0 = id.plane - b * g.m0;
  const T* X = (const T*)g.X + (long long)id.plane * m1 * m2;
  T* Y = (T*)g.Y + (g.offs ? g.offs[b] : (long long)b * n0 * n1 * n2) + ((long long)(i0 + 1) * n1 + 1) * n2 + 1;
  const T* gy = (const T*)(g.mem ? g.mem[g.sys[b]].out[1] : g.ty);
  const T* gz = (const T*)(g.mem ? g.mem[g.sys[b]].out[2] : g.tz);
  const int ld = d.ld, rows = d.rows(false), hb = d.hb, b0 = id.h * hb;
  const int nyb = b0 + hb <= d.by ? hb : d.by - b0;  // row blocks of a parity of this half
  T* ty = (T*)smem;
  T* tz = ty + d.ytab(false);
  T* S = tz + d.ztab();
  // this wave's columns of the y modes, in flight behind the tables
  constexpr int SMAX = 4 * RB;
  const int c = 16 * wave + li, cc = c < m2 ? c : m2 - 1;
  const bool yrun = 16 * wave < m2;
  T xs[SMAX], xa[SY ? SMAX : 1];
  if (yrun) {
#pragma unroll
    for (int ks = 0; ks < SMAX; ++ks) {
      const int k = fdm_kmap(ks, lk, F32);
      if (SY) {
        xs[ks] = X[(long long)(k < ps1 ? k : ps1 - 1) * m2 + cc];
        xa[SY ? ks : 0] = X[(long long)(ps1 + k < m1 ? ps1 + k : m1 - 1) * m2 + cc];
      } else {
        xs[ks] = X[(long long)(k < m1 ? k : m1 - 1) * m2 + cc];
      }
    }
  }
  const int part = nyb * d.sy * 64 * (int)sizeof(T);
  plane_copy(gy + b0 * d.sy * 64, ty, part, tid, nt);
  if (SY) plane_copy(gy + (d.by + b0) * d.sy * 64, ty + hb * d.sy * 64, part, tid, nt);
  plane_copy(gz, tz, d.ztab() * (int)sizeof(T), tid, nt);
  if (!live) return;
  {
    // the boundary nodes: this plane's edges, and a share of the field's x faces
    T* P = Y - n2 - 1;
    if (id.h == 0)
      for (int t = tid; t < 2 * n2; t += nt) P[t < n2 ? t : (long long)(n1 - 2) * n2 + t] = T(0);
    if (id.h == g.halves - 1)
      for (int t = tid; t < 2 * m1; t += nt) P[(long long)(1 + (t >> 1)) * n2 + (t & 1) * (n2 - 1)] = T(0);
    T* P0 = P - (long long)(i0 + 1) * n1 * n2;
    const int face = n1 * n2;
    for (int t = (i0 * g.halves + id.h) * nt + tid; t < 2 * face; t += g.m0 * g.halves * nt)
      P0[t < face ? t : (long long)(n0 - 2) * face + t] = T(0);
  }
  __syncthreads();
  if (yrun) {
    V4 a[HB], o[SY ? HB : 1];
#pragma unroll
    for (int q = 0; q < HB; ++q) {
      a[q] = V4{0, 0, 0, 0};
      if (SY) o[SY ? q : 0] = V4{0, 0, 0, 0};
    }
    const T* ta = ty + lane;
    const T* to = ty + hb * d.sy * 64 + lane;
#pragma unroll
    for (int kb = 0; kb < RB; ++kb) {
      if (kb >= d.by) break;
#pragma unroll
      for (int ks = 4 * kb; ks < 4 * kb + 4; ++ks)
#pragma unroll
        for (int q = 0; q < HB; ++q) {
          const int qq = ((q < nyb ? q : 0) * d.sy + ks) * 64;
          a[q] = Mfma<T>::mac(ta[qq], xs[ks], a[q]);
          if (SY) o[SY ? q : 0] = Mfma<T>::mac(to[qq], xa[SY ? ks : 0], o[SY ? q : 0]);
        }
    }
    // rows 16 q + r of the first set, their mirrors in the second; blocks past
    // this half's are not read
    if (c < ld) {
#pragma unroll
      for (int q = 0; q < HB; ++q) {
        if (q >= hb) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * q + Mfma<T>::row(lk, r);
          if (SY) {
            S[plane_at<T>(row, c, ld)] = a[q][r] + o[SY ? q : 0][r];
            S[plane_at<T>(16 * hb + row, c, ld)] = a[q][r] - o[SY ? q : 0][r];
          } else {
            S[plane_at<T>(row, c, ld)] = a[q][r];
          }
        }
      }
    }
  }
  __syncthreads();
  // z: unit = 16 rows and half of the row blocks
  const int zt = wave >> 1, zp = wave & 1, zh = (d.bz + 1) / 2;
  const int zb0 = zp * zh, nzb = zp ? d.bz - zh : zh;
  if (16 * zt >= rows || nzb == 0) return;
  constexpr int ZB = (RB + 1) / 2;
  constexpr int ZN = SZ ? ZB : RB;
  V4 a[ZN], o[SZ ? ZB : 1];
#pragma unroll
  for (int q = 0; q < ZN; ++q) {
    a[q] = V4{0, 0, 0, 0};
    if (SZ) o[SZ ? q : 0] = V4{0, 0, 0, 0};
  }
  const T* ta = tz + zb0 * d.sz * 64 + lane;
  const T* to = tz + (d.bz + zb0) * d.sz * 64 + lane;
  const int r = 16 * zt + li;
#pragma unroll 4
  for (int ks = 0; ks < d.sz; ++ks) {
    const int k = fdm_kmap(ks, lk, F32);
    T x, y = T(0);
    if (SZ) {
      x = S[plane_at<T>(r, k < ps2 ? k : ps2 - 1, ld)];
      y = S[plane_at<T>(r, ps2 + k < m2 ? ps2 + k : m2 - 1, ld)];
    } else {
      x = S[plane_at<T>(r, k < m2 ? k : m2 - 1, ld)];
    }
#pragma unroll
    for (int q = 0; q < ZN; ++q) {
      const int qq = ((q < nzb ? q : 0) * d.sz + ks) * 64;
      a[q] = Mfma<T>::mac(x, ta[qq], a[q]);
      if (SZ) o[SZ ? q : 0] = Mfma<T>::mac(y, to[qq], o[SZ ? q : 0]);
    }
  }
#pragma unroll
  for (int rr = 0; rr < 4; ++rr) {
    const int lr = 16 * zt + Mfma<T>::row(lk, rr);
    int yr;
    if (SY) {
      const bool mir = lr >= 16 * hb;
      const int i = 16 * b0 + (mir ? lr - 16 * hb : lr);
      // blocks past this half's belong to no row of it
      yr = (mir ? lr - 16 * hb : lr) >= 16 * nyb ? -1 : mir ? (i < m1 - ps1 ? m1 - 1 - i : -1) : (i < ps1 ? i : -1);
    } else {
      yr = lr < m1 ? lr : -1;
    }
    if (yr < 0) continue;
    T* out = Y + (long long)yr * n2;
#pragma unroll
    for (int q = 0; q < ZN; ++q) {
      if (q >= nzb) break;
      const int i = 16 * (zb0 + q) + li;
      if (SZ) {
        if (i < ps2) out[i] = a[q][rr] + o[SZ ? q : 0][rr];
        if (i < m2 - ps2) out[m2 - 1 - i] = a[q][rr] - o[SZ ? q : 0][rr];
      } else if (i < m2) {
        out[i] = a[q][rr];
      }
    }
  }
}

constexpr int kPlaneLds = 160 * 1024;

// whether both directions take an m1 x m2 plane: at most four row blocks per unit
// and the tables and rows within LDS
template <typename T>
bool plane_ok(int m1, int m2, bool sy, bool sz) {
  if (m1 > (sy ? 128 : 64) || m2 > 128) return false;
  auto fits = [&](auto d1, auto d2) { return d1.lds(true) <= kPlaneLds && d2.lds(false) <= kPlaneLds; };
  const int hf = sy ? 2 : 1, hb = sy && m1 > 32 ? 2 : 1;
  if (sy) {
    if (sz) return fits(PlaneDims<T, true, true>(m1, m2, hf), PlaneDims<T, true, true>(m1, m2, hb));
    return fits(PlaneDims<T, true, false>(m1, m2, hf), PlaneDims<T, true, false>(m1, m2, hb));
  }
  if (sz) return fits(PlaneDims<T, false, true>(m1, m2, hf), PlaneDims<T, false, true>(m1, m2, hb));
  return fits(PlaneDims<T, false, false>(m1, m2, hf), PlaneDims<T, false, false>(m1, m2, hb));
}

template <typename T, int RB, bool SY, bool SZ, bool FWD>
int launch_plane_inst(PlaneArgs a, hipStream_t s) {
  a.halves = SY && (FWD || a.m1 > 32) ? 2 : 1;
  const PlaneDims<T, SY, SZ> d(a.m1, a.m2, a.halves);
  const int lds = d.lds(FWD);
  const void* kern = FWD ? (const void*)k_fdm_plane_fwd<T, RB, SY, SZ> : (const void*)k_fdm_plane_bwd<T, RB, SY, SZ>;
  if (lds > 64 * 1024) {
    static DeviceCache attr;  // 1 once the LDS attribute is set on the device
    int dev = 0;
    if (int rc = current_device(&dev)) return rc;
    if (!attr.v[dev].load(std::memory_order_relaxed)) {
      if (int rc = hip_check(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, kPlaneLds),
                             "plane contraction LDS attribute"))
        return rc;
      attr.v[dev].store(1, std::memory_order_relaxed);
    }
  }
  const int planes = a.m0 * a.nb;
  const int grid = a.halves == 2 ? (planes + 7) / 8 * 16 : planes;
  int nw = 2 * d.rows(FWD) / 16;
  if (nw < (a.m2 + 15) / 16) nw = (a.m2 + 15) / 16;
  if (nw < 4) nw = 4;
  if constexpr (FWD) hipLaunchKernelGGL((k_fdm_plane_fwd<T, RB, SY, SZ>), dim3(grid), dim3(64 * nw), lds, s, a);
  else hipLaunchKernelGGL((k_fdm_plane_bwd<T, RB, SY, SZ>), dim3(grid), dim3(64 * nw), lds, s, a);
  return hip_check(hipGetLastError(), "plane contraction");
}

// row blocks that a kernel of the pair has to hold (its RB)
template <typename T>
int plane_blocks(int m1, int m2, bool sy, bool sz) {
  const int by = ((sy ? (m1 + 1) / 2 : m1) + 15) / 16, bz = ((sz ? (m2 + 1) / 2 : m2) + 15) / 16;
  const int z = sz ? bz : (bz + 1) / 2;
  return by > z ? by : z;
}

template <typename T, int RB>
int launch_plane_rb(const PlaneArgs& a, bool fwd, bool sy, bool sz, hipStream_t s) {
  if (fwd) {
    if (sy) return sz ? launch_plane_inst<T, RB, true, true, true>(a, s) : launch_plane_inst<T, RB, true, false, true>(a, s);
    return sz ? launch_plane_inst<T, RB, false, true, true>(a, s) : launch_plane_inst<T, RB, false, false, true>(a, s);
  }
  if (sy) return sz ? launch_plane_inst<T, RB, true, true, false>(a, s) : launch_plane_inst<T, RB, true, false, false>(a, s);
  return sz ? launch_plane_inst<T, RB, false, true, false>(a, s) : launch_plane_inst<T, RB, false, false, false>(a, s);
}

#define PLANE_EXTERN(T, RB) extern template int launch_plane_rb<T, RB>(const PlaneArgs&, bool, bool, bool, hipStream_t)
#define PLANE_INSTANCE(T, RB) template int launch_plane_rb<T, RB>(const PlaneArgs&, bool, bool, bool, hipStream_t)

}  // namespace cheb

// Matrix-core pass along one axis for N <= 128 (at most four 16-row blocks):
// one wave owns a task of 16 pencils and computes every row of them.
//
// The operands never leave the wave: the pencils' pair sums and differences are
// the B operand in registers, the fragments of D come from a table in LDS that
// the workgroup copies once, and the k order of the steps is the row order of
// the accumulators (line_kmap), so the flux formed from the first product's
// accumulators is the second product's B operand in place.  Nothing is exchanged
// between waves and there is no barrier behind the table copy; eight
// accumulator chains (even and odd part of four row blocks) run at once, and
// with two waves per SIMD one's loads and stores pass under the other's
// products.  Bound by the matrix cores: 264 FP64 instructions of 64 cycles per
// task at N = 128.
//
// Along x and y 16 consecutive lanes hold 16 consecutive values of the pencils'
// common row.  Along z (CG) the pencils are the contiguous direction: values
// pass between the coalesced order (lane % 16 along the pencil) and the
// accumulator order through a 16 x 16 patch of LDS of the wave's own.
#pragma once

#include "dense_pass.h"

namespace cheb {

// lane moves across the four 16-lane rows of a wave
template <typename T>
__device__ __forceinline__ T rows_sum(T v) {
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

template <typename T>
__host__ __device__ constexpr int wave_lds_bytes(int MT, int NW, bool CG) {
  return line_tab(MT).size * (int)sizeof(T) + (CG ? NW * 16 * 17 * (int)sizeof(T) : 0);
}

// orders the wave's LDS writes before its later reads of other lanes' values
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

template <typename T>
__host__ __device__ constexpr int wave_simd_waves(int MT, int MODE, int NW) {
  if (sizeof(T) == sizeof(float)) return MT <= 3 ? 4 : 3;
  return MODE == LINE_JAC ? (MT <= 2 ? 2 : 1) : MT <= 2 ? 3 : 2;
}

template <typename T, int MT, int MODE, bool FIRST, bool CG, int NW>
__global__ __launch_bounds__(64 * NW, wave_simd_waves<T>(MT, MODE, NW)) void k_line_wave(LineArgs<T> a) {
  const int live = a.gate ? *a.gate : 1;  // looked at once the first loads are out
  typedef typename Mfma<T>::v4 V4;
  constexpr bool FULL = MODE == LINE_FULL, DMUL = MODE == LINE_DMUL, DER = MODE == LINE_DERIV || DMUL;
  constexpr bool JAC = MODE == LINE_JAC;
  constexpr bool LIFT = MODE == LINE_REDUCED || MODE == LINE_JAC, TRA = MODE == LINE_TRANSP;
  constexpr bool ALLP = FULL || DER;   // every pencil, end values of u included
  constexpr bool YADD = CG && !FIRST;  // the last pass of a two-axis apply adds yadd
  constexpr bool F32 = sizeof(T) == sizeof(float);
  static_assert(!DER || FIRST, "derivatives do not accumulate");
  constexpr int KS = 4 * MT, NT = 64 * NW;
  constexpr LineTab LT = line_tab(MT);

  extern __shared__ __align__(16) unsigned char smem[];
  T* tab = (T*)smem;
  const T* te = tab;
  const T* to = tab + LT.off_o;
  const T* amid = tab + LT.off_mid;
  const T* dc0 = tab + LT.off_c0;
  const T* dcN = tab + LT.off_cN;
  const T* linv = tab + LT.off_lift;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int li = lane & 15, lk = lane >> 4;
  T* patch = tab + LT.size + wave * 16 * 17;
  const int seg = a.nseg == 2 ? (blockIdx.x >> 3) & 1 : 0;
  const int vb = a.nseg == 2 ? (int)(((blockIdx.x >> 4) << 3) | (blockIdx.x & 7)) : (int)blockIdx.x;
  const int vg = a.nseg == 2 ? (int)(gridDim.x >> 1) : (int)gridDim.x;
  const LineAxis<T> A = seg ? a.ax[1] : a.ax[0];
  const int axis = A.axis, N = A.N;
  const int R = line_pairs(N);
  const bool midv = line_midv(N, MT);
  const int RM = midv ? R - 1 : R;  // rows on the matrix cores
  const int half = N >> 1;
  const int n0 = a.n[0], n1 = a.n[1], n2 = a.n[2];
  const int stride = CG ? 1 : axis == 1 ? n2 : n1 * n2;
  int st = stride;
  constexpr int po = ALLP ? 0 : 1;  // transverse offset of the first pencil
  const int na = axis == 0 ? n1 : n0, nb = axis == 2 ? n1 : n2;
  const int nbi = nb - 2 * po;
  const int npen = (na - 2 * po) * nbi;
  const int tps = (npen + 15) >> 4;  // tasks per system
  const int nsys = a.sys ? a.nact : 1;
  const int ntasks = nsys * tps;

  // XCD-aware order: workgroups are dealt round-robin to the 8 XCDs, so
  // workgroup b serves a contiguous range of tasks of XCD b % 8 and tasks that
  // share cache lines at their edges meet in the same L2
  const int per = (ntasks + 7) >> 3, xcd = vb & 7;
  const int t_step = (vg >> 3) * a.wpw, t_end = min(ntasks, (xcd + 1) * per);
  int task = wave < a.wpw ? xcd * per + (vb >> 3) * a.wpw + wave : t_end;

  // this lane's pencil of a task: pencil li, its index, first node and flags;
  // CG: also the first nodes of the pencils of the coalesced order
  int q = 0, b0 = -1, fl = 0, bp[CG ? 4 : 1];
  bool valid = false;
  const T *pu, *pk;
  T* py;
  int bm;
  auto locate = [&](int t) __attribute__((always_inline)) {
    pu = a.u;
    pk = a.K;
    py = A.y;
    bm = a.bcmask;
    if (a.sys) {
      const int sy = t / tps;
      const DenseSys d = dense_sys_at(a, sy);
      pu = a.u + d.off;
      pk = a.K + d.koff;
      py = A.y + d.off;
      bm = d.bcmask;
      t -= sy * tps;
    }
    q = t * 16 + li;
    valid = q < npen;
    const int qv = valid ? q : npen - 1;
    const int qa = fast_div(qv, nbi, A.inv_nbi);
    const int ia = po + qa, ib = po + qv - __mul24(qa, nbi);
    b0 = axis == 2 ? (ia * n1 + ib) * n2 : axis == 1 ? ia * n1 * n2 + ib : ia * n2 + ib;
    if (FULL) {
      long long bb;
      fl = valid ? pencil_flags(axis, q, npen, n0, n1, n2, a.bcmask, &bb) : 0;
    }
    if (CG) {
      const int bv = valid && (!FULL || (fl & PF_TIN)) ? b0 : -1 - b0;  // negative: not stored
#pragma unroll
      for (int r = 0; r < 4; ++r) bp[CG ? r : 0] = __shfl(DER ? (valid ? b0 : -1 - b0) : bv, lk + 4 * r, 64);
    }
  };
  // row of step ks (and of accumulator register ks % 4 of block ks / 4) in this
  // lane, and the node of the coalesced order
  auto row_of = [&](int ks) __attribute__((always_inline)) { return line_kmap(ks, lk, F32); };
  // loads l = 0..7 of block m of a field: along x and y the lower and upper
  // node of the lane's rows, along z those of the coalesced order
  auto at = [&](const T* p, int m, int r, bool upper) __attribute__((always_inline)) {
    int i = CG ? 16 * m + li : row_of(4 * m + r);
    i = i < N ? i : N;
    const int bb = CG ? bp[CG ? r : 0] : b0;
    const int b = CG ? (bb < 0 ? -1 - bb : bb) : bb;
    return dense_at(p, b + __mul24(upper ? N - i : i, st));
  };
  // coalesced order -> accumulator order (and back) of one block's four values
  auto to_rows = [&](T (&v)[4]) __attribute__((always_inline)) {
    if constexpr (CG) {
#pragma unroll
      for (int r = 0; r < 4; ++r) patch[li * 17 + lk + 4 * r] = v[r];
      wave_lds_sync();
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = patch[Mfma<T>::row(lk, r) * 17 + li];
      wave_lds_sync();
    }
  };
  auto to_lines = [&](T (&v)[4]) __attribute__((always_inline)) {
    if constexpr (CG) {
#pragma unroll
      for (int r = 0; r < 4; ++r) patch[Mfma<T>::row(lk, r) * 17 + li] = v[r];
      wave_lds_sync();
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = patch[li * 17 + lk + 4 * r];
      wave_lds_sync();
    }
  };

  // u of a task: pairs (j, N - j)
  T be[KS + 1], bo[KS];
  auto load_u = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        be[4 * m + r] = at(pu, m, r, false);
        bo[4 * m + r] = at(pu, m, r, true);
      }
    be[KS] = dense_at(pu, b0 + __mul24(half, st));
  };

  // the table into LDS, 16 bytes per lane, all loads of a thread in flight
  // together, then the first task's u
  {
    constexpr int W = LT.size * (int)sizeof(T) / 16, PER = (W + NT - 1) / NT;
    static_assert(LT.size * sizeof(T) % 16 == 0, "table of whole 16-byte words");
    typedef int __attribute__((ext_vector_type(4))) v4i;
    const v4i* src = (const v4i*)A.tab;
    v4i* dst = (v4i*)tab;
    v4i v[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = src[tid + i * NT < W ? tid + i * NT : W - 1];
    if (task < t_end) {
      locate(task);
      load_u();
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (tid + i * NT < W) dst[tid + i * NT] = v[i];
  }
  lds_barrier();
  if (!live) return;

  // z pencils in a face: every node is a boundary node of the reduced system
  bool clear = FIRST && !ALLP;
  auto clear_faces = [&]() __attribute__((always_inline)) {
    clear = false;
    const int nface = 2 * (n0 + n1) - 4;
    for (int fs = blockIdx.x * NW + wave; fs < nsys * nface; fs += gridDim.x * NW) {
      const int sy = a.sys ? fs / nface : 0, f = fs - sy * nface;
      T* ys = a.ax[0].y + (a.sys ? a.sys[a.act[sy]].off : 0);
      const int g = f - 2 * n1;
      const int ia = f < n1 ? 0 : f < 2 * n1 ? n0 - 1 : 1 + (g >> 1);
      const int ib = f < n1 ? f : f < 2 * n1 ? f - n1 : (g & 1) ? n1 - 1 : 0;
      const int b = (__mul24(ia, n1) + ib) * n2;
      for (int j = lane; j < n2; j += 64) dense_ref(ys, b + j) = T(0);
    }
  };

  // copies of the stride and the lane that the compiler takes for new: offsets
  // are formed where they are used instead of being kept in registers (64 of
  // them) from one phase of a task to the next
  auto renew = [&]() __attribute__((always_inline)) {
    int lv = lane;
    st = stride;
    asm volatile("" : "+s"(st), "+v"(lv));
    li = lv & 15;
    lk = lv >> 4;
  };
  for (; task < t_end; task += t_step) {
    renew();
    const bool nlo = (bm >> (2 * axis)) & 1, nhi = (bm >> (2 * axis + 1)) & 1;
    // raw values -> pair sums and differences; the reduced forms clear the end
    // nodes, rows past R are zeros
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      T lo[4], hi[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) lo[r] = be[4 * m + r], hi[r] = bo[4 * m + r];
      to_rows(lo);
      to_rows(hi);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = row_of(4 * m + r);
        const bool ok = (ALLP || m > 0 || j != 0) && (m + 2 < MT || j < R);
        const T x = ok ? lo[r] : T(0), y = ok ? hi[r] : T(0);
        be[4 * m + r] = x + y;
        bo[4 * m + r] = x - y;
      }
    }
    be[KS] = midv && lk == 0 ? be[KS] + be[KS] : T(0);

    V4 acce[MT], acco[MT];
    T mid;
    // both parts of the product, all row blocks at once, and the middle row's
    // dot product; hook(ks) issues some global loads
    auto product = [&](auto hook) __attribute__((always_inline)) {
      mid = T(0);
#pragma unroll
      for (int m = 0; m < MT; ++m) acce[m] = acco[m] = V4{0, 0, 0, 0};
      T fe[2][MT], fo[2][MT], fm[2];
      auto frags = [&](int ks) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          fe[ks & 1][m] = te[(m * (KS + 1) + ks) * 64 + lane];
          if (ks < KS) fo[ks & 1][m] = to[(m * KS + ks) * 64 + lane];
        }
        if (ks < KS) fm[ks & 1] = amid[line_kmap(ks, lk, F32)];
      };
      frags(0);
#pragma unroll
      for (int ks = 0; ks <= KS; ++ks) {
        if (ks < KS) frags(ks + 1);
        hook(ks);
        if (ks < KS || midv) {
#pragma unroll
          for (int m = 0; m < MT; ++m) acce[m] = Mfma<T>::mac(fe[ks & 1][m], be[ks], acce[m]);
        }
        if (ks < KS) {
#pragma unroll
          for (int m = 0; m < MT; ++m) acco[m] = Mfma<T>::mac(fo[ks & 1][m], bo[ks < KS ? ks : 0], acco[m]);
          mid += fm[ks & 1] * bo[ks < KS ? ks : 0];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (midv) mid = rows_sum(mid);
    };

    // first product, K's loads under it
    T klo[KS], khi[KS], kmid = T(0);
    product([&](int ks) __attribute__((always_inline)) {
      if (DER && !DMUL) return;
      if (ks < KS) {
        klo[ks] = at(pk, ks / 4, ks % 4, false);
        khi[ks] = at(pk, ks / 4, ks % 4, true);
      } else {
        kmid = dense_at(pk, b0 + __mul24(half, st));
      }
    });
    if (clear) clear_faces();
    renew();

    // store one block's rows: nodes i and N - i
    T ylo[FIRST ? 1 : KS], yhi[FIRST ? 1 : KS], zlo[YADD ? 8 : 1], zhi[YADD ? 8 : 1], ymid = T(0);
    auto store = [&](int m, T (&lo)[4], T (&hi)[4]) __attribute__((always_inline)) {
      to_lines(lo);
      to_lines(hi);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = CG ? 16 * m + li : row_of(4 * m + r);
        const int bb = CG ? bp[CG ? r : 0] : b0;
        const bool on = CG ? bb >= 0 : valid && (!FULL || (fl & PF_TIN));
        if (!on || i >= RM) continue;
        const int olo = bb + __mul24(i, st), ohi = bb + __mul24(N - i, st);
        if (!ALLP && (m > 0 ? false : i == 0)) {
          // the reduced forms' end nodes: zeros, written along z
          if (CG) {
            dense_ref(py, olo) = T(0);
            dense_ref(py, ohi) = T(0);
          }
          continue;
        }
        if (FULL && m == 0 && i == 0) continue;
        T x = lo[r], y = hi[r];
        if (DMUL) x *= klo[4 * m + r], y *= khi[4 * m + r];  // (the loads are in the stores' order)
        if (!FIRST) x += ylo[FIRST ? 0 : 4 * m + r], y += yhi[FIRST ? 0 : 4 * m + r];
        if (YADD) x += zlo[YADD ? (4 * m + r) % 8 : 0], y += zhi[YADD ? (4 * m + r) % 8 : 0];
        dense_ref(py, olo) = x;
        if (2 * i != N) dense_ref(py, ohi) = y;
      }
    };

    if (DER) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        T lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) lo[r] = acco[m][r] + acce[m][r], hi[r] = acco[m][r] - acce[m][r];
        store(m, lo, hi);
      }
      if (midv && valid && lk == 0) dense_ref(py, b0 + __mul24(half, st)) = DMUL ? mid * kmid : mid;
    } else {
      // the first product's rows 0 and N, at the lanes lk = 0, broadcast over lk
      T u0 = T(0), uN = T(0);
      const bool lift = LIFT && (nlo || nhi);
      auto ends = [&](T& x, T& y) __attribute__((always_inline)) {  // E [x, y] with E the inverse of the end-value block (rows, or columns for TRA)
        T e0, e1, e2, e3;
        if (A.rinv) {
          const int qv = valid ? q : npen - 1, qa = fast_div(qv, nbi, A.inv_nbi);
          const T* e = A.rinv + 4 * ((po + qa) * nb + po + qv - __mul24(qa, nbi));
          e0 = e[0], e1 = e[1], e2 = e[2], e3 = e[3];
        } else {
          const T* e = linv + 4 * ((nlo ? 1 : 0) + (nhi ? 2 : 0));
          e0 = e[0], e1 = e[1], e2 = e[2], e3 = e[3];
        }
        const T p = TRA ? e0 * x + e2 * y : e0 * x + e1 * y;
        const T s = TRA ? e1 * x + e3 * y : e2 * x + e3 * y;
        x = p;
        y = s;
      };
      if (lift) {
        // end values of the homogeneous lift (Section 2.3.1): M [u0, uN] = -[s0, sN]
        const T s0 = acco[0][0] + acce[0][0], sN = acco[0][0] - acce[0][0];
        u0 = __shfl(s0, li, 64);
        uN = __shfl(sN, li, 64);
        ends(u0, uN);
        u0 = -u0;
        uN = -uN;
      }
      if (FULL && lk == 0) {
        // the face rows at the end nodes this axis owns: u on a Dirichlet face,
        // the outward derivative plus sigma u on a Neumann one
        const T dlo = acco[0][0] + acce[0][0], dhi = acco[0][0] - acce[0][0];
        if (fl & PF_OWN_LO) {
          T v = dense_at(pu, b0);
          if (nlo) v = (A.slo + (A.rlo ? A.rlo[q] : T(0))) * v - dlo;
          dense_ref(A.yb, b0) = v;
        }
        if (fl & PF_OWN_HI) {
          const int o = b0 + __mul24(N, st);
          T v = dense_at(pu, o);
          if (nhi) v = dhi + (A.shi + (A.rhi ? A.rhi[q] : T(0))) * v;
          dense_ref(A.yb, o) = v;
        }
      }

      // flux K (M u) (+ C v) as the second product's operand; with the lift, M u
      // gains u0 M[:][0] + uN M[:][N], whose row N-i is -(u0 M[i][N] + uN M[i][0])
      T clo[JAC ? 4 : 1], chi[JAC ? 4 : 1];
      auto load_c = [&](int m) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < (JAC ? 4 : 0); ++r) {
          clo[JAC ? r : 0] = at(A.c, m, r, false);
          chi[JAC ? r : 0] = at(A.c, m, r, true);
        }
      };
      if (JAC) load_c(0);
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        T lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) lo[r] = klo[4 * m + r], hi[r] = khi[4 * m + r];
        to_rows(lo);
        to_rows(hi);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          T x = acco[m][r] + acce[m][r], y = acco[m][r] - acce[m][r];
          if (lift) {
            const int i = row_of(4 * m + r);
            const T c0 = dc0[i], cN = dcN[i];
            x += u0 * c0 + uN * cN;
            y -= u0 * cN + uN * c0;
          }
          lo[r] *= x;
          hi[r] *= y;
        }
        if constexpr (JAC) {
          T c[4], d[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) c[r] = clo[r], d[r] = chi[r];
          if (m + 1 < MT) load_c(m + 1);
          to_rows(c);
          to_rows(d);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            // the lifted direction itself
            const bool end = m == 0 && row_of(r) == 0;
            const T ev = be[4 * m + r], od = bo[4 * m + r];
            lo[r] += c[r] * (end ? u0 : T(0.5) * (ev + od));
            hi[r] += d[r] * (end ? uN : T(0.5) * (ev - od));
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = row_of(4 * m + r);
          const bool pair = 2 * i != N;  // not the middle node (then hi repeats lo, with the other sign of the odd part)
          be[4 * m + r] = pair ? lo[r] + hi[r] : lo[r] + lo[r];
          bo[4 * m + r] = pair ? lo[r] - hi[r] : T(0);
          if (m + 2 >= MT && i >= RM) be[4 * m + r] = bo[4 * m + r] = T(0);
        }
      }
      {
        T m = mid;
        if (lift) m += u0 * dc0[half] + uN * dcN[half];
        m *= kmid;
        if (JAC) {
          if (midv) m += dense_at(A.c, b0 + __mul24(half, st)) * (T(0.5) * __shfl(be[KS], li, 64));
        }
        be[KS] = midv && lk == 0 ? m + m : T(0);
      }

      renew();

      // divergence part, with the loads of the partial sums under it (of yadd
      // block by block with the stores: registers)
      auto load_z = [&](int m) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          zlo[YADD ? (4 * m + r) % 8 : 0] = at(a.yadd, m, r, false);
          zhi[YADD ? (4 * m + r) % 8 : 0] = at(a.yadd, m, r, true);
        }
      };
      product([&](int ks) __attribute__((always_inline)) {
        if (FIRST) return;
        if (ks < KS) {
          ylo[FIRST ? 0 : ks] = at(py, ks / 4, ks % 4, false);
          yhi[FIRST ? 0 : ks] = at(py, ks / 4, ks % 4, true);
        } else {
          ymid = dense_at(py, b0 + __mul24(half, st));
          if (YADD) ymid += dense_at(a.yadd, b0 + __mul24(half, st));
          if (YADD) load_z(0);
        }
      });

      renew();
      const bool tl = TRA && (nlo || nhi);
      if (tl) {
        // transposed lift: mu = M^{-T} [z_0, z_N]; interior -= mu0 D[0][:] + muN D[N][:]
        // (D[0][j] and D[N][j] are the end columns of the table of D^T)
        const T z0 = acco[0][0] + acce[0][0], zN = acco[0][0] - acce[0][0];
        u0 = __shfl(z0, li, 64);
        uN = __shfl(zN, li, 64);
        ends(u0, uN);
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        if (YADD && m + 1 < MT) load_z(m + 1);
        T lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          lo[r] = acco[m][r] + acce[m][r];
          hi[r] = acco[m][r] - acce[m][r];
          if (tl) {
            const int i = row_of(4 * m + r);
            const T d0 = dc0[i], dN = dcN[i];
            lo[r] -= u0 * d0 + uN * dN;
            hi[r] += u0 * dN + uN * d0;
          }
        }
        store(m, lo, hi);
      }
      if (midv && valid && lk == 0 && (!FULL || (fl & PF_TIN))) {
        T m = mid;
        if (tl) m -= u0 * dc0[half] + uN * dcN[half];
        dense_ref(py, b0 + __mul24(half, st)) = FIRST ? m : m + ymid;
      }
    }
    if (task + t_step < t_end) {
      locate(task + t_step);
      load_u();
    }
  }
  if (clear) clear_faces();
}

}  // namespace cheb

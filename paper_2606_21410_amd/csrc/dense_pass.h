// Matrix-core pass along one axis, for axes with N <= 256: the reduced
// operator's axis term and its transpose, the Newton Jacobian's axis term, the
// full operator's rows and the plain derivative.
//
// For every pencil of the pass (D the collocation derivative of the axis,
// Section 2.2; L the homogeneous lift of the pencil's end values from the face
// rows, Section 2.3.1)
//   LINE_REDUCED  y_int (+)= [ D (K .* (D L u_int)) ]_int
//   LINE_TRANSP   y_int (+)= L^T D^T (K .* (D^T w)),   w zero at the two ends
//   LINE_JAC      y_int (+)= [ D (K .* (D L v) + C .* L v) ]_int   (FP64)
//   LINE_FULL     y_int (+)= [ D (K .* (D u)) ]_int, and the face rows' values
//                 at the end nodes the axis owns (all pencils)
//   LINE_DERIV    y = D u, or D^T u with the transposed table (all pencils)
//   LINE_DMUL     y = K .* D u (all pencils; FP64)
// The derivative of a tile of pencils is a small dense contraction, so it runs
// on the matrix cores: D cut into 16-row blocks, one block per wave, its
// fragments in that wave's registers for the whole launch.
//
// Even-odd split: D (and D^T) is centro-antisymmetric, M[N-i][N-j] = -M[i][j],
// so with e_j = u_j + u_{N-j} and o_j = u_j - u_{N-j} over the pairs
// j < R = N/2 + 1 (an even N has the self-mirrored middle node j = N/2, with
// e = 2 u and o = 0)
//   (Mu)_i = s_i + d_i,  (Mu)_{N-i} = s_i - d_i,   i < R,
//   s_i = sum_j Ao[i][j] o_j,   d_i = sum_j Ae[i][j] e_j,
//   Ao[i][j] = (M[i][j] - M[i][N-j]) / 2,  Ae[i][j] = (M[i][j] + M[i][N-j]) / 2
// (Ae[i][N/2] = M[i][N/2] / 2), which halves the multiply-adds.  N is a launch
// argument; the kernel is compiled per number of row blocks MT, and rows and
// k-steps past R meet zero fragments.
//
// Two kernels.  With up to four row blocks one wave computes every row of its
// pencils (line_wave.h).  Past that the fragments and accumulators of one wave do
// not fit its registers, and k_line_pass below gives each wave of a workgroup one
// row block, with the split tile shared through LDS; launches of few tasks on
// three or four row blocks take it too (launch_line_mt).
//
// k_line_pass: only that operand, e / o, is in LDS.  What belongs to an output
// row (K, C, the partial sums y, the stores) goes between memory and the
// registers of the lane whose accumulators hold the row: along x and y the
// pencils are the accumulator columns, along z the nodes are (the two operands
// of the matrix instruction exchanged), so 16 consecutive lanes always meet 16
// consecutive values.  Bound by the matrix cores: at 257^3 in FP64 the products
// take 21k of a tile's 26k cycles, 16.6k of them the instructions themselves;
// an apply takes 0.56 ms, where the FFT route (the route at N > 128 before)
// takes 0.96 ms (FP32: 0.31 against 0.65 ms; a size without a compiled FFT,
// 179^3: 0.23 against 5.3 ms).
#pragma once

#include "dev_common.h"
#include "pencil.h"

namespace cheb {

enum LineMode { LINE_REDUCED = 0, LINE_TRANSP = 1, LINE_JAC = 2, LINE_FULL = 3, LINE_DERIV = 4, LINE_DMUL = 5 };

constexpr int kLineMaxN = 256;  // 8 row blocks
constexpr int kLineMaxMT = 8;

__host__ __device__ constexpr bool line_supported(int N) { return N >= 2 && N <= kLineMaxN; }

// row pairs, row blocks, and whether the lone middle row of an even N goes to
// the vector ALUs (when it would open a 16-row block of its own; a table of mt
// blocks may have one more than line_mt(N))
__host__ __device__ constexpr int line_pairs(int N) { return N / 2 + 1; }
__host__ __device__ constexpr int line_mt(int N) { return N % 32 == 0 ? N / 32 : (line_pairs(N) + 15) / 16; }
__host__ __device__ constexpr bool line_midv(int N, int mt) { return N == 32 * mt; }

// k index of step ks for lane group lk = lane / 16.  Up to four blocks
// (k_line_wave) it is the row that the accumulator of the type holds in register
// ks % 4 of block ks / 4; past those rows are read from LDS in natural order
constexpr int kWaveMaxMT = 4;
__host__ __device__ constexpr int line_kmap(int ks, int lk, bool f32) {
  return f32 ? 16 * (ks / 4) + 4 * lk + (ks % 4) : 4 * ks + lk;
}

// fragment table of one matrix (mt = line_mt(N) row blocks): Ae [mt][4 mt + 1][64],
// Ao [mt][4 mt][64] in lane order, the middle row of Ao (16 mt), the end
// columns M[i][0] and M[i][N] for i <= 16 mt, then the lift's end-value inverse
// E = M^{-1} (row-major 2 x 2) for each pair of face types, index 1 for a
// Neumann lo face plus 2 for a Neumann hi one (1 / m00 or 1 / mNN alone, the
// other entries 0, with one of them)
struct LineTab {
  int off_o, off_mid, off_c0, off_cN, off_lift, size;
};
__host__ __device__ constexpr LineTab line_tab(int mt) {
  LineTab t{};
  t.off_o = mt * (4 * mt + 1) * 64;
  t.off_mid = t.off_o + mt * 4 * mt * 64;
  t.off_c0 = t.off_mid + 16 * mt;
  t.off_cN = t.off_c0 + 16 * mt + 1;
  t.off_lift = t.off_cN + 16 * mt + 1;
  t.size = (t.off_lift + 16 + 3) / 4 * 4;
  return t;
}

// LDS of one workgroup (elements of T, then 2 x C ints twice): the split tile
// (e rows, o rows), middle row, end columns, per-pencil end values
__host__ __device__ constexpr int line_lds_elems(int MT) {
  return (16 * MT + 4 + 16 * MT) * 17 + 16 * MT + 2 * (16 * MT + 1) + 16 + 2 * 16;
}
template <typename T>
__host__ __device__ constexpr int line_lds_bytes(int MT) {
  return (line_lds_elems(MT) * (int)sizeof(T) + 15) / 16 * 16 + 4 * 16 * (int)sizeof(int);
}

// element i of a system's field at base (uniform): a system's field stays
// below 4 GiB, so the byte offset fits 32 bits and the address is a scalar
// base plus one vector offset register
template <typename T>
__device__ __forceinline__ T dense_at(const T* base, int i) {
  return *(const T*)((const char*)base + (unsigned)i * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ T& dense_ref(T* base, int i) {
  return *(T*)((char*)base + (unsigned)i * (unsigned)sizeof(T));
}

// lane move across a DPP pattern (quad permutation, half-row or row mirror)
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// sum over aligned groups of G <= 16 consecutive lanes (within one DPP row),
// left in every lane of the group: swaps within pairs and quads, then the
// half-row mirror pairs the two quads of each 8, the row mirror the two 8s
template <int G, typename T>
__device__ __forceinline__ T row_sum(T v) {
  static_assert(G == 1 || G == 2 || G == 4 || G == 8 || G == 16, "row_sum: group of 1 to 16 lanes");
  if (G >= 2) v += dpp_move<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  if (G >= 4) v += dpp_move<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  if (G >= 8) v += dpp_move<0x141>(v);  // row_half_mirror
  if (G >= 16) v += dpp_move<0x140>(v); // row_mirror
  return v;
}

__host__ __device__ constexpr int pow2_floor(int x) {
  int p = 1;
  while (2 * p <= x) p *= 2;
  return p;
}

// one system of a batched pass (same n and box as the others): its offset in
// the packed fields, the offset of its conductivity in the packed K (systems
// given the same K, e.g. the load cases of one microstructure, share one copy)
// and its face types
struct DenseSys {
  long long off;
  long long koff;
  int bcmask;
  int pad_;
};

// one axis of a launch
template <typename T>
struct LineAxis {
  const T* tab;  // fragment table of D (or D^T)
  T* y;          // output (single system; batches: the packed base)
  T* yb;         // LINE_FULL: where the face rows' values go
  const T* c;    // LINE_JAC: the axis' coefficient C of the lifted direction; null otherwise
  // per-node Robin coefficients: each pencil's own end-block inverse, 4 entries
  // per pencil of the axis (face numbering), laid out as i00, i0N, iN0, iNN
  // with 1 / m00 or 1 / mNN in place of the inverse when one end is Dirichlet;
  // null without them (always for batches)
  const T* rinv;
  // LINE_FULL: the coefficients themselves at the lo and hi face's nodes (face
  // numbering; null without per-node ones), and the faces' own
  const T *rlo, *rhi;
  T slo, shi;
  int axis;
  int N;
  float inv_nbi, inv_pairs;  // 1 / (pencils per row of the pass), 1 / line_pairs(N)
};

template <typename T>
struct LineArgs {
  const int* gate;  // null, or a device flag: the pass does nothing while it reads 0
  const T* u;  // single system (sys == nullptr)
  const T* K;
  const DenseSys* sys;  // batched: system table (device) and the active systems' indices
  const int* act;
  int nact;
  int n[3];
  int bcmask;  // face types of the single system
  // nseg = 2 (first passes of a single system, along x and y): the launch serves
  // two axes, ax[0] and ax[1], each into its own output; workgroup b takes axis
  // ax[(b >> 3) & 1], so every XCD holds workgroups of both (the grid is a
  // multiple of 16)
  int nseg;
  int wpw;  // k_line_wave: waves of a workgroup that take tasks
  int tasks;  // 16-pencil tasks of the launch, of x and y together where they can share one
  // accumulating pass along the unit-stride axis: y += yadd + this pass (yadd
  // is the second output of a two-axis launch); unused by the other passes
  const T* yadd;
  LineAxis<T> ax[2];
};

// entry i of the active-system list, read through the constant address space
// (scalar loads; the tables are not written while a pass runs)
template <typename T>
__device__ inline DenseSys dense_sys_at(const LineArgs<T>& a, int i) {
  typedef const __attribute__((address_space(4))) int ci4;
  typedef const __attribute__((address_space(4))) long long cl4;
  const DenseSys* e = a.sys + ((ci4*)a.act)[i];
  DenseSys s;
  s.off = *(cl4*)&e->off;
  s.koff = *(cl4*)&e->koff;
  s.bcmask = *(ci4*)&e->bcmask;
  s.pad_ = 0;
  return s;
}

// waves per SIMD that the register budget is held to: as many as compile
// without spills (a spilled register's reload waits for every load in flight),
// except FP32 with six blocks: its accumulating z passes spill 2 and 6 registers
// with four, and are faster so (193^3 apply 131 us, 144 with three)
template <typename T>
__host__ __device__ constexpr int line_waves(int MT) {
  return sizeof(T) == sizeof(double) ? 2 : MT <= 6 ? 4 : 3;
}

// q / d for 0 <= q < 2^24 with inv = 1 / d rounded to FP32
__device__ __forceinline__ int fast_div(int q, int d, float inv) {
  int t = (int)((float)q * inv);
  const int r = q - __mul24(t, d);
  t += r >= d ? 1 : 0;
  t -= r < 0 ? 1 : 0;
  return t;
}

// Persistent: each workgroup (MT waves, wave mt owning row block mt) walks its
// XCD's contiguous range of tiles of 16 pencils (in a two-axis launch,
// within its axis' half of the grid).  CG: the axis is the unit-stride one (z).
// In the reduced forms the boundary nodes' zeros are written along z alone: the
// first pass clears the z pencils that lie in a face (contiguous runs), the z
// pass the ends of the others; x and y passes write interior nodes only.
template <typename T, int MT, int MODE, bool FIRST, bool CG>
__global__ __launch_bounds__(64 * MT, line_waves<T>(MT)) void k_line_pass(LineArgs<T> a) {
  if (a.gate && !*a.gate) return;
  typedef typename Mfma<T>::v4 V4;
  constexpr bool FULL = MODE == LINE_FULL, DMUL = MODE == LINE_DMUL, DER = MODE == LINE_DERIV || DMUL;
  constexpr bool JAC = MODE == LINE_JAC;
  constexpr bool LIFT = MODE == LINE_REDUCED || MODE == LINE_JAC;  // in-pencil lift after the first product
  constexpr bool TRA = MODE == LINE_TRANSP;
  constexpr bool ALLP = FULL || DER;   // every pencil, end values of u included
  constexpr bool YADD = CG && !FIRST;  // the last pass of a two-axis apply adds yadd
  static_assert(!DER || FIRST, "derivatives do not accumulate");
  constexpr int C = 16, SC = C + 1;  // odd LDS row stride
  constexpr int NT = 64 * MT;
  constexpr int EROWS = 16 * MT + 4, OB = EROWS * SC;
  constexpr int KS = 4 * MT;             // odd-part k-steps; the even part has one more (middle row)
  constexpr int EPP = 4 + 1;         // node pairs staged per thread
  // the next tile's u into registers during the second product: one workgroup
  // fills a CU and nothing else would cover its latency (without it at 257^3,
  // FP64: 754 against 590 us); the last pass at the largest sizes has no
  // registers left for it
  constexpr bool PREF = !(sizeof(T) == 8 && YADD && MT > 6);
  constexpr int LPC = pow2_floor(NT / C) < 16 ? pow2_floor(NT / C) : 16;  // lanes per column of the middle row
  constexpr LineTab LT = line_tab(MT);

  extern __shared__ __align__(16) unsigned char smem[];
  T* U = (T*)smem;
  T* amid = U + (EROWS + 16 * MT) * SC;
  T* dc0 = amid + 16 * MT;            // end columns M[i][0], M[i][N], i <= N/2
  T* dcN = dc0 + 16 * MT + 1;
  T* linv = dcN + 16 * MT + 1;        // end-value inverses of the lift
  T* cend = linv + 16;                // per pencil: end values of the lift / multipliers of its transpose
  int(*cbase)[C] = (int(*)[C])(smem + (line_lds_elems(MT) * sizeof(T) + 15) / 16 * 16);
  int(*cflag)[C] = cbase + 2;

  const int tid = threadIdx.x, lane = tid & 63;
  const int mt = __builtin_amdgcn_readfirstlane(tid >> 6);
  int li = lane & 15, lk = lane >> 4, tq = tid / C, tc = tid % C;
  const int seg = a.nseg == 2 ? (blockIdx.x >> 3) & 1 : 0;
  const int vb = a.nseg == 2 ? (int)(((blockIdx.x >> 4) << 3) | (blockIdx.x & 7)) : (int)blockIdx.x;
  const int vg = a.nseg == 2 ? (int)(gridDim.x >> 1) : (int)gridDim.x;
  const LineAxis<T> A = seg ? a.ax[1] : a.ax[0];
  const int axis = A.axis, N = A.N, n = N + 1;
  const int R = line_pairs(N), KO = (N & 1) ? R : R - 1;
  const bool midv = line_midv(N, MT);
  const int RM = midv ? R - 1 : R;            // rows on the matrix cores
  // steps that hold columns of the axis (in the FP32 order of line_kmap a block's
  // four steps share its columns)
  constexpr bool K32 = sizeof(T) == sizeof(float) && MT <= kWaveMaxMT;
  auto steps = [&](int cols) {
    const int last = cols - 16 * (MT - 1);
    return !K32 ? (cols + 3) >> 2 : last > 16 ? KS + 1 : KS - 4 + min(max(last, 0), 4);
  };
  const int nke = steps(R), nko = steps(KO);
  const int half = N >> 1;
  const int n0 = a.n[0], n1 = a.n[1], n2 = a.n[2];
  const int stride = CG ? 1 : axis == 1 ? n2 : n1 * n2;
  constexpr int po = ALLP ? 0 : 1;  // transverse offset of the first pencil
  const int na = axis == 0 ? n1 : n0, nb = axis == 2 ? n1 : n2;
  const int nbi = nb - 2 * po;
  const int npen = (na - 2 * po) * nbi;
  const int tps = (npen + C - 1) / C;  // tiles per system
  const int nsys = a.sys ? a.nact : 1;
  const int ntiles = nsys * tps;

  // XCD-aware tile order: workgroups are dealt round-robin to the 8 XCDs, so
  // workgroup b serves a contiguous range of tiles of XCD b % 8 and tiles that
  // share cache lines at their edges meet in the same L2
  int t_step = vg, t_end = ntiles, tile = vb;
  if ((vg & 7) == 0 && ntiles >= vg) {
    const int per = (ntiles + 7) >> 3;
    const int x = vb & 7;
    tile = x * per + (vb >> 3);
    t_step = vg >> 3;
    t_end = min(ntiles, (x + 1) * per);
  }

  // index of tile t within its system
  auto tile_in = [&](int t) { return a.sys ? t % tps : t; };
  // linear offset of pencil c of tile t (-1 past the last one) and, for the
  // full rows, its flags
  auto columns = [&](int t, int slot) {
    if (tid < C) {
      const int q = tile_in(t) * C + tid;
      int b = -1, fl = 0;
      if (q < npen) {
        const int qa = fast_div(q, nbi, A.inv_nbi);
        const int ia = po + qa, ib = po + q - __mul24(qa, nbi);
        b = axis == 2 ? (ia * n1 + ib) * n2 : axis == 1 ? ia * n1 * n2 + ib : ia * n2 + ib;
        if (FULL) {
          long long bb;
          fl = pencil_flags(axis, q, npen, n0, n1, n2, a.bcmask, &bb);
        }
      }
      cbase[slot][tid] = b;
      if (FULL) cflag[slot][tid] = fl;
    }
  };
  // face numbering of pencil q (index among all pencils along the axis)
  auto face_index = [&](int q) {
    return q < npen ? (po + q / nbi) * nb + po + q % nbi : 0;
  };

  // Staged pairs of this thread: along x and y pencil tid % C, rows tid / C + q
  // NT / C (a fixed step); along z consecutive lanes take consecutive nodes of
  // a pencil, so row and pencil are kept per step.  Rows past R are staged as
  // zeros; step EPP - 1 is the lone middle row (midv), the other lanes writing
  // zeros to the spare rows behind it.
  int pjc[CG ? EPP : 1];
  if (CG) {
#pragma unroll
    for (int q = 0; q < EPP; ++q) {
      const int p = tid + q * NT, c = fast_div(p, R, A.inv_pairs);
      pjc[CG ? q : 0] = c < C ? ((p - c * R) << 8) | c : C;  // past the tile: node 0 of pencil 0 into the padding column
    }
  }
  auto stage_row = [&](int q) {
    if (CG) return pjc[CG ? q : 0] >> 8;
    return q == EPP - 1 ? half : tq + q * (NT / C);
  };
  auto stage_col = [&](int q) { return CG ? pjc[CG ? q : 0] & 255 : tc; };

  // row i of accumulator register r of this lane: along x and y the rows of
  // row(lk, r) with pencil li, along z node li with the pencils of row(lk, r).
  // Rows past R read a node of the pencil and store nothing.
  auto node_of = [&](int r) { return 16 * mt + (CG ? li : Mfma<T>::row(lk, r)); };
  auto node_at = [&](int r) {
    const int i = node_of(r);
    return i < N ? i : N;
  };
  auto col_of = [&](int r) { return CG ? Mfma<T>::row(lk, r) : li; };

  // middle row (midv): LPC lanes per column
  int lc = tid / LPC, lg = tid % LPC, lcc = lc < C ? lc : 0;

  // pointers and face types of the system that owns a tile
  struct Sys {
    const T *u, *k;
    T* y;
    int bm;
  };
  auto system_of = [&](int t) {
    Sys s{a.u, a.K, A.y, a.bcmask};
    if (a.sys) {
      const DenseSys d = dense_sys_at(a, t / tps);
      s.u = a.u + d.off;
      s.k = a.K + d.koff;
      s.y = A.y + d.off;
      s.bm = d.bcmask;
    }
    return s;
  };
  auto base_of = [&](int sl, int c) {
    const int b = cbase[sl][c];
    return b > 0 ? b : 0;
  };

  // u of one tile into registers, pair by pair: load l is the lower (even l) or
  // upper node of pair l / 2.  Every load is issued, and with st = 0 all lanes
  // read the same two nodes (no next tile), so the waits stay exact.
  T ulo[EPP], uhi[EPP];
  auto load_u = [&](int l, const T* pu, int sl, int st) {
    const int q = l >> 1;
    const int c = stage_col(q);
    int j = stage_row(q);
    if (!CG && q < EPP - 1) j = j < N ? j : N;
    const int b = st ? base_of(sl, c < C ? c : 0) : 0;
    if (l & 1) uhi[q] = dense_at(pu, b + __mul24(N - j, st));
    else ulo[q] = dense_at(pu, b + __mul24(j, st));
  };

  // prologue: the first tile's u in flight before this wave's fragments, the
  // table's vectors and the zeros of the boundary
  int slot = 0;
  columns(tile, 0);
  lds_barrier();
  if (tile < t_end) {
    const Sys s = system_of(tile);
#pragma unroll
    for (int l = 0; l < 2 * EPP; ++l) load_u(l, s.u, 0, stride);
  }
  // z pencils in a face: every node is a boundary node of the reduced system
  auto clear_faces = [&]() {
    const int nface = 2 * (n0 + n1) - 4;
    for (int fs = blockIdx.x; fs < nsys * nface; fs += gridDim.x) {
      const int sy = a.sys ? fs / nface : 0, f = fs - sy * nface;
      T* ys = a.ax[0].y + (a.sys ? a.sys[a.act[sy]].off : 0);
      const int g = f - 2 * n1;
      const int ia = f < n1 ? 0 : f < 2 * n1 ? n0 - 1 : 1 + (g >> 1);
      const int ib = f < n1 ? f : f < 2 * n1 ? f - n1 : (g & 1) ? n1 - 1 : 0;
      const int b = (__mul24(ia, n1) + ib) * n2;
      for (int j = tid; j < n2; j += NT) dense_ref(ys, b + j) = T(0);
    }
  };
  bool clear = true;
  if (FIRST && !ALLP && tile >= t_end) clear_faces();
  T ae[KS + 1], ao[KS];
#pragma unroll
  for (int ks = 0; ks <= KS; ++ks) ae[ks] = A.tab[(mt * (KS + 1) + ks) * 64 + lane];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) ao[ks] = A.tab[LT.off_o + (mt * KS + ks) * 64 + lane];
  if (tid < 16 * MT) amid[tid] = A.tab[LT.off_mid + tid];
  if (tid < 16) linv[tid] = A.tab[LT.off_lift + tid];
  for (int i = tid; i < R; i += NT) {
    dc0[i] = A.tab[LT.off_c0 + i];
    dcN[i] = A.tab[LT.off_cN + i];
  }
  if (CG) {
    // rows that no pair is staged into (they meet zero fragments and must be finite)
    for (int e = tid; e < (EROWS - R) * SC; e += NT) U[R * SC + e] = T(0);
    for (int e = tid; e < (16 * MT - KO) * SC; e += NT) U[OB + KO * SC + e] = T(0);
  }
  for (; tile < t_end; tile += t_step, slot ^= 1) {
    const bool more = tile + t_step < t_end;
    const int nxt = more ? tile + t_step : tile;
    lds_barrier();  // the previous tile's readers of U are done; cbase[slot] is there
    const Sys S = system_of(tile);
    const T *pu = S.u, *pk = S.k;
    T* py = S.y;
    T* pyb = A.yb;
    const int bct = (S.bm >> (2 * axis)) & 3;
    const bool nlo = bct & 1, nhi = bct & 2;
    // copies of the stride and the lane that the compiler takes for new in every
    // tile: offsets are formed where they are used instead of being kept in
    // registers over the whole loop
    int st = stride, tv = tid;
    asm volatile("" : "+s"(st), "+v"(tv));
    li = tv & 15;
    lk = (tv >> 4) & 3;
    tq = tv / C;
    tc = tv % C;
    lc = tv / LPC;
    lg = tv % LPC;
    lcc = lc < C ? lc : 0;
    // K (and C) at this lane's accumulator rows, needed after the first product
    // and requested between its steps
    T klo[4], khi[4], clo[JAC ? 4 : 1], chi[JAC ? 4 : 1], kmid = T(0), cmid = T(0);
    const int bmid0 = cbase[slot][lcc];
    const int bmid = (bmid0 > 0 ? bmid0 : 0) + __mul24(half, st);
    int cb[CG ? 4 : 1];  // first nodes of this lane's accumulator pencils (negative past the last)
#pragma unroll
    for (int r = 0; r < (CG ? 4 : 1); ++r) cb[r] = cbase[slot][col_of(r)];
    auto load_k = [&](int r) {
      const int b0 = cb[CG ? r : 0], b = b0 > 0 ? b0 : 0, i = node_at(r);
      const int olo = b + __mul24(i, st), ohi = b + __mul24(N - i, st);
      klo[r] = dense_at(pk, olo);
      khi[r] = dense_at(pk, ohi);
      if (JAC) {
        clo[JAC ? r : 0] = dense_at(A.c, olo);
        chi[JAC ? r : 0] = dense_at(A.c, ohi);
      }
      if (r == 3 && midv) {
        kmid = dense_at(pk, bmid);
        if (JAC) cmid = dense_at(A.c, bmid);
      }
    };
    // the partial sums this pass adds to, needed after the second product
    T ylo[4], yhi[4], zlo[YADD ? 4 : 1], zhi[YADD ? 4 : 1], ymid = T(0), zmid = T(0);
    auto load_y = [&](int r) {
      const int b0 = cb[CG ? r : 0], b = b0 > 0 ? b0 : 0, i = node_at(r);
      const int olo = b + __mul24(i, st), ohi = b + __mul24(N - i, st);
      ylo[r] = dense_at(py, olo);
      yhi[r] = dense_at(py, ohi);
      if (YADD) {
        zlo[YADD ? r : 0] = dense_at(a.yadd, olo);
        zhi[YADD ? r : 0] = dense_at(a.yadd, ohi);
      }
      if (r == 3 && midv) {
        ymid = dense_at(py, bmid);
        if (YADD) zmid = dense_at(a.yadd, bmid);
      }
    };
    // registers -> LDS in split form; the reduced forms clear the end nodes
#pragma unroll
    for (int q = 0; q < EPP; ++q) {
      const int j = stage_row(q), c = stage_col(q);
      T x = ulo[q], y = uhi[q];
      if (!ALLP && j == 0) x = y = T(0);
      if (CG) {
        U[j * SC + c] = x + y;
        if (j < KO) U[OB + j * SC + c] = x - y;
      } else if (q < EPP - 1) {
        if (j >= R) x = y = T(0);
        U[j * SC + c] = x + y;
        U[OB + j * SC + c] = x - y;
      } else {
        if (!(midv && tq == 0)) x = y = T(0);
        U[(16 * MT + (tq < 3 ? tq : 3)) * SC + c] = x + y;
      }
    }
    columns(nxt, slot ^ 1);
    lds_barrier();
    if (FIRST && !ALLP && clear) {
      clear = false;  // behind this tile's loads, which would otherwise wait for the stores
      clear_faces();
    }

    V4 acce, acco;
    T mid = T(0);
    // both parts of the product with the split tile, and the middle row's dot
    // product; hook(ks) issues some global loads at each k-step
    auto product = [&](auto hook) {
      if (midv) {
        mid = T(0);
#pragma unroll
        for (int q = 0; q < 16 * MT / LPC; ++q) mid += amid[lg + q * LPC] * U[OB + (lg + q * LPC) * SC + lcc];
        mid = row_sum<LPC>(mid);
      }
      acce = V4{0, 0, 0, 0};
      acco = V4{0, 0, 0, 0};
      // the operands of the step two ahead are read while a step multiplies; the
      // scheduling barriers keep it so (left alone, the compiler reads the whole
      // column ahead and runs out of registers)
      // row line_kmap(ks, lk); of the middle row's step only lane group 0 meets
      // entries that are not zero
      const T* Ue = U + (K32 ? 4 * lk : lk) * SC + li;
      T be[3], bo[3];
      auto operands = [&](int ks) {
        const int k0 = K32 ? line_kmap(ks, 0, true) : 4 * ks;
        be[ks % 3] = Ue[k0 * SC];
        if (ks < KS) bo[ks % 3] = Ue[OB + k0 * SC];
      };
      operands(0);
      operands(1);
#pragma unroll
      for (int ks = 0; ks <= KS; ++ks) {
        if (ks + 2 <= KS) operands(ks + 2);
        hook(ks);
        // the last steps of a block are skipped when the axis has no rows there
        if (ks < KS - 3 || ks < nke) {
          acce = CG ? Mfma<T>::mac(be[ks % 3], ae[ks], acce) : Mfma<T>::mac(ae[ks], be[ks % 3], acce);
        }
        if (ks < KS && (ks < KS - 3 || ks < nko)) {
          const T f = ao[ks < KS ? ks : 0];
          acco = CG ? Mfma<T>::mac(bo[ks % 3], f, acco) : Mfma<T>::mac(f, bo[ks % 3], acco);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    product([&](int ks) {
      if ((!DER || DMUL) && ks < 4) load_k(ks);
    });

    if (DER) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int b = cb[CG ? r : 0], i = node_of(r);
        if (b >= 0 && i < RM) {
          const T s = acco[r], d = acce[r];
          dense_ref(py, b + __mul24(i, st)) = DMUL ? (s + d) * klo[r] : s + d;
          if (2 * i != N) dense_ref(py, b + __mul24(N - i, st)) = DMUL ? (s - d) * khi[r] : s - d;
        }
      }
      if (midv && lc < C && lg == 0 && bmid0 >= 0) dense_ref(py, bmid) = DMUL ? mid * kmid : mid;
      if (more) {
        const Sys s = system_of(nxt);
#pragma unroll
        for (int l = 0; l < 2 * EPP; ++l) load_u(l, s.u, slot ^ 1, st);
      }
      continue;
    }

    if (LIFT && mt == 0) {
      // end values of the homogeneous lift (Section 2.3.1): the product's rows 0
      // and N are the face-row dot products s0 = D[0][:] u, sN = D[N][:] u of the
      // interior values, and M [u0, uN] = -[s0, sN] on the Neumann ends
#pragma unroll
      for (int r = 0; r < (CG ? 4 : 1); ++r)
        if (CG ? li == 0 : lk == 0) {
          const int c = col_of(r);
          const T s0 = acco[r] + acce[r], sN = acco[r] - acce[r];
          const T* e = A.rinv ? A.rinv + 4 * face_index(tile_in(tile) * C + c) : linv + 4 * bct;
          cend[2 * c] = -(e[0] * s0 + e[1] * sN);
          cend[2 * c + 1] = -(e[2] * s0 + e[3] * sN);
        }
    }
    if (FULL && mt == 0) {
      // the face rows at the end nodes this axis owns: u on a Dirichlet face,
      // the outward derivative plus sigma u on a Neumann one
#pragma unroll
      for (int r = 0; r < (CG ? 4 : 1); ++r)
        if (CG ? li == 0 : lk == 0) {
          const int c = col_of(r), b = cb[CG ? r : 0], fl = cflag[slot][c];
          const T dlo = acco[r] + acce[r], dhi = acco[r] - acce[r];
          const int q = tile_in(tile) * C + c;
          if (fl & PF_OWN_LO) {
            T v = dense_at(pu, b);
            if (nlo) v = (A.slo + (A.rlo ? A.rlo[q] : T(0))) * v - dlo;
            dense_ref(pyb, b) = v;
          }
          if (fl & PF_OWN_HI) {
            T v = dense_at(pu, b + __mul24(N, st));
            if (nhi) v = dhi + (A.shi + (A.rhi ? A.rhi[q] : T(0))) * v;
            dense_ref(pyb, b + __mul24(N, st)) = v;
          }
        }
    }
    lds_barrier();

    // flux K (M u) (+ C v), split into the tile for the second product; with
    // the lift, M u gains the rank-2 term u0 M[:][0] + uN M[:][N], whose row
    // N-i is -(u0 M[i][N] + uN M[i][0])
    const bool lift = LIFT && (nlo || nhi);
    {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = node_of(r), c = col_of(r);
        if (i < RM) {
          T lo = acco[r] + acce[r], hi = acco[r] - acce[r];
          T u0 = T(0), uN = T(0);
          if (lift) {
            u0 = cend[2 * c];
            uN = cend[2 * c + 1];
            const T c0 = dc0[i], cN = dcN[i];
            lo += u0 * c0 + uN * cN;
            hi -= u0 * cN + uN * c0;
          }
          lo *= klo[r];
          hi *= khi[r];
          if (JAC) {
            // the lifted direction itself, from its rows of the tile
            T vlo = u0, vhi = uN;
            if (i != 0) {
              const T ev = U[i * SC + c], od = i < KO ? U[OB + i * SC + c] : T(0);
              vlo = T(0.5) * (ev + od);
              vhi = T(0.5) * (ev - od);
            }
            lo += clo[JAC ? r : 0] * vlo;
            hi += chi[JAC ? r : 0] * vhi;
          }
          if (2 * i == N) {
            U[i * SC + c] = lo + lo;
          } else {
            U[i * SC + c] = lo + hi;
            U[OB + i * SC + c] = lo - hi;
          }
        }
        __builtin_amdgcn_sched_barrier(0);  // one row pair at a time: registers
      }
      if (midv && lc < C && lg == 0) {
        T m = mid;
        if (lift) m += cend[2 * lc] * dc0[half] + cend[2 * lc + 1] * dcN[half];
        m *= kmid;
        if (JAC) m += cmid * (T(0.5) * U[half * SC + lc]);
        U[half * SC + lc] = m + m;
      }
    }
    lds_barrier();

    // divergence part, with the partial sums and the next tile's u in flight
    const T* pun = PREF ? system_of(nxt).u : nullptr;
    const int stn = more ? st : 0;
    product([&](int ks) {
      constexpr int NY = FIRST ? 0 : 4, NL = NY + (PREF ? 2 * EPP : 0), PER = (NL + KS) / (KS + 1);
#pragma unroll
      for (int x = 0; x < PER; ++x) {
        const int l = ks * PER + x;
        if (l < NY) load_y(l < NY ? l : 0);
        else if (l < NL) load_u(l - NY, pun, slot ^ 1, stn);
      }
    });

    if (TRA && (nlo || nhi)) {
      // transposed lift: mu = M^{-T} [z_0, z_N]; interior -= mu0 D[0][:] + muN D[N][:]
      // (D[0][j] and D[N][j] are the end columns of the table of D^T)
      if (mt == 0) {
#pragma unroll
        for (int r = 0; r < (CG ? 4 : 1); ++r)
          if (CG ? li == 0 : lk == 0) {
            const int c = col_of(r);
            const T z0 = acco[r] + acce[r], zN = acco[r] - acce[r];
            const T* e = A.rinv ? A.rinv + 4 * face_index(tile_in(tile) * C + c) : linv + 4 * bct;
            cend[2 * c] = e[0] * z0 + e[2] * zN;
            cend[2 * c + 1] = e[1] * z0 + e[3] * zN;
          }
      }
      lds_barrier();
    }

    // store: interior nodes; the reduced forms write 0 to the two end nodes
    {
      auto put = [&](int off, T v, T y0, T y1) {
        if (!FIRST) v += y0;
        if (YADD) v += y1;
        dense_ref(py, off) = v;
      };
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = node_of(r), c = col_of(r), b = cb[CG ? r : 0];
        if (b >= 0 && i < RM && (!FULL || (cflag[slot][c] & PF_TIN))) {
          T lo = acco[r] + acce[r], hi = acco[r] - acce[r];
          if (TRA && (nlo || nhi)) {
            const T m0 = cend[2 * c], mN = cend[2 * c + 1], d0 = dc0[i], dN = dcN[i];
            lo -= m0 * d0 + mN * dN;
            hi += m0 * dN + mN * d0;
          }
          const int olo = b + __mul24(i, st), ohi = b + __mul24(N - i, st);
          if (i == 0) {
            if (CG && !FULL) {
              dense_ref(py, olo) = T(0);
              dense_ref(py, ohi) = T(0);
            }
          } else {
            put(olo, lo, FIRST ? T(0) : ylo[r], YADD ? zlo[YADD ? r : 0] : T(0));
            if (2 * i != N) put(ohi, hi, FIRST ? T(0) : yhi[r], YADD ? zhi[YADD ? r : 0] : T(0));
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (midv && lc < C && lg == 0 && bmid0 >= 0 && (!FULL || (cflag[slot][lc] & PF_TIN))) {
        T m = mid;
        if (TRA && (nlo || nhi)) m -= cend[2 * lc] * dc0[half] + cend[2 * lc + 1] * dcN[half];
        put(bmid, m, ymid, zmid);
      }
    }
    if (!PREF && more) {
      const Sys s = system_of(nxt);
#pragma unroll
      for (int l = 0; l < 2 * EPP; ++l) load_u(l, s.u, slot ^ 1, st);
    }
  }
}

}  // namespace cheb

// Matrix-core route: the fragment tables of D and D^T written into the plan,
// and the launches of the axis passes.
#include <cstdlib>
#include <vector>

#include "cheb_host.h"
#include "dense_launch.h"

namespace cheb {

LINE_EXTERN(double, 1);
LINE_EXTERN(double, 2);
LINE_EXTERN(double, 3);
LINE_EXTERN(double, 4);
LINE_EXTERN(double, 5);
LINE_EXTERN(double, 6);
LINE_EXTERN(double, 7);
LINE_EXTERN(double, 8);
LINE_EXTERN(float, 1);
LINE_EXTERN(float, 2);
LINE_EXTERN(float, 3);
LINE_EXTERN(float, 4);
LINE_EXTERN(float, 5);
LINE_EXTERN(float, 6);
LINE_EXTERN(float, 7);
LINE_EXTERN(float, 8);

namespace {

// fragment table (line_tab) of a centro-antisymmetric n x n matrix M, in the
// lane order the kernels load: entry (mt, ks, lane) holds the operand of row
// 16 mt + lane % 16 and column line_kmap(ks, lane / 16), zero past the axis' rows
template <typename F>
void line_table(int N, int mts, bool f32, const AxisConst& c, F m, double* tab) {
  const int R = line_pairs(N), KO = (N & 1) ? R : R - 1;
  const bool midv = line_midv(N, mts);
  const int RM = midv ? R - 1 : R;
  const bool kmap32 = f32 && mts <= kWaveMaxMT;
  const LineTab lt = line_tab(mts);
  for (int i = 0; i < lt.size; ++i) tab[i] = 0.0;
  auto ao = [&](int i, int j) { return 0.5 * (m(i, j) - m(i, N - j)); };
  for (int mt = 0; mt < mts; ++mt)
    for (int ks = 0; ks <= 4 * mts; ++ks)
      for (int l = 0; l < 64; ++l) {
        const int i = 16 * mt + (l & 15), j = line_kmap(ks, l >> 4, kmap32);
        if (i >= RM || j >= R) continue;
        const double x = m(i, j), y = m(i, N - j);
        tab[(mt * (4 * mts + 1) + ks) * 64 + l] = 2 * j == N ? 0.5 * x : 0.5 * (x + y);
        if (j < KO && ks < 4 * mts) tab[lt.off_o + (mt * 4 * mts + ks) * 64 + l] = 0.5 * (x - y);
      }
  if (midv)
    for (int j = 0; j < KO; ++j) tab[lt.off_mid + j] = ao(N / 2, j);
  for (int i = 0; i < R; ++i) {
    tab[lt.off_c0 + i] = m(i, 0);
    tab[lt.off_cN + i] = m(i, N);
  }
  // the face rows' end-value block M = [m00 m0N; mN0 mNN]; entries that belong
  // to a Dirichlet end are never used, kept finite
  double* e = tab + lt.off_lift;
  const double det = c.m00 * c.mNN - c.m0N * c.mN0, id = det != 0.0 ? 1.0 / det : 0.0;
  e[4] = c.m00 != 0.0 ? 1.0 / c.m00 : 0.0;
  e[8 + 3] = c.mNN != 0.0 ? 1.0 / c.mNN : 0.0;
  e[12] = c.mNN * id;
  e[13] = -c.m0N * id;
  e[14] = -c.mN0 * id;
  e[15] = c.m00 * id;
}

template <typename T>
const T* tables(const cheb_plan* p);
template <>
const double* tables<double>(const cheb_plan* p) { return p->dd64; }
template <>
const float* tables<float>(const cheb_plan* p) { return p->dd32; }

template <typename T>
constexpr int prec_index() {
  return sizeof(T) == sizeof(double) ? 0 : 1;
}

template <typename T>
const T* robin_array(const cheb_plan* p);
template <>
const double* robin_array<double>(const cheb_plan* p) { return p->rn64; }
template <>
const float* robin_array<float>(const cheb_plan* p) { return p->rn32; }

bool is_deriv(int mode) { return mode == LINE_DERIV || mode == LINE_DMUL; }

// whether a pass along the axis reads its tables of one block more
bool raised_pass(const cheb_plan* p, int axis, int mode, bool batch, int pi) {
  return p->raised == axis + 1 && p->raised_use[pi] && !batch && !is_deriv(mode);
}
int pass_blocks(const cheb_plan* p, int axis, int mode, bool batch, int pi) {
  return p->dd_mt[axis] + (raised_pass(p, axis, mode, batch, pi) ? 1 : 0);
}

// whether the x and y passes of an apply can share a launch
bool share_launch(const cheb_plan* p, int pi) {
  return p->dd_ok[0] && p->dd_ok[1] && p->dense_var[0][pi] == p->dense_var[1][pi] &&
         pass_blocks(p, 0, LINE_REDUCED, false, pi) == pass_blocks(p, 1, LINE_REDUCED, false, pi);
}

// the launch fields of one axis: tables, lift entries, per-node inverses, output
template <typename T>
LineAxis<T> line_axis(const cheb_plan* p, int axis, int mode, int transpose, bool batch, T* y, T* yb) {
  const bool all = mode == LINE_FULL || is_deriv(mode);  // every pencil, not only the interior ones
  LineAxis<T> x;
  x.tab = tables<T>(p) + (raised_pass(p, axis, mode, batch, prec_index<T>()) ? p->raised_off : p->dd_off[axis])[transpose];
  x.y = y;
  x.yb = yb;
  x.c = nullptr;
  x.axis = axis;
  x.N = p->ax[axis].N;
  {
    const int nb = axis == 2 ? p->g.n[1] : p->g.n[2];
    x.inv_nbi = 1.0f / float(all ? nb : nb - 2);
    x.inv_pairs = 1.0f / float(line_pairs(x.N));
  }
  x.slo = T(p->g.robin[2 * axis]);
  x.shi = T(p->g.robin[2 * axis + 1]);
  const T* rn = batch ? nullptr : robin_array<T>(p);
  x.rinv = rn ? rn + robin_inv_offset(p, axis) : nullptr;
  x.rlo = rn ? rn + face_offset(2 * axis, p->g.n) : nullptr;
  x.rhi = rn ? rn + face_offset(2 * axis + 1, p->g.n) : nullptr;
  return x;
}

template <typename T>
LineArgs<T> line_args(const cheb_plan* p, const T* K, const T* u, const DenseSys* sys, const int* act, int nact) {
  LineArgs<T> a;
  a.gate = sys ? nullptr : p->gate;
  a.u = u;
  a.K = K;
  a.sys = sys;
  a.act = act;
  a.nact = nact;
  for (int i = 0; i < 3; ++i) a.n[i] = p->g.n[i];
  a.bcmask = bc_mask(p->g.bc);
  a.nseg = 1;
  a.wpw = 0;
  a.tasks = 0;
  a.yadd = nullptr;
  return a;
}

template <typename T>
int dispatch_line(const cheb_plan* p, LineArgs<T>& a, int mode, int first, hipStream_t s) {
  const int axis = a.ax[0].axis, shape = p->dense_var[axis][prec_index<T>()];
  const int mt = pass_blocks(p, axis, mode, a.sys != nullptr, prec_index<T>());
  const bool der = is_deriv(mode);
  const int o = der || mode == LINE_FULL ? 0 : 2;
  auto tasks = [&](int x) {
    return ((a.n[x == 0 ? 1 : 0] - o) * (a.n[x == 2 ? 1 : 2] - o) + 15) / 16;
  };
  a.tasks = axis < 2 && !der && share_launch(p, prec_index<T>()) ? tasks(0) + tasks(1) : tasks(axis);
  switch (mt) {
    case 1: return launch_line_mt<T, 1>(a, mode, first, shape, s);
    case 2: return launch_line_mt<T, 2>(a, mode, first, shape, s);
    case 3: return launch_line_mt<T, 3>(a, mode, first, shape, s);
    case 4: return launch_line_mt<T, 4>(a, mode, first, shape, s);
    case 5: return launch_line_mt<T, 5>(a, mode, first, shape, s);
    case 6: return launch_line_mt<T, 6>(a, mode, first, shape, s);
    case 7: return launch_line_mt<T, 7>(a, mode, first, shape, s);
    case 8: return launch_line_mt<T, 8>(a, mode, first, shape, s);
    default: set_error("matrix-core pass: unsupported N"); return CHEB_ERR_UNSUPPORTED;
  }
}

// Whether an apply on stream s may write its second partial sum into the plan's
// buffer.  A plan's calls may be in flight on several streams at once, and a
// captured apply runs whenever its graph is replayed, so the one buffer serves the
// creation stream alone, outside a capture (the legacy stream is never captured;
// the per-thread handle stands for a stream per thread).  Others bring a field of
// their own (cheb_apply_scratch, the solves' workspace) or take three launches:
// 129^3 FP64 59 us against 50.5, 33^3 15.8 against 13.
bool pair_usable(const cheb_plan* p, hipStream_t s) {
  if (!p->pair_buf || s != p->home || s == hipStreamPerThread) return false;
  if (s == nullptr) return true;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return st == hipStreamCaptureStatusNone;
}

}  // namespace

template <typename T>
int launch_line_pass(const cheb_plan* p, int axis, int mode, int transpose, int first, const T* K, const T* c,
                     const T* u, T* y, hipStream_t s) {
  if (axis == 2 && !first) {
    // the accumulating unit-stride kernel always adds the second partial sum
    set_error("matrix-core pass: along z only the first pass of an apply runs alone");
    return CHEB_ERR_INVALID_ARG;
  }
  LineArgs<T> a = line_args<T>(p, K, u, nullptr, nullptr, 0);
  a.ax[0] = line_axis<T>(p, axis, mode, transpose, false, y, y);
  a.ax[0].c = c;
  a.ax[1] = a.ax[0];
  return dispatch_line<T>(p, a, mode, first, s);
}

template <typename T>
int launch_line_apply(const cheb_plan* p, int mode, const T* K, const T* const* c, const T* u, T* y, hipStream_t s,
                      T* second) {
  const int tr = mode == LINE_TRANSP ? 1 : 0;
  const int pi = prec_index<T>();
  // the x and y passes share a launch, each into its own output
  T* y1 = nullptr;
  if (share_launch(p, pi)) y1 = second ? second : pair_usable(p, s) ? (T*)p->pair_buf : nullptr;
  if (y1) {
    LineArgs<T> a = line_args<T>(p, K, u, nullptr, nullptr, 0);
    a.nseg = 2;
    a.ax[0] = line_axis<T>(p, 0, mode, tr, false, y, y);
    a.ax[1] = line_axis<T>(p, 1, mode, tr, false, y1, y);
    if (c) {
      a.ax[0].c = c[0];
      a.ax[1].c = c[1];
    }
    int rc = dispatch_line<T>(p, a, mode, 1, s);
    if (rc) return rc;
    a.nseg = 1;
    a.yadd = y1;
    a.ax[0] = line_axis<T>(p, 2, mode, tr, false, y, y);
    if (c) a.ax[0].c = c[2];
    a.ax[1] = a.ax[0];
    return dispatch_line<T>(p, a, mode, 0, s);
  }
  // (z + x) + y, as above (the one-wave kernel adds a lone middle row along z as z +
  // (x + y) there: the last bit may differ)
  for (int axis : {2, 0, 1})
    if (int rc = launch_line_pass<T>(p, axis, mode, tr, axis == 2, K, c ? c[axis] : nullptr, u, y, s)) return rc;
  return CHEB_OK;
}

template <typename T>
int launch_dense_batch(const cheb_plan* rep, int axis, int first, const T* K, const T* u, T* y,
                       const DenseSys* sys, const int* act, int nact, hipStream_t s) {
  if (nact <= 0) return CHEB_OK;
  if (axis == 2 && !first) {
    set_error("matrix-core pass: along z only the first pass of an apply runs alone");
    return CHEB_ERR_INVALID_ARG;
  }
  LineArgs<T> a = line_args<T>(rep, K, u, sys, act, nact);
  a.ax[0] = line_axis<T>(rep, axis, LINE_REDUCED, 0, true, y, nullptr);
  a.ax[1] = a.ax[0];
  return dispatch_line<T>(rep, a, LINE_REDUCED, first, s);
}

template int launch_line_pass<double>(const cheb_plan*, int, int, int, int, const double*, const double*,
                                      const double*, double*, hipStream_t);
template int launch_line_pass<float>(const cheb_plan*, int, int, int, int, const float*, const float*, const float*,
                                     float*, hipStream_t);
template int launch_line_apply<double>(const cheb_plan*, int, const double*, const double* const*, const double*,
                                       double*, hipStream_t, double*);
template int launch_line_apply<float>(const cheb_plan*, int, const float*, const float* const*, const float*, float*,
                                      hipStream_t, float*);
template int launch_dense_batch<double>(const cheb_plan*, int, int, const double*, const double*, double*,
                                        const DenseSys*, const int*, int, hipStream_t);
template int launch_dense_batch<float>(const cheb_plan*, int, int, const float*, const float*, float*, const DenseSys*,
                                       const int*, int, hipStream_t);

int dense_setup(cheb_plan* p, const cheb_plan* box, bool second) {
  if (box) {
    for (int a = 0; a < 3; ++a) {
      p->dd_mt[a] = box->dd_mt[a];
      p->dd_ok[a] = box->dd_ok[a];
      for (int q = 0; q < 2; ++q) {
        p->dd_off[a][q] = box->dd_off[a][q];
        p->dense_var[a][q] = box->dense_var[a][q];
      }
    }
    p->raised = box->raised;
    for (int q = 0; q < 2; ++q) {
      p->raised_use[q] = box->raised_use[q];
      p->raised_off[q] = box->raised_off[q];
    }
    p->dd64 = box->dd64;
    p->dd32 = box->dd32;
    p->dd_lent = 1;
    return CHEB_OK;
  }
  size_t total = 0;
  int src[3];
  for (int a = 0; a < 3; ++a) {
    p->dd_mt[a] = line_mt(p->ax[a].N);
    p->dd_ok[a] = line_supported(p->ax[a].N) ? 1 : 0;
    // default tile shape (16 pencils per tile); cheb_plan_autotune replaces it
    // by timing
    p->dense_var[a][0] = 1;
    p->dense_var[a][1] = 1;
    // axes with the same N, length and end-value block share their tables
    src[a] = a;
    for (int b = 0; b < a; ++b)
      if (p->ax[b].N == p->ax[a].N && p->ax[b].L == p->ax[a].L && p->ax[b].m00 == p->ax[a].m00 &&
          p->ax[b].mNN == p->ax[a].mNN) {
        src[a] = b;
        break;
      }
    for (int t = 0; t < 2; ++t) {
      if (src[a] != a) {
        p->dd_off[a][t] = p->dd_off[src[a]][t];
        continue;
      }
      p->dd_off[a][t] = total;
      if (p->dd_ok[a]) total += round_up((size_t)line_tab(p->dd_mt[a]).size, 64);
    }
  }
  // The x and y passes share a launch when their tables have the same number of
  // row blocks.  An axis with one block fewer has a second pair of tables with an
  // idle block, for the applies (derivatives run alone): a third launch costs more.
  // 33x65x65 FP64 15.5 us against 19.6, 97x129x129 48 against 51, 161x193x33 41
  // against 53; FP32 12.7 against 16.5, 29.7 against 35, 26 against 38.  From four
  // blocks to five the axis also changes kernels, from a wave to a task to a wave to
  // a row block, which in FP64 only small grids stand: x and y of 116 tasks
  // (140x128x9) 18.9 us against 26.2, of 477 (150x100x33) 33.3 against 35.2, of 1000
  // (131x127x65) 45.3 against 46.4 but of 1568 (160x100x100) 80 against 63, of 2050
  // (130x129x130) 95 against 84; FP32 gains at every size (150x129x129 48 against 53).
  p->raised = 0;
  if (p->dd_ok[0] && p->dd_ok[1] && p->dd_ok[2] && std::abs(p->dd_mt[0] - p->dd_mt[1]) == 1) {
    const int a = p->dd_mt[0] < p->dd_mt[1] ? 0 : 1;
    const int* n = p->g.n;
    const int tasks = ((n[1] - 2) * (n[2] - 2) + 15) / 16 + ((n[0] - 2) * (n[2] - 2) + 15) / 16;
    p->raised = a + 1;
    p->raised_use[0] = p->dd_mt[a] != kWaveMaxMT || tasks <= 1024;
    p->raised_use[1] = 1;
    for (int t = 0; t < 2; ++t) {
      p->raised_off[t] = total;
      total += round_up((size_t)line_tab(p->dd_mt[a] + 1).size, 64);
    }
  }
  p->dd64 = nullptr;
  p->dd32 = nullptr;
  if (total == 0) return CHEB_OK;
  std::vector<double> D[3];
  for (int a = 0; a < 3; ++a)
    if (p->dd_ok[a] && src[a] == a) dense_D(p->ax[a].N, p->ax[a].L, D[a]);
  auto fill = [&](bool f32, std::vector<double>& h) {
    h.resize(total);
    auto pair = [&](int a, int mt, const size_t* off) {
      const int N = p->ax[a].N, n = N + 1;
      const double* M = D[src[a]].data();
      line_table(N, mt, f32, p->ax[a], [=](int i, int j) { return M[(size_t)i * n + j]; }, h.data() + off[0]);
      line_table(N, mt, f32, p->ax[a], [=](int i, int j) { return M[(size_t)j * n + i]; }, h.data() + off[1]);
    };
    for (int a = 0; a < 3; ++a)
      if (p->dd_ok[a] && src[a] == a) pair(a, p->dd_mt[a], p->dd_off[a]);
    if (p->raised) pair(p->raised - 1, p->dd_mt[p->raised - 1] + 1, p->raised_off);
  };
  // each precision that the plan's passes run in
  int rc = CHEB_OK;
  std::vector<double> h;
  if (p->prec != CHEB_F32) {
    fill(false, h);
    rc = hip_check(hipMalloc((void**)&p->dd64, total * sizeof(double)), "hipMalloc(matrix-core tables)");
    if (!rc)
      rc = hip_check(hipMemcpy(p->dd64, h.data(), total * sizeof(double), hipMemcpyHostToDevice),
                     "hipMemcpy(matrix-core tables)");
  }
  if (!rc && p->prec != CHEB_F64) {
    fill(true, h);
    std::vector<float> h32(h.begin(), h.end());
    rc = hip_check(hipMalloc((void**)&p->dd32, total * sizeof(float)), "hipMalloc(matrix-core tables)");
    if (!rc)
      rc = hip_check(hipMemcpy(p->dd32, h32.data(), total * sizeof(float), hipMemcpyHostToDevice),
                     "hipMemcpy(matrix-core tables)");
  }
  // second output of the two-axis launch (x and y passes together), for plans
  // whose three axes can all take the matrix-core route; optional: without it
  // an apply takes three launches
  if (!rc && second && p->dd_ok[0] && p->dd_ok[1] && p->dd_ok[2]) {
    const size_t bytes = p->npts * (p->prec == CHEB_F32 ? sizeof(float) : sizeof(double));
    if (hipMalloc(&p->pair_buf, bytes) != hipSuccess) {
      (void)hipGetLastError();
      p->pair_buf = nullptr;
    }
  }
  return rc;
}

}  // namespace cheb

// Modal prolongation (Section 2.3.3): along each axis, the DCT-I of the coarse
// pencil gives its Chebyshev coefficients, the coefficients are zero-padded to
// the fine degree and the fine pencil is their cosine sum at the fine CGL
// nodes.  z, then y, then x: (nc,nc,nc) -> (nc,nc,nf) -> (nc,nf,nf) -> (nf,nf,nf).
//
// The three steps along an axis are one matrix P (nf x nc) with a closed form
// (the coefficient sums are Dirichlet kernels; theta_i = pi i / Nf, phi_j = pi j / Nc)
//   P_ij = (-1)^j sin(Nc theta_i) sin(theta_i)
//          / (Nc c_j 2 sin((theta_i + phi_j) / 2) sin((theta_i - phi_j) / 2)),
// c_j = 2 at the two ends, 1 inside, and 1 where theta_i = phi_j.  It is
// centro-symmetric, so it runs as an even-odd split contraction on the matrix
// cores (FP64 for both field types): with e_j = u_j + u_{Nc-j} and
// o_j = u_j - u_{Nc-j},
//   (Pu)_i = s_i + d_i, (Pu)_{Nf-i} = s_i - d_i,
//   s_i = sum_j (P_ij + P_{i,Nc-j}) / 2 e_j,  d_i = sum_j (P_ij - P_{i,Nc-j}) / 2 o_j.
// A workgroup forms the fragments of 32 or 48 row pairs in LDS (two sines of
// exact integer fractions and a division per entry pair, so the entries keep
// their relative accuracy where nodes nearly meet) and its waves run tasks of 16
// pencils over them, the pencils read straight from memory.  65^3 -> 129^3 in
// FP64 takes 41 us, where direct cosine sums on the vector ALUs took 166 us
// (129^3 -> 257^3: 185 and 1495 us, 17^3 -> 33^3: 15.5 both); what is left is three launches, each
// with its table (about 3 us) and one or two rounds of tasks against 5 us of HBM
// traffic and 4 us of matrix-core time in all.  Largest error against long
// double arithmetic over sizes 9 to 129: 1.3e-15 of the largest value, the
// sums' 1.5e-15.
#include <cmath>
#include <mutex>

#include "dev_common.h"
#include "internal.h"

namespace cheb {

namespace {

constexpr int kPW = 4;      // waves per workgroup
constexpr int kPWG = 512;   // workgroups of a launch: 768 and 1024 (more tables formed) take up to 3 us longer at 129^3

__device__ __forceinline__ void pencil_geom(int axis, int p, const int* n, size_t* base, int* stride) {
  if (axis == 2) {
    *base = (size_t)p * n[2];
    *stride = 1;
  } else if (axis == 1) {
    const int ia = p / n[2], ib = p - ia * n[2];
    *base = (size_t)ia * n[1] * n[2] + ib;
    *stride = n[2];
  } else {
    *base = p;
    *stride = n[1] * n[2];
  }
}

// RB: 16-row blocks of row pairs per workgroup
constexpr int prolong_lds_bytes(int Nc, int RB) {
  return (32 * RB + (8 + RB * 128) * ((Nc / 2 + 4) / 4)) * (int)sizeof(double);
}

template <typename T, int RB>
__global__ __launch_bounds__(64 * kPW) void k_prolong_axis(const T* __restrict__ src, T* __restrict__ dst, int axis,
                                                          int s0, int s1, int s2, int d0, int d1, int d2) {
  extern __shared__ __align__(16) unsigned char smem[];
  typedef Mfma<double>::v4 V4;
  const int ns[3] = {s0, s1, s2}, nd[3] = {d0, d1, d2};
  const int Nc = ns[axis] - 1, Nf = nd[axis] - 1;
  const int npen = axis == 2 ? s0 * s1 : axis == 1 ? s0 * s2 : s1 * s2;
  const int Rc = Nc / 2 + 1, Rf = Nf / 2 + 1, KS = (Rc + 3) / 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int row0 = blockIdx.y * 16 * RB;
  const int ntasks = (npen + 15) / 16;
  // the loads of U steps of pairs (j, Nc - j) are in flight at once, those of
  // the first task behind the tables (rows past Rc read the pencil's first node
  // and count as zeros)
  constexpr int U = 8;
  T lo[U], hi[U];
  auto load = [&](const T* u, int st, int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < U; ++x) {
      const int j = 4 * (k0 + x) + lk, jj = j < Rc ? j : 0;
      lo[x] = u[(size_t)jj * st];
      hi[x] = u[(size_t)(Nc - jj) * st];
    }
  };
  int task = blockIdx.x * kPW + wave;
  auto pencil = [&](int t) __attribute__((always_inline)) {
    const int p = t * 16 + li;
    return p < npen ? p : npen - 1;
  };
  size_t bs;
  int ss;
  pencil_geom(axis, pencil(task), ns, &bs, &ss);
  load(src + bs, ss, 0);
  // row factors sin(Nc theta_i) sin(theta_i) / Nc and cos(theta_i), column
  // factors (-1)^j / c_j and cos(phi_j); every angle is an exact fraction in the
  // first quadrant
  double* rf = (double*)smem;            // 16 RB x 2
  double* cf = rf + 32 * RB;           // 4 KS x 2
  double* tab = cf + 8 * KS;             // fragments [block][even, odd][step][lane]
  for (int e = tid; e < 16 * RB + 4 * KS; e += 64 * kPW) {
    if (e < 16 * RB) {
      const int i = row0 + e < Rf ? row0 + e : Rf - 1;
      int t = (int)((long long)i * Nc % (2 * Nf));
      const bool neg = t >= Nf;
      if (neg) t -= Nf;
      if (2 * t > Nf) t = Nf - t;
      const double v = sinpi(double(t) / double(Nf)) * sinpi(double(i) / double(Nf)) / double(Nc);
      rf[2 * e] = neg ? -v : v;
      rf[2 * e + 1] = sinpi(double(Nf - 2 * i) / double(2 * Nf));
    } else {
      const int j = e - 16 * RB;
      cf[2 * j] = j == 0 ? 0.5 : 2 * j == Nc ? ((j & 1) ? -0.5 : 0.5) : (j & 1) ? -1.0 : 1.0;
      cf[2 * j + 1] = j < Rc ? sinpi(double(Nc - 2 * j) / double(2 * Nc)) : 0.0;
    }
  }
  __syncthreads();
  // lane l of a fragment: row 16 block + l % 16, column 4 step + l / 16
  const double inv = 1.0 / (double(Nf) * double(Nc));
  for (int e = tid; e < RB * KS * 64; e += 64 * kPW) {
    const int l = e & 63, bk = e >> 6, blk = bk / KS, ks = bk - blk * KS;
    const int r = 16 * blk + (l & 15), j = 4 * ks + (l >> 4), i = row0 + r;
    double pe = 0.0, po = 0.0;
    if (i < Rf && j < Rc) {
      const int m = i * Nc, q = j * Nf;
      if (m == q) {
        pe = 0.5;
        po = 0.5;
      } else {
        const int t = 2 * (m + q) > Nf * Nc ? Nf * Nc - m - q : m + q;
        const double f = rf[2 * r] * cf[2 * j] / (sinpi(double(t) * inv) * sinpi(double(m - q) * inv));
        pe = f * ((Nc & 1) ? cf[2 * j + 1] : rf[2 * r + 1]);
        po = f * ((Nc & 1) ? rf[2 * r + 1] : cf[2 * j + 1]);
      }
    }
    tab[((blk * 2) * KS + ks) * 64 + l] = pe;
    tab[((blk * 2 + 1) * KS + ks) * 64 + l] = po;
  }
  __syncthreads();
  for (; task < ntasks; task += gridDim.x * kPW) {
    V4 se[RB], so[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) se[b] = so[b] = V4{0, 0, 0, 0};
    for (int k0 = 0; k0 < KS; k0 += U) {
      if (k0) load(src + bs, ss, k0);
#pragma unroll
      for (int x = 0; x < U; ++x) {
        if (k0 + x >= KS) break;
        const bool in = 4 * (k0 + x) + lk < Rc;
        const double a = in ? double(lo[x]) : 0.0, b = in ? double(hi[x]) : 0.0;
#pragma unroll
        for (int q = 0; q < RB; ++q) {
          se[q] = Mfma<double>::mac(tab[((q * 2) * KS + k0 + x) * 64 + lane], a + b, se[q]);
          so[q] = Mfma<double>::mac(tab[((q * 2 + 1) * KS + k0 + x) * 64 + lane], a - b, so[q]);
        }
      }
    }
    size_t bd;
    int sd;
    pencil_geom(axis, pencil(task), nd, &bd, &sd);
    const bool valid = task * 16 + li < npen;
    const int next = task + gridDim.x * kPW;
    if (next < ntasks) {
      pencil_geom(axis, pencil(next), ns, &bs, &ss);
      load(src + bs, ss, 0);
    }
    if (!valid) continue;
#pragma unroll
    for (int q = 0; q < RB; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = row0 + 16 * q + Mfma<double>::row(lk, r);
        if (i >= Rf) continue;
        dst[bd + (size_t)i * sd] = T(se[q][r] + so[q][r]);
        if (2 * i != Nf) dst[bd + (size_t)(Nf - i) * sd] = T(se[q][r] - so[q][r]);
      }
  }
}

}  // namespace

namespace {

template <typename T, int RB>
int launch_prolong_axis(const T* in, T* out, int axis, const int* cur, const int* nxt, hipStream_t s) {
  const int npen = axis == 2 ? cur[0] * cur[1] : axis == 1 ? cur[0] * cur[2] : cur[1] * cur[2];
  const int lds = prolong_lds_bytes(cur[axis] - 1, RB);
  if (lds > 64 * 1024)
    if (int rc = hip_check(hipFuncSetAttribute((const void*)k_prolong_axis<T, RB>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, lds),
                           "prolongation LDS attribute"))
      return rc;
  // a workgroup for RB row blocks and a task per wave, up to kPWG in all (each
  // forms its own tables)
  const int groups = ((nxt[axis] - 1) / 2 + 16 * RB) / (16 * RB);
  const int need = (npen + 16 * kPW - 1) / (16 * kPW), most = kPWG / groups > 0 ? kPWG / groups : 1;
  hipLaunchKernelGGL((k_prolong_axis<T, RB>), dim3(need < most ? need : most, groups), dim3(64 * kPW), lds, s, in, out,
                     axis, cur[0], cur[1], cur[2], nxt[0], nxt[1], nxt[2]);
  return hip_check(hipGetLastError(), "prolongation");
}

}  // namespace

template <typename T>
int prolong_t(const cheb_plan* pc, const cheb_plan* pf, const T* uc, T* uf, T* tmp1, T* tmp2, hipStream_t s) {
  int cur[3] = {pc->g.n[0], pc->g.n[1], pc->g.n[2]};
  const T* in = uc;
  for (int step = 0; step < 3; ++step) {
    const int axis = 2 - step;
    int nxt[3] = {cur[0], cur[1], cur[2]};
    nxt[axis] = pf->g.n[axis];
    T* out = step == 2 ? uf : (step == 0 ? tmp1 : tmp2);
    const int Nc = cur[axis] - 1, Nf = nxt[axis] - 1;
    // three row blocks per workgroup read a pencil fewer times and two form
    // smaller tables: 257^3, 4129 tasks a pass, takes 185 us with three and
    // 220 us with two, 181^3, 2048 tasks, 81 and 76 us, 129^3 47 and 41 us
    const int blocks = (Nf / 2 + 16) / 16;
    const int npen = axis == 2 ? cur[0] * cur[1] : axis == 1 ? cur[0] * cur[2] : cur[1] * cur[2];
    const bool three = npen > 16 * 3072 && (blocks + 2) / 3 < (blocks + 1) / 2 && prolong_lds_bytes(Nc, 3) <= 80 * 1024;
    int rc = three ? launch_prolong_axis<T, 3>(in, out, axis, cur, nxt, s)
                   : launch_prolong_axis<T, 2>(in, out, axis, cur, nxt, s);
    if (rc) return rc;
    in = out;
    for (int i = 0; i < 3; ++i) cur[i] = nxt[i];
  }
  return CHEB_OK;
}

template int prolong_t<double>(const cheb_plan*, const cheb_plan*, const double*, double*, double*, double*,
                               hipStream_t);
template int prolong_t<float>(const cheb_plan*, const cheb_plan*, const float*, float*, float*, float*,
                              hipStream_t);

}  // namespace cheb

using namespace cheb;

extern "C" int cheb_prolong(const cheb_plan* coarse, const cheb_plan* fine, const void* u_c, void* u_f,
                            const void* u_f_solved, double* e_ref) {
  if (!coarse || !fine || !u_c || !u_f || u_c == u_f) {
    set_error("invalid argument");
    return CHEB_ERR_INVALID_ARG;
  }
  if (coarse->prec != fine->prec) {
    set_error("coarse and fine plans must have the same precision");
    return CHEB_ERR_INVALID_ARG;
  }
  for (int a = 0; a < 3; ++a) {
    if (fine->g.n[a] < coarse->g.n[a]) {
      set_error("fine grid must not be smaller than the coarse grid");
      return CHEB_ERR_INVALID_ARG;
    }
    if (std::fabs(fine->g.lo[a] - coarse->g.lo[a]) > 0 || std::fabs(fine->g.hi[a] - coarse->g.hi[a]) > 0) {
      set_error("coarse and fine plans must describe the same box");
      return CHEB_ERR_INVALID_ARG;
    }
  }
  cheb_plan* pf = const_cast<cheb_plan*>(fine);
  const size_t esz = fine->prec == CHEB_F32 ? sizeof(float) : sizeof(double);
  const size_t fb = round_up(fine->npts * esz, 256);
  const size_t plen = multidot_partials_len(fine->npts, 1);
  const size_t need = 2 * fb + round_up((plen + 16) * sizeof(double), 256);
  if (!pf->ws || pf->ws_bytes < need) {
    set_error("prolongation needs the fine plan's workspace");
    return CHEB_ERR_WORKSPACE;
  }
  char* ws = (char*)pf->ws;
  int rc;
  if (fine->prec == CHEB_F32)
    rc = prolong_t<float>(coarse, fine, (const float*)u_c, (float*)u_f, (float*)ws, (float*)(ws + fb),
                          pf->stream);
  else
    rc = prolong_t<double>(coarse, fine, (const double*)u_c, (double*)u_f, (double*)ws, (double*)(ws + fb),
                           pf->stream);
  if (rc) return rc;
  if (u_f_solved && e_ref) {
    double* part = (double*)(ws + 2 * fb);
    double* res = part + plen;
    if (fine->prec == CHEB_F32) {
      float* d = (float*)ws;
      rc = copy_scale<float>(d, (const float*)u_f_solved, 1.0, fine->npts, pf->stream);
      if (!rc) rc = axpby<float>(d, (const float*)u_f, -1.0, 1.0, fine->npts, pf->stream);
      if (!rc) rc = multidot<float>(nullptr, 0, 0, d, fine->npts, part, res, pf->stream);
      if (!rc) rc = multidot<float>(nullptr, 0, 0, (const float*)u_f_solved, fine->npts, part, res + 1, pf->stream);
    } else {
      double* d = (double*)ws;
      rc = copy_scale<double>(d, (const double*)u_f_solved, 1.0, fine->npts, pf->stream);
      if (!rc) rc = axpby<double>(d, (const double*)u_f, -1.0, 1.0, fine->npts, pf->stream);
      if (!rc) rc = multidot<double>(nullptr, 0, 0, d, fine->npts, part, res, pf->stream);
      if (!rc)
        rc = multidot<double>(nullptr, 0, 0, (const double*)u_f_solved, fine->npts, part, res + 1, pf->stream);
    }
    if (!rc)
      rc = hip_check(hipMemcpyAsync(pf->hpinned, res, 2 * sizeof(double), hipMemcpyDeviceToHost, pf->stream),
                     "hipMemcpyAsync");
    if (!rc) rc = hip_check(hipStreamSynchronize(pf->stream), "hipStreamSynchronize");
    if (rc) return rc;
    *e_ref = pf->hpinned[1] > 0 ? std::sqrt(pf->hpinned[0] / pf->hpinned[1]) : 0.0;
  }
  return CHEB_OK;
}

// ---- allocation-free prolongation ------------------------------------------
// The two intermediate fields of the three axis passes live in a file-scope
// device array instead of the fine plan's workspace.  Every GPU that runs this
// library holds one copy of it (at its own address) until the process ends.
namespace cheb {
namespace {

constexpr size_t kScratchBytes = size_t(128) << 20;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_scratch_mu;
void* g_scratch_ptr[64] = {};

// device address of `scratch` on `dev`, looked up once per device with that
// device current (the array's name is a host-side stand-in, not an address)
int scratch_address(int dev, void** out) {
  if (dev < 0 || dev >= 64) {
    set_error("device index out of range");
    return CHEB_ERR_DEVICE;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    int cur = -1;
    int rc = hip_check(hipGetDevice(&cur), "hipGetDevice");
    if (rc) return rc;
    if (cur != dev && (rc = hip_check(hipSetDevice(dev), "hipSetDevice"))) return rc;
    void* ptr = nullptr;
    rc = hip_check(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (cur != dev) {
      const int rc2 = hip_check(hipSetDevice(cur), "hipSetDevice");
      if (!rc) rc = rc2;
    }
    if (rc) return rc;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return CHEB_OK;
}

}  // namespace
}  // namespace cheb

extern "C" int cheb_prolong_noalloc(const cheb_plan* coarse, const cheb_plan* fine, const void* u_c, void* u_f) {
  if (!coarse || !fine || !u_c || !u_f || u_c == u_f) {
    set_error("invalid argument");
    return CHEB_ERR_INVALID_ARG;
  }
  if (coarse->prec != fine->prec || coarse->device != fine->device) {
    set_error("coarse and fine plans must have the same precision and device");
    return CHEB_ERR_INVALID_ARG;
  }
  for (int a = 0; a < 3; ++a) {
    if (fine->g.n[a] < coarse->g.n[a]) {
      set_error("fine grid must not be smaller than the coarse grid");
      return CHEB_ERR_INVALID_ARG;
    }
    if (std::fabs(fine->g.lo[a] - coarse->g.lo[a]) > 0 || std::fabs(fine->g.hi[a] - coarse->g.hi[a]) > 0) {
      set_error("coarse and fine plans must describe the same box");
      return CHEB_ERR_INVALID_ARG;
    }
  }
  // intermediates after the z pass (nc0, nc1, nf2) and the y pass (nc0, nf1, nf2)
  const size_t esz = fine->prec == CHEB_F32 ? sizeof(float) : sizeof(double);
  const size_t nc0 = coarse->g.n[0], nc1 = coarse->g.n[1], nf1 = fine->g.n[1], nf2 = fine->g.n[2];
  const size_t b1 = round_up(nc0 * nc1 * nf2 * esz, 256);
  const size_t b2 = round_up(nc0 * nf1 * nf2 * esz, 256);
  if (b1 + b2 > kScratchBytes) {
    set_error("prolongation intermediates (" + std::to_string(b1 + b2) + " bytes) exceed the " +
              std::to_string(kScratchBytes) + "-byte static scratch of cheb_prolong_noalloc");
    return CHEB_ERR_WORKSPACE;
  }
  void* base = nullptr;
  int rc = scratch_address(fine->device, &base);
  if (rc) return rc;
  char* ws = (char*)base;
  if (fine->prec == CHEB_F32)
    return prolong_t<float>(coarse, fine, (const float*)u_c, (float*)u_f, (float*)ws, (float*)(ws + b1),
                            fine->stream);
  return prolong_t<double>(coarse, fine, (const double*)u_c, (double*)u_f, (double*)ws, (double*)(ws + b1),
                           fine->stream);
}

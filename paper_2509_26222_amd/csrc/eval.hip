// Evaluation of the terrain model and its adjoint.
//
// f(x) = sum_j w_j phi(x, c_j) (eq. RBF_fml), grad f = -sum_j w_j phi
// (x - c_j)/sigma^2 (eq. manidolf_grad_detail with the sign of d/dx exp
// restored), the manifold residual r = xi_z - z_off - f(xi_xy) at
// xi = R p + t (eq. residual_manifold_left_wheel) and its pose Jacobian
// J = [(p x R^T g)^T, g^T], g = (-f_x, -f_y, 1) (eqs. manifold_derivative,
// manifold_grad_2, right perturbation, body-frame point).
//
// Candidates. The grid keeps the centers sorted by evaluation bins of side
// eh ~ rc/3 (rc = cutoff sigma, row-major bins), so a point's support
// circle meets at most 7 bin rows, and in each row only the bins whose x
// range meets the circle are read: one contiguous run of the sorted table
// per row. About 42 candidates per point are tested against 28 in the
// support (a 3x3 neighbourhood of bins of side rc tests about 81).
//
// Four lanes per point: each forms two of the point's (at most 8) row runs
// and the quad shares them by DPP broadcasts; in every run lane j takes
// entries j, j + 4, ..., so the quad's loads cover consecutive entries (a
// wave's gather touches 16 cache lines, not 64), two loads per lane in
// flight. The partial sums meet in a quad butterfly. The packed table holds
// (x', y', w, index) with coordinates relative to the grid origin and
// scaled by ks, so that phi = exp(-d'^2) (FP64) or exp2(-d'^2) (FP32,
// v_exp_f32): per candidate two subtractions, the squared distance, the
// exponential, the support test and three accumulations.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "internal.hpp"

namespace rbf {

template <typename T>
struct Vec4;
template <>
struct Vec4<float> {
  using type = float4;
};
template <>
struct Vec4<double> {
  using type = double4;
};
template <typename T>
struct Vec2;
template <>
struct Vec2<float> {
  using type = float2;
};
template <>
struct Vec2<double> {
  using type = double2;
};

// Constants of one evaluation call (see the header of this file).
template <typename T>
struct EvalK {
  T x0, y0;  // grid origin
  T ks;      // coordinate scale: phi = exp(-(ks d)^2) or exp2(-(ks d)^2)
  T rc2s;    // (ks cutoff sigma)^2: support test on the scaled squared distance
  T gscale;  // -1/(ks sigma^2): grad f = gscale * sum w phi (x' - c')
  T inv_eh;  // 1/eh: bin coordinates
  T R[9];
  T t[3];
  T z_off;
};

// Linearisation pose (R0 row-major, t0) passed by value.
struct Pose0 {
  double v[12];
};

// Evaluation-bin geometry in bin units. Row range and half-widths carry a
// pad that absorbs the FP32 rounding of the bin coordinates (the grid
// limits both bin counts to 2^14, so |u|, |v| < 2^14 and their rounding
// stays below 2^-9) and of the support test.
struct EGeom {
  float rbp;  // rb + pad: rows within this distance
  float rb2;  // (rb (1 + 1e-5))^2, rb = support radius in bins
  float pad;
  int32_t nbx, nby;
};
constexpr float EVAL_PAD = 1.0f / 64.0f;

// Fused multiply-adds written out where several kernels have to round alike
// (left to the compiler, the choice of the product to fuse varies).
__device__ inline double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ inline float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

__device__ inline double kexp_eval(double a) { return exp(a); }
__device__ inline float kexp_eval(float a) { return __builtin_amdgcn_exp2f(a); }

__device__ inline float idx_bits(int32_t i, float) { return __int_as_float(i); }
__device__ inline double idx_bits(int32_t i, double) { return (double)i; }
__device__ inline int32_t bits_idx(float v) { return __float_as_int(v); }
__device__ inline int32_t bits_idx(double v) { return (int32_t)v; }

// tab[s] = ((x - x0) ks, (y - y0) ks, w, original index) in evaluation-bin
// order.
template <typename T>
__global__ void __launch_bounds__(256) k_pack_centers(const double* __restrict__ ecxy,
                                                      const int32_t* __restrict__ eidx,
                                                      const double* __restrict__ w, int64_t n,
                                                      double x0, double y0, double ks,
                                                      typename Vec4<T>::type* __restrict__ tab) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= n) return;
  const int32_t i = eidx[s];
  typename Vec4<T>::type v;
  v.x = (T)((ecxy[2 * s] - x0) * ks);
  v.y = (T)((ecxy[2 * s + 1] - y0) * ks);
  v.z = (T)w[i];
  v.w = idx_bits(i, T(0));
  tab[s] = v;
}

// Mesh form: wt[n] = weight of the center on dense node n, 0 where none.
template <typename T>
__global__ void __launch_bounds__(256) k_pack_mesh(const int32_t* __restrict__ map,
                                                   const double* __restrict__ w, int64_t n,
                                                   T* __restrict__ wt) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= n) return;
  const int32_t c = map[s];
  wt[s] = c >= 0 ? (T)w[c] : (T)0;
}

// Lanes per point: the four lanes of a quad share a point and read
// consecutive table entries (one 64-byte segment per load instruction), so a
// wave's gather touches 16 cache lines instead of 64.
constexpr int LPP = 4;

// Value of lane SRC (0..3) of this lane's quad (DPP quad_perm broadcast).
template <int SRC>
__device__ inline int quad_bcast(int v) {
  return __builtin_amdgcn_mov_dpp(v, SRC * 0x55, 0xf, 0xf, false);
}
// Value of the lane whose quad index differs in the bits of CTRL's pattern
// (quad_perm [1,0,3,2] = 0xb1: lane ^ 1; [2,3,0,1] = 0x4e: lane ^ 2).
template <int CTRL>
__device__ inline float quad_swap(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ inline double quad_swap(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
// Value of lane SRC of this lane's quad, for a float or a double.
template <int SRC>
__device__ inline float quad_bcast_v(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), SRC * 0x55, 0xf, 0xf, false));
}
template <int SRC>
__device__ inline double quad_bcast_v(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), SRC * 0x55, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), SRC * 0x55, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <typename T>
__device__ inline T quad_bcast_any(T v, int src) {  // src known at compile time
  return src == 0 ? quad_bcast_v<0>(v)
                  : src == 1 ? quad_bcast_v<1>(v) : src == 2 ? quad_bcast_v<2>(v)
                                                             : quad_bcast_v<3>(v);
}

// Sum over the quad (butterfly over lanes ^1 and ^2; every lane gets it).
template <typename T>
__device__ inline T quad_sum(T v) {
  v += quad_swap<0xb1>(v);
  v += quad_swap<0x4e>(v);
  return v;
}

// Candidate run of one bin row of the point at bin coordinates (u, v): the
// eval-sorted entries [s0, s1) of the row's bins that the support circle
// meets, from the bin holding u - hw to the one holding u + hw (hw: the
// circle's half-width over the row, taken at the row's nearest edge less
// the pad, plus the pad); empty if the row is out of range (by > by1).
__device__ inline void row_run(float u, float v, int by, int by1, const EGeom& g,
                               const int32_t* __restrict__ estart, int& s0, int& s1) {
  const float fb = (float)by;
  const float dy = fmaxf(fmaxf(fb - v, v - fb - 1.f) - g.pad, 0.f);
  const float hw = sqrtf(fmaxf(g.rb2 - dy * dy, 0.f)) + g.pad;
  const int bx0 = max((int)floorf(u - hw), 0);
  const int bx1 = min((int)floorf(u + hw), g.nbx - 1);
  const bool valid = by <= by1 && bx0 <= bx1;
  const int row = min(by, g.nby - 1) * g.nbx;  // in range whether or not valid
  s0 = estart[valid ? row + bx0 : 0];
  s1 = valid ? estart[row + bx1 + 1] : s0;
}

// The point's candidate runs, one per bin row within the support (at most
// EVAL_MAX_ROWS = 8): lane `part` of the quad forms rows part and part + 4,
// and every lane receives all eight by quad broadcasts.
__device__ inline void quad_runs(float u, float v, int part, const EGeom& g,
                                 const int32_t* __restrict__ estart, int (&s0)[EVAL_MAX_ROWS],
                                 int (&s1)[EVAL_MAX_ROWS]) {
  static_assert(EVAL_MAX_ROWS == 2 * LPP, "two rows per lane");
  const bool ok = fabsf(u) < 16777216.f && fabsf(v) < 16777216.f;  // also NaN
  const int by0 = ok ? max((int)floorf(v - g.rbp), 0) : 0;
  const int by1 = ok ? min((int)floorf(v + g.rbp), g.nby - 1) : -1;
  int a0, a1, b0, b1;
  row_run(u, v, by0 + part, by1, g, estart, a0, a1);
  row_run(u, v, by0 + part + LPP, by1, g, estart, b0, b1);
  s0[0] = quad_bcast<0>(a0);
  s1[0] = quad_bcast<0>(a1);
  s0[1] = quad_bcast<1>(a0);
  s1[1] = quad_bcast<1>(a1);
  s0[2] = quad_bcast<2>(a0);
  s1[2] = quad_bcast<2>(a1);
  s0[3] = quad_bcast<3>(a0);
  s1[3] = quad_bcast<3>(a1);
  s0[4] = quad_bcast<0>(b0);
  s1[4] = quad_bcast<0>(b1);
  s0[5] = quad_bcast<1>(b0);
  s1[5] = quad_bcast<1>(b1);
  s0[6] = quad_bcast<2>(b0);
  s1[6] = quad_bcast<2>(b1);
  s0[7] = quad_bcast<3>(b0);
  s1[7] = quad_bcast<3>(b1);
}

// The packed table read through a buffer resource: 32-bit offsets, one
// address add per step with the second load's offset in the instruction,
// and reads past the table return zeros (a slot past a run's end needs no
// clamp; it is masked out by its index).
template <typename T>
struct TabReader {
  static constexpr bool AHEAD = false;
  using Slot = typename Vec4<T>::type;
  __amdgpu_buffer_rsrc_t r;
  __device__ TabReader(const typename Vec4<T>::type* tab, int64_t n) {
    r = __builtin_amdgcn_make_buffer_rsrc((void*)tab, (short)0,
                                          (int)(n * (int64_t)sizeof(typename Vec4<T>::type)),
                                          0x00020000);
  }
  // (x', y', w) of entry a + u, and its original index if IDX
  template <bool IDX>
  __device__ Slot load(int a, int off) const;
  template <bool IDX>
  __device__ Slot fetch(int a, int u) const {
    return load<IDX>(a, u * (int)sizeof(Slot));
  }
  __device__ void complete(Slot&) const {}
  __device__ Slot value(const Slot& s) const { return s; }
};
// (One 16-byte load; the compiler narrows it to the components used.)
template <>
template <bool IDX>
__device__ inline float4 TabReader<float>::load(int a, int off) const {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, a * 16 + off, 0, 0));
}
template <>
template <bool IDX>
__device__ inline double4 TabReader<double>::load(int a, int off) const {
  const double2 xy =
      __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, a * 32 + off, 0, 0));
  double4 c;
  c.x = xy.x;
  c.y = xy.y;
  if (IDX) {
    const double2 wi = __builtin_bit_cast(
        double2, __builtin_amdgcn_raw_buffer_load_b128(r, a * 32 + off + 16, 0, 0));
    c.z = wi.x;
    c.w = wi.y;
  } else {
    c.z = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, a * 32 + off + 16,
                                                                        0, 0));
    c.w = 0.0;
  }
  return c;
}

// The same entries formed from the grid's arrays and the weights as they are
// read: no packing launch, one more load behind the index. The operations are
// those of k_pack_centers. A slot behind the arrays' end has weight 0, as in the
// packed table: its index reads 0, and `off` takes the weight's load out of its
// resource (the weight of center 0 may not be finite, and phi = 0 would not mask
// it). The first slot of a step lies in its run.
template <typename T>
struct RawReader {
  static constexpr bool AHEAD = true;
  using Out = typename Vec4<T>::type;
  struct Slot {
    double2 xy;
    int32_t i, off;
    double w;
  };
  __amdgpu_buffer_rsrc_t rc, ri, rw;
  int32_t n;
  double x0, y0, ks;
  __device__ RawReader(const double* ecxy, const int32_t* eidx, const double* w, int64_t n_,
                       double x0_, double y0_, double ks_)
      : n((int32_t)n_), x0(x0_), y0(y0_), ks(ks_) {
    rc = __builtin_amdgcn_make_buffer_rsrc((void*)ecxy, (short)0, (int)(n_ * 16), 0x00020000);
    ri = __builtin_amdgcn_make_buffer_rsrc((void*)eidx, (short)0, (int)(n_ * 4), 0x00020000);
    rw = __builtin_amdgcn_make_buffer_rsrc((void*)w, (short)0, (int)(n_ * 8), 0x00020000);
  }
  template <bool IDX>
  __device__ Slot fetch(int a, int u) const {
    Slot s;
    s.xy = __builtin_bit_cast(double2,
                              __builtin_amdgcn_raw_buffer_load_b128(rc, a * 16 + u * 16, 0, 0));
    s.i = (int)__builtin_amdgcn_raw_buffer_load_b32(ri, a * 4 + u * 4, 0, 0);
    s.off = u > 0 && a + u >= n ? INT32_MIN : 0;
    s.w = 0.0;
    return s;
  }
  __device__ void complete(Slot& s) const {
    s.w = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rw, s.i * 8 | s.off, 0, 0));
  }
  __device__ Out value(const Slot& s) const {
#pragma clang fp contract(off)
    Out c;
    c.x = (T)((s.xy.x - x0) * ks);
    c.y = (T)((s.xy.y - y0) * ks);
    c.z = (T)s.w;
    c.w = idx_bits(s.i, T(0));
    return c;
  }
};

// Candidates per lane and step: the table loads of EU candidates (4 apart,
// the quad covering 4 EU consecutive entries) are issued together; a slot
// past the run is masked out.
template <typename T>
constexpr int eval_unroll() { return 2; }

// This lane's share of the point's candidates: in every run, the entries
// s0 + part, s0 + part + 4, ...; op(c, dx', dy', e) with e = phi, or 0
// outside the support (and for masked slots). c.w holds the original index
// only if IDX. Tab::AHEAD: the first step of a run is loaded while the run
// before it is summed (a load past a run's end is not used), so that a point's
// eight runs do not wait for memory one after the other; with enough
// wavefronts to hide the waits the registers it takes cost more.
template <typename T, bool IDX, typename Tab, typename Op>
__device__ inline void for_candidates(T xs, T ys, const Tab& tab,
                                      const int (&s0)[EVAL_MAX_ROWS],
                                      const int (&s1)[EVAL_MAX_ROWS], int part, T rc2s,
                                      Op op) {
  constexpr int EU = eval_unroll<T>();
  typename Tab::Slot next[EU];
  if constexpr (Tab::AHEAD) {
#pragma unroll
    for (int u = 0; u < EU; ++u) next[u] = tab.template fetch<IDX>(s0[0] + part, u * LPP);
  }
#pragma unroll
  for (int k = 0; k < EVAL_MAX_ROWS; ++k) {
    const int e = s1[k];
    typename Tab::Slot s[EU];
    if constexpr (Tab::AHEAD) {
#pragma unroll
      for (int u = 0; u < EU; ++u) {
        s[u] = next[u];
        tab.complete(s[u]);
      }
      if (k + 1 < EVAL_MAX_ROWS)
#pragma unroll
        for (int u = 0; u < EU; ++u) next[u] = tab.template fetch<IDX>(s0[k + 1] + part, u * LPP);
    }
    for (int a = s0[k] + part; a < e; a += EU * LPP) {
      if (!Tab::AHEAD || a != s0[k] + part) {
#pragma unroll
        for (int u = 0; u < EU; ++u) {
          s[u] = tab.template fetch<IDX>(a, u * LPP);
          tab.complete(s[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < EU; ++u) {
        const typename Vec4<T>::type c = tab.value(s[u]);
        const T dx = xs - c.x, dy = ys - c.y;
        const T d2 = fma_t(dx, dx, dy * dy);
        const T e0 = kexp_eval(-d2);
        const T ph = ((u == 0 || a + u * LPP < e) && d2 <= rc2s) ? e0 : (T)0;
        op(c, dx, dy, ph);
      }
    }
  }
}

// Point i: world coordinates relative to the grid origin (POSE: from the
// body point p, xi = R p + t).
template <typename T>
__device__ inline void pose_apply(const EvalK<T>& k, T px, T py, T pz, T& xr, T& yr, T& zw) {
  xr = (k.R[0] * px + k.R[1] * py + k.R[2] * pz + k.t[0]) - k.x0;
  yr = (k.R[3] * px + k.R[4] * py + k.R[5] * pz + k.t[1]) - k.y0;
  zw = k.R[6] * px + k.R[7] * py + k.R[8] * pz + k.t[2];
}
template <typename T, bool POSE>
__device__ inline void point_rel(const T* __restrict__ pts, int64_t i, const EvalK<T>& k, T& xr,
                                 T& yr, T& zw, T& px, T& py, T& pz) {
  if (POSE) {
    px = pts[3 * i];
    py = pts[3 * i + 1];
    pz = pts[3 * i + 2];
    pose_apply<T>(k, px, py, pz, xr, yr, zw);
  } else {
    const typename Vec2<T>::type p = reinterpret_cast<const typename Vec2<T>::type*>(pts)[i];
    xr = p.x - k.x0;
    yr = p.y - k.y0;
    zw = px = py = pz = (T)0;
  }
}

// The pose from device memory (R row-major, then t), when given there.
template <typename T>
__device__ inline void load_pose(EvalK<T>& k, const double* __restrict__ dpose) {
  if (!dpose) return;
#pragma unroll
  for (int q = 0; q < 9; ++q) k.R[q] = (T)dpose[q];
#pragma unroll
  for (int q = 0; q < 3; ++q) k.t[q] = (T)dpose[9 + q];
}

// f, sum w phi dx', sum w phi dy' at a point (coordinates relative to the
// grid origin), summed over the quad: every lane of the quad gets them.
template <typename T, typename Tab>
__device__ inline void sum_point(T xr, T yr, int part, const Tab& tab,
                                 const int32_t* __restrict__ estart, const EGeom& g,
                                 const EvalK<T>& k, T& f, T& sx, T& sy) {
  int s0[EVAL_MAX_ROWS], s1[EVAL_MAX_ROWS];
  quad_runs((float)(xr * k.inv_eh), (float)(yr * k.inv_eh), part, g, estart, s0, s1);
  T f_ = 0, sx_ = 0, sy_ = 0;
  for_candidates<T, false>(xr * k.ks, yr * k.ks, tab, s0, s1, part, k.rc2s,
                    [&](const typename Vec4<T>::type& c, T dx, T dy, T e) {
                      const T we = c.z * e;
                      f_ = fma_t(c.z, e, f_);
                      sx_ = fma_t(we, dx, sx_);
                      sy_ = fma_t(we, dy, sy_);
                    });
  f = quad_sum(f_);
  sx = quad_sum(sx_);
  sy = quad_sum(sy_);
}

// ---- mesh form (centers on the nodes of a square mesh)
//
// With every center a node (x0 + i res, y0 + j res) the Gaussian factors
// over the axes: phi = exp(-dx'^2) exp(-dy'^2). A point's support lies in a
// window of MW x MW nodes, whose weights are read from a dense node array
// (zero where no center, and in a margin of MW nodes around the mesh, so
// that no window needs a bounds test). Lane j of the quad takes the window
// columns j, j + 4, ...: per column one exponential, per row one; per node
// the support test, one product and two accumulations. Every quad does the
// same work, and the quad's loads cover consecutive nodes.

// Node geometry of one call.
template <typename T>
struct MGeom {
  T hs;       // node spacing in scaled coordinates (res ks)
  T inv_res;  // 1/res: node coordinates of a point relative to the mesh origin
  float rp;   // support radius in nodes plus MESH_PAD
  int32_t ilo, ihi, jlo, jhi;  // range of the window's first column / row
  int32_t ioff, joff;          // dense column / row of node 0
  int32_t pw;                  // dense row length (nodes)
};

// The dense node weights through a buffer resource (reads past the array
// return zeros; the clamped windows never reach them).
template <typename T>
struct MeshReader {
  __amdgpu_buffer_rsrc_t r;
  __device__ MeshReader(const T* wt, int64_t n) {
    r = __builtin_amdgcn_make_buffer_rsrc((void*)wt, (short)0, (int)(n * (int64_t)sizeof(T)),
                                          0x00020000);
  }
  __device__ T load(int voff, int soff) const;
};
template <>
__device__ inline float MeshReader<float>::load(int voff, int soff) const {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
template <>
__device__ inline double MeshReader<double>::load(int voff, int soff) const {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}

// f, sum w phi dx', sum w phi dy' at a point (coordinates relative to the
// mesh origin), summed over the quad.
template <typename T, int MW>
__device__ inline void sum_point_mesh(T xr, T yr, int part, const MeshReader<T>& wt,
                                      const MGeom<T>& m, const EvalK<T>& k, T& f, T& sx,
                                      T& sy) {
  constexpr int CPL = MW / LPP;  // columns per lane
  static_assert(CPL * LPP == MW, "window of whole quads");
  const float u = (float)(xr * m.inv_res), v = (float)(yr * m.inv_res);
  const bool ok = fabsf(u) < 16777216.f && fabsf(v) < 16777216.f;  // also NaN
  const int i0 = ok ? min(max((int)ceilf(u - m.rp), m.ilo), m.ihi) : m.ilo;
  const int j0 = ok ? min(max((int)ceilf(v - m.rp), m.jlo), m.jhi) : m.jlo;
  // a point with no finite node coordinates is moved far off the mesh (no
  // node in its support, every factor exp(-d'^2) zero): f = 0, as binned
  const T xs = ok ? xr * k.ks : (T)1e18, ys = ok ? yr * k.ks : (T)1e18;
  T dx[CPL], dx2[CPL], cs[CPL], cy[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    dx[q] = xs - (T)(i0 + part + LPP * q) * m.hs;
    dx2[q] = dx[q] * dx[q];
    cs[q] = 0;
    cy[q] = 0;
  }
  // row factors: lane j forms those of rows j, j + 4, ... and the quad
  // shares them by broadcasts
  T eown[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const T dyq = ys - (T)(j0 + part + LPP * q) * m.hs;
    eown[q] = kexp_eval(-(dyq * dyq));
  }
  constexpr int SZ = (int)sizeof(T);
  const int voff = ((j0 + m.joff) * m.pw + (i0 + m.ioff + part)) * SZ;
  const int rowb = m.pw * SZ;
#pragma unroll
  for (int r = 0; r < MW; ++r) {
    const T dy = ys - (T)(j0 + r) * m.hs;
    const T dy2 = dy * dy;
    const T ey = quad_bcast_any(eown[r / LPP], r % LPP);
    const T lim = k.rc2s - dy2;  // node in the support iff dx'^2 <= lim
    T w[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) w[q] = wt.load(voff + q * LPP * SZ, r * rowb);
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const T pq = w[q] * ey;
      const T pm = dx2[q] <= lim ? pq : (T)0;
      cs[q] += pm;
      cy[q] += pm * dy;
    }
  }
  T f_ = 0, sx_ = 0, sy_ = 0;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    const T ex = kexp_eval(-dx2[q]);
    const T a = ex * cs[q];
    f_ += a;
    sx_ += a * dx[q];
    sy_ += ex * cy[q];
  }
  f = quad_sum(f_);
  sx = quad_sum(sx_);
  sy = quad_sum(sy_);
}

// ---- mesh form with the node weights in LDS
//
// One workgroup per CU keeps the whole dense node array in LDS,
// filled straight from the weights (no packing launch), and takes a share of
// the points, one lane per point. The quad form forms a point's setup, pose
// and outputs in four lanes and its window loads keep the L1 busy (a wave's 16
// loads of a window touch 64 to 128 lines each); here a lane reads its window's
// rows from LDS. Every sum is taken in the quad form's order (columns j,
// j + 4, ... of lane j, then the butterfly), so the two forms agree bit for
// bit. 5,000,000 FP32 points on 100 x 100 centers: 174 -> 85 us; 200,000: 9.7 +
// 2.4 (packing) -> 11.2 us and a launch less. Bound by the FP32 VALU (about 600
// instructions per wavefront of 64 points), at a scan's size by filling the LDS
// and the launch.

// Nodes of the dense array that one CU's LDS holds beside the reductions.
constexpr int64_t MESH_LDS_BYTES = 152 * 1024;

template <typename T>
struct MeshTab {
  const int32_t* map;  // center of each dense node, -1: none
  const double* w;
  int32_t n;           // dense nodes
  MGeom<T> mg;
};

// Fill the LDS table. All loads of a step are issued before the first use.
template <typename T>
__device__ inline void fill_mesh(const MeshTab<T>& t, T* wt, int tid, int nt) {
  constexpr int U = 16;
  for (int e0 = tid; e0 < t.n; e0 += U * nt) {
    int c[U];
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = t.map[min(e0 + u * nt, t.n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = t.w[max(c[u], 0)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (e0 + u * nt < t.n) wt[e0 + u * nt] = c[u] >= 0 ? (T)v[u] : (T)0;
  }
}

// f, sum w phi dx', sum w phi dy' of one lane's point.
template <typename T, int MW>
__device__ inline void sum_lane_mesh(T xr, T yr, const T* wt, const MGeom<T>& m,
                                     const EvalK<T>& k, T& f, T& sx, T& sy) {
  const float u = (float)(xr * m.inv_res), v = (float)(yr * m.inv_res);
  const bool ok = fabsf(u) < 16777216.f && fabsf(v) < 16777216.f;  // also NaN
  const int i0 = ok ? min(max((int)ceilf(u - m.rp), m.ilo), m.ihi) : m.ilo;
  const int j0 = ok ? min(max((int)ceilf(v - m.rp), m.jlo), m.jhi) : m.jlo;
  const T xs = ok ? xr * k.ks : (T)1e18, ys = ok ? yr * k.ks : (T)1e18;
  T dx[MW], dx2[MW], cs[MW], cy[MW];
#pragma unroll
  for (int q = 0; q < MW; ++q) {
    dx[q] = xs - (T)(i0 + q) * m.hs;
    dx2[q] = dx[q] * dx[q];
    cs[q] = 0;
    cy[q] = 0;
  }
  const T* row = wt + (j0 + m.joff) * m.pw + (i0 + m.ioff);
#pragma unroll
  for (int r = 0; r < MW; ++r, row += m.pw) {
    T w[MW];
#pragma unroll
    for (int q = 0; q < MW; ++q) w[q] = row[q];
    const T dy = ys - (T)(j0 + r) * m.hs;
    const T dy2 = dy * dy;
    const T ey = kexp_eval(-dy2);
    const T lim = k.rc2s - dy2;
#pragma unroll
    for (int q = 0; q < MW; ++q) {
      const T pq = w[q] * ey;
      const T pm = dx2[q] <= lim ? pq : (T)0;
      cs[q] += pm;
      cy[q] += pm * dy;
    }
  }
  T f_[LPP], sx_[LPP], sy_[LPP];
#pragma unroll
  for (int j = 0; j < LPP; ++j) {
    f_[j] = sx_[j] = sy_[j] = 0;
#pragma unroll
    for (int q = j; q < MW; q += LPP) {
      const T ex = kexp_eval(-dx2[q]);
      const T a = ex * cs[q];
      f_[j] += a;
      sx_[j] += a * dx[q];
      sy_[j] += ex * cy[q];
    }
  }
  f = (f_[0] + f_[1]) + (f_[2] + f_[3]);
  sx = (sx_[0] + sx_[1]) + (sx_[2] + sx_[3]);
  sy = (sy_[0] + sy_[1]) + (sy_[2] + sy_[3]);
}

// Threads of a workgroup: as many waves as the registers of a window allow.
template <typename T, int MW>
constexpr int mesh_threads() {
  return MW == 4 || (sizeof(T) == 4 && MW == 8) ? 1024 : 512;
}
// Points of a workgroup: whole waves, over MESH_WGS workgroups at most.
constexpr int64_t MESH_WGS = 256;
static inline int64_t mesh_share(int64_t Q) { return ceil_div(ceil_div(Q, MESH_WGS), 64) * 64; }

// Neighbour structure of a call: the binned table (MW = 0), the grid's arrays
// (MW = -1) or the dense node weights of the mesh form (MW = window).
template <typename T>
struct Nbr {
  const void* tab;        // packed table (n entries) or node weights (n nodes)
  int64_t n;
  const int32_t* estart;  // binned form
  EGeom eg;               // binned form
  MGeom<T> mg;            // mesh form
  const double* ecxy;     // binned form read as it is (MW = -1)
  const int32_t* eidx;
  const double* w;
  double x0, y0, ks;
};

template <typename T, int MW>
__device__ inline void sum_nbr(T xr, T yr, int part, const Nbr<T>& nb, const EvalK<T>& k, T& f,
                               T& sx, T& sy) {
  if constexpr (MW == 0) {
    const TabReader<T> tab((const typename Vec4<T>::type*)nb.tab, nb.n);
    sum_point<T>(xr, yr, part, tab, nb.estart, nb.eg, k, f, sx, sy);
  } else if constexpr (MW < 0) {
    const RawReader<T> tab(nb.ecxy, nb.eidx, nb.w, nb.n, nb.x0, nb.y0, nb.ks);
    sum_point<T>(xr, yr, part, tab, nb.estart, nb.eg, k, f, sx, sy);
  } else {
    const MeshReader<T> wt((const T*)nb.tab, nb.n);
    sum_point_mesh<T, MW>(xr, yr, part, wt, nb.mg, k, f, sx, sy);
  }
}

// A point's outputs; its LP lanes share the stores.
template <typename T, bool POSE, int LP>
__device__ inline void write_point(int64_t i, int part, const EvalK<T>& k, T px, T py, T pz, T zw,
                                   T f, T sx, T sy, T* __restrict__ f_out,
                                   T* __restrict__ grad_out, T* __restrict__ r_out,
                                   T* __restrict__ jac_out) {
  using T2 = typename Vec2<T>::type;
  const T fx = sx * k.gscale, fy = sy * k.gscale;
  if (part == 0) f_out[i] = f;
  if (grad_out && part == 1 % LP) {
    T2 gv;
    gv.x = fx;
    gv.y = fy;
    reinterpret_cast<T2*>(grad_out)[i] = gv;
  }
  if (POSE) {
    if (r_out && part == 2 % LP) r_out[i] = zw - k.z_off - f;
    if (jac_out && part == 3 % LP) {
      // g = (-fx, -fy, 1); q = R^T g; J_rot = p x q
      const T g0 = -fx, g1 = -fy, g2 = (T)1;
      const T q0 = k.R[0] * g0 + k.R[3] * g1 + k.R[6] * g2;
      const T q1 = k.R[1] * g0 + k.R[4] * g1 + k.R[7] * g2;
      const T q2 = k.R[2] * g0 + k.R[5] * g1 + k.R[8] * g2;
      T2* J = reinterpret_cast<T2*>(jac_out + 6 * i);  // 6 i elements: T2-aligned
      T2 j01, j23, j45;
      j01.x = py * q2 - pz * q1;
      j01.y = pz * q0 - px * q2;
      j23.x = px * q1 - py * q0;
      j23.y = g0;
      j45.x = g1;
      j45.y = g2;
      J[0] = j01;
      J[1] = j23;
      J[2] = j45;
    }
  }
}

template <typename T, bool POSE, int MW>
__global__ void __launch_bounds__(256) k_eval(const T* __restrict__ pts, int64_t Q, Nbr<T> nb,
                                              EvalK<T> k0, const double* __restrict__ dpose,
                                              T* __restrict__ f_out, T* __restrict__ grad_out,
                                              T* __restrict__ r_out, T* __restrict__ jac_out) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LPP;
  const int part = threadIdx.x % LPP;
  if (i >= Q) return;  // the lanes of a quad leave together
  EvalK<T> k = k0;
  if (POSE) load_pose(k, dpose);
  T xr, yr, zw, px, py, pz;
  point_rel<T, POSE>(pts, i, k, xr, yr, zw, px, py, pz);
  T f, sx, sy;
  sum_nbr<T, MW>(xr, yr, part, nb, k, f, sx, sy);
  write_point<T, POSE, LPP>(i, part, k, px, py, pz, zw, f, sx, sy, f_out, grad_out, r_out,
                            jac_out);
}

template <typename T, bool POSE, int MW>
__global__ void __launch_bounds__((mesh_threads<T, MW>())) k_eval_lds(
    const T* __restrict__ pts, int64_t Q, int64_t share, MeshTab<T> mt, EvalK<T> k0,
    const double* __restrict__ dpose, T* __restrict__ f_out, T* __restrict__ grad_out,
    T* __restrict__ r_out, T* __restrict__ jac_out) {
  extern __shared__ char smem[];
  T* wt = (T*)smem;
  const int tid = threadIdx.x;
  constexpr int NT = mesh_threads<T, MW>();
  fill_mesh<T>(mt, wt, tid, NT);
  EvalK<T> k = k0;
  if (POSE) load_pose(k, dpose);
  __syncthreads();
  const int64_t end = min((blockIdx.x + 1) * share, Q);
  for (int64_t i = blockIdx.x * share + tid; i < end; i += NT) {
    T xr, yr, zw, px, py, pz;
    point_rel<T, POSE>(pts, i, k, xr, yr, zw, px, py, pz);
    T f, sx, sy;
    sum_lane_mesh<T, MW>(xr, yr, wt, mt.mg, k, f, sx, sy);
    write_point<T, POSE, 1>(i, 0, k, px, py, pz, zw, f, sx, sy, f_out, grad_out, r_out, jac_out);
  }
}

// ---- Gauss-Newton terms of the manifold residual (fused, J not written)

constexpr int GN_TERMS = 28;  // 21 upper entries of J^T J, 6 of J^T r, r^2
constexpr int64_t GN_MAX_BLOCKS = 1536;  // six waves per SIMD of 256 CUs

// Products of the 28 terms, the quad's lanes taking 7 each: lane j of a
// quad accumulates terms 7 j .. 7 j + 6 of the list (J0J0, J0J1, ..., J0J5,
// J1J1, ..., J5J5, J0 r, ..., J5 r, r r) into v[0..6]. Every lane of the
// quad holds the point's J and r, so the lanes' shares need no exchange.
__device__ inline void gn_share(int lp, const double (&J)[6], double r, double (&v)[7]) {
  switch (lp) {
    case 0:  // J0 J0..J5, J1 J1
      v[0] += J[0] * J[0]; v[1] += J[0] * J[1]; v[2] += J[0] * J[2]; v[3] += J[0] * J[3];
      v[4] += J[0] * J[4]; v[5] += J[0] * J[5]; v[6] += J[1] * J[1];
      break;
    case 1:  // J1 J2..J5, J2 J2..J4
      v[0] += J[1] * J[2]; v[1] += J[1] * J[3]; v[2] += J[1] * J[4]; v[3] += J[1] * J[5];
      v[4] += J[2] * J[2]; v[5] += J[2] * J[3]; v[6] += J[2] * J[4];
      break;
    case 2:  // J2 J5, J3 J3..J5, J4 J4, J4 J5, J5 J5
      v[0] += J[2] * J[5]; v[1] += J[3] * J[3]; v[2] += J[3] * J[4]; v[3] += J[3] * J[5];
      v[4] += J[4] * J[4]; v[5] += J[4] * J[5]; v[6] += J[5] * J[5];
      break;
    default:  // J0..J5 r, r r
      v[0] += J[0] * r; v[1] += J[1] * r; v[2] += J[2] * r; v[3] += J[3] * r;
      v[4] += J[4] * r; v[5] += J[5] * r; v[6] += r * r;
      break;
  }
}

// A point's residual and pose Jacobian row, in FP64.
template <typename T>
__device__ inline void gn_row(const EvalK<T>& k, T px, T py, T pz, T zw, T f, T sx, T sy,
                              double (&J)[6], double& r) {
  const double fx = (double)sx * (double)k.gscale, fy = (double)sy * (double)k.gscale;
  r = (double)zw - (double)k.z_off - (double)f;
  const double g0 = -fx, g1 = -fy, g2 = 1.0;
  const double q0 = (double)k.R[0] * g0 + (double)k.R[3] * g1 + (double)k.R[6] * g2;
  const double q1 = (double)k.R[1] * g0 + (double)k.R[4] * g1 + (double)k.R[7] * g2;
  const double q2 = (double)k.R[2] * g0 + (double)k.R[5] * g1 + (double)k.R[8] * g2;
  J[0] = (double)py * q2 - (double)pz * q1;
  J[1] = (double)pz * q0 - (double)px * q2;
  J[2] = (double)px * q1 - (double)py * q0;
  J[3] = g0;
  J[4] = g1;
  J[5] = g2;
}

// Term q's sum to its place: J^T J (both triangles), J^T r, r^T r.
__device__ inline void gn_store(int q, double s, double* __restrict__ JtJ,
                                double* __restrict__ Jtr, double* __restrict__ rtr) {
  if (q < 21) {
    int a = 0, rem = q;
    while (rem >= 6 - a) {
      rem -= 6 - a;
      ++a;
    }
    const int b = a + rem;
    JtJ[a * 6 + b] = s;
    JtJ[b * 6 + a] = s;
  } else if (q < 27) {
    Jtr[q - 21] = s;
  } else if (rtr) {
    *rtr = s;
  }
}

// Each quad takes points i, i + stride, ... (grid-stride; the launch is a
// fixed function of Q) and its lanes accumulate their shares of the points'
// 28 products in FP64 registers (gn_share). The block's sums go through
// LDS: the 64 lane values of each term (16 quads x 4 waves) are added in
// eight runs of eight by 224 threads, then the eight run sums in order by 28
// threads, into part[term][block] (term-major, gridDim.x blocks).
template <typename T, int MW>
__global__ void __launch_bounds__(256) k_eval_gn(const T* __restrict__ pts, int64_t Q, Nbr<T> nb,
                                                 EvalK<T> k, double* __restrict__ part) {
  static_assert(GN_TERMS == 7 * LPP, "seven terms per lane of a quad");
  __shared__ double lv[256 * 7];           // [thread][7]
  __shared__ double runs[GN_TERMS * 8];    // [term][run]
  const int tid = threadIdx.x;
  const int lp = tid % LPP;
  double v[7] = {0, 0, 0, 0, 0, 0, 0};
  const int64_t stride = (int64_t)gridDim.x * (256 / LPP);
  for (int64_t i = ((int64_t)blockIdx.x * 256 + tid) / LPP; i < Q; i += stride) {
    T xr, yr, zw, px, py, pz;
    point_rel<T, true>(pts, i, k, xr, yr, zw, px, py, pz);
    T f, sx, sy;
    sum_nbr<T, MW>(xr, yr, lp, nb, k, f, sx, sy);
    double J[6], r;
    gn_row<T>(k, px, py, pz, zw, f, sx, sy, J, r);
    gn_share(lp, J, r, v);
  }
#pragma unroll
  for (int q = 0; q < 7; ++q) lv[tid * 7 + q] = v[q];
  __syncthreads();
  if (tid < GN_TERMS * 8) {
    // term 7 lp + q lives in the threads of lane lp of every quad
    const int term = tid >> 3, run = tid & 7;
    const int tl = term / 7, tq = term % 7;
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) s += lv[((run * 8 + j) * LPP + tl) * 7 + tq];
    runs[tid] = s;
  }
  __syncthreads();
  if (tid < GN_TERMS) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) s += runs[tid * 8 + j];
    part[(int64_t)tid * gridDim.x + blockIdx.x] = s;
  }
}

// Sum the block partials in a fixed order, one workgroup per term:
// thread t adds the partials t, t + 256, ... of its term (every load issued
// before the first add), then the 256 sums meet in a fixed tree. Writes
// J^T J (6x6, both triangles), J^T r (6) and r^T r.
constexpr int GN_SUM_T = 256;
constexpr int GN_SUM_LOADS = (int)((GN_MAX_BLOCKS + GN_SUM_T - 1) / GN_SUM_T);
__global__ void __launch_bounds__(GN_SUM_T) k_eval_gn_sum(const double* __restrict__ part,
                                                          int64_t nblocks,
                                                          double* __restrict__ JtJ,
                                                          double* __restrict__ Jtr,
                                                          double* __restrict__ rtr) {
  __shared__ double red[GN_SUM_T];
  const int t = threadIdx.x, q = blockIdx.x;
  const double* __restrict__ p = part + (int64_t)q * nblocks;
  double v[GN_SUM_LOADS];
#pragma unroll
  for (int u = 0; u < GN_SUM_LOADS; ++u) {
    const int64_t e = t + (int64_t)u * GN_SUM_T;
    v[u] = e < nblocks ? p[e] : 0.0;
  }
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < GN_SUM_LOADS; ++u) s += v[u];
  red[t] = s;
  __syncthreads();
#pragma unroll
  for (int o = GN_SUM_T / 2; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  if (t == 0) gn_store(q, red[0], JtJ, Jtr, rtr);
}

// Mesh form with the node weights in LDS, one lane per point: the lane adds its
// point's 28 products itself (the quad's lanes each formed J and took turns
// with 7). Fixed orders throughout: a lane's points, the lanes of a term.
constexpr int GN_LDS_NT = 512;
template <typename T, int MW>
__global__ void __launch_bounds__(GN_LDS_NT) k_gn_lds(
    const T* __restrict__ pts, int64_t Q, int64_t share, MeshTab<T> mt, EvalK<T> k,
    double* __restrict__ part) {
  extern __shared__ char smem[];
  T* wt = (T*)smem;
  constexpr int NT = GN_LDS_NT;
  const int tid = threadIdx.x;
  fill_mesh<T>(mt, wt, tid, NT);
  __syncthreads();
  double v[GN_TERMS];
#pragma unroll
  for (int q = 0; q < GN_TERMS; ++q) v[q] = 0.0;
  const int64_t end = min((blockIdx.x + 1) * share, Q);
  for (int64_t i = blockIdx.x * share + tid; i < end; i += NT) {
    T xr, yr, zw, px, py, pz;
    point_rel<T, true>(pts, i, k, xr, yr, zw, px, py, pz);
    T f, sx, sy;
    sum_lane_mesh<T, MW>(xr, yr, wt, mt.mg, k, f, sx, sy);
    double J[6], r;
    gn_row<T>(k, px, py, pz, zw, f, sx, sy, J, r);
#pragma unroll
    for (int a = 0, q = 0; a < 6; ++a)
#pragma unroll
      for (int b = a; b < 6; ++b, ++q) v[q] += J[a] * J[b];
#pragma unroll
    for (int a = 0; a < 6; ++a) v[21 + a] += J[a] * r;
    v[27] += r * r;
  }
  // the LDS serves the reduction from here on, [term][thread]: 16 lanes per term
  // add 32 values each, then meet in a butterfly (one barrier; seven terms at a
  // time took nine: 200,000 FP32 points 15.9 -> 13.5 us)
  double* lv = (double*)smem;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < GN_TERMS; ++q) lv[q * NT + tid] = v[q];
  __syncthreads();
  if (tid < GN_TERMS * 16) {
    const double* p = lv + (tid >> 4) * NT + (tid & 15);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < NT / 16; ++j) s[j & 3] += p[16 * j];
    double t = (s[0] + s[1]) + (s[2] + s[3]);
    for (int o = 8; o > 0; o >>= 1) t += __shfl_xor(t, o, 16);
    if ((tid & 15) == 0) part[(tid >> 4) * (int64_t)gridDim.x + blockIdx.x] = t;
  }
}

// Adjoint: L = sum_i gf_i f_i + gr_i r_i. With a_i = gf_i - gr_i:
//   dL/dw_j   = sum_i a_i phi(xi_i, c_j)            (scattered)
//   dL/dxi_i  = (a_i f_x, a_i f_y, gr_i),  dL/dp_i = R^T dL/dxi_i
//   dL/dpose  = sum_i [p_i x (R^T dL/dxi_i), dL/dxi_i]  (block-reduced)
//
// dL/dw takes about 28 FP64 additions per point. PLANES: one workgroup per CU
// takes a share of the points, adds in LDS (ds_add_f64) and leaves its N sums
// in a plane of its own, which k_adjoint_sum adds up. Else every addition is a
// device atomic, and these bound the kernel (5.6 million of them at 200,000
// points). 200,000 FP64 points, 10,000 centers: 192 us with device atomics,
// 40 + 7 us with planes (30 + 7 by the mesh form), bound by the FP64
// exponentials of the candidates and the LDS additions.
constexpr int64_t ADJ_PLANES = 256;            // one workgroup per CU
// Its threads: four waves per SIMD; three for the mesh form's 8-node windows,
// whose FP64 registers do not fit four (200,000 points 42.0 -> 41.3 us).
template <int MW>
constexpr int adj_threads() { return MW == 8 ? 768 : 1024; }
constexpr int64_t ADJ_LDS_N = 18 * 1024;       // 144 KB of sums
constexpr int64_t ADJ_MIN_PLANES = 16;         // 256 points each

// Mesh form of a point's share in the planes form: sum w phi dx', sum w phi dy'
// and a phi added to the nodes of hw (a node without a center collects what
// k_adjoint_sum leaves out). Laid out as sum_point_mesh; one exponential per
// window row and column instead of one per candidate.
template <typename T, int MW>
__device__ inline void adjoint_point_mesh(T xr, T yr, int part, const MeshReader<T>& wt,
                                          const MGeom<T>& m, const EvalK<T>& k, T a, bool scatter,
                                          double* hw, T& sx, T& sy) {
  constexpr int CPL = MW / LPP;
  const float u = (float)(xr * m.inv_res), v = (float)(yr * m.inv_res);
  const bool ok = fabsf(u) < 16777216.f && fabsf(v) < 16777216.f;  // also NaN
  const int i0 = ok ? min(max((int)ceilf(u - m.rp), m.ilo), m.ihi) : m.ilo;
  const int j0 = ok ? min(max((int)ceilf(v - m.rp), m.jlo), m.jhi) : m.jlo;
  const T xs = ok ? xr * k.ks : (T)1e18, ys = ok ? yr * k.ks : (T)1e18;
  T dx[CPL], dx2[CPL], ex[CPL], cs[CPL], cy[CPL], eown[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    dx[q] = xs - (T)(i0 + part + LPP * q) * m.hs;
    dx2[q] = dx[q] * dx[q];
    ex[q] = kexp_eval(-dx2[q]);
    cs[q] = 0;
    cy[q] = 0;
    const T dyq = ys - (T)(j0 + part + LPP * q) * m.hs;
    eown[q] = kexp_eval(-(dyq * dyq));
  }
  constexpr int SZ = (int)sizeof(T);
  const int node = (j0 + m.joff) * m.pw + (i0 + m.ioff + part);
#pragma unroll
  for (int r = 0; r < MW; ++r) {
    const T dy = ys - (T)(j0 + r) * m.hs;
    const T ey = quad_bcast_any(eown[r / LPP], r % LPP);
    const T lim = k.rc2s - dy * dy;  // node in the support iff dx'^2 <= lim
    T w[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) w[q] = wt.load(node * SZ + q * LPP * SZ, r * m.pw * SZ);
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      const bool in = dx2[q] <= lim;
      const T pm = in ? w[q] * ey : (T)0;
      cs[q] += pm;
      cy[q] += pm * dy;
      const T e = ex[q] * ey;
      if (scatter && in && e != (T)0)
        atomicAdd(&hw[node + q * LPP + r * m.pw], (double)(a * e));
    }
  }
  T sx_ = 0, sy_ = 0;
#pragma unroll
  for (int q = 0; q < CPL; ++q) {
    sx_ += ex[q] * cs[q] * dx[q];
    sy_ += ex[q] * cy[q];
  }
  sx = quad_sum(sx_);
  sy = quad_sum(sy_);
}

// MW: 0, the binned form, or (PLANES) the mesh form's window.
template <typename T, bool POSE, bool PLANES, int MW>
__global__ void __launch_bounds__((PLANES ? adj_threads<MW>() : 256)) k_eval_adjoint(
    const T* __restrict__ pts, int64_t Q, Nbr<T> nb, EvalK<T> k0,
    const double* __restrict__ dpose,
    const T* __restrict__ gbar_f, const T* __restrict__ gbar_r, T* __restrict__ d_pts,
    double* __restrict__ d_w, double* __restrict__ d_pose) {
  constexpr int NT = PLANES ? adj_threads<MW>() : 256, PPB = NT / LPP;
  extern __shared__ double hw[];  // PLANES: this workgroup's dL/dw
  const int64_t N = nb.n;
  const int part = threadIdx.x % LPP;
  EvalK<T> k = k0;
  if (POSE) load_pose(k, dpose);
  double acc[6] = {0, 0, 0, 0, 0, 0};
  // one point of a quad (its lanes come together)
  const auto point = [&](int64_t i) {
    T xr, yr, zw, px, py, pz;
    point_rel<T, POSE>(pts, i, k, xr, yr, zw, px, py, pz);
    const T gf = gbar_f ? gbar_f[i] : (T)0;
    const T gr = (POSE && gbar_r) ? gbar_r[i] : (T)0;
    const T a = gf - gr;
    T sx = 0, sy = 0;
    const bool scatter = d_w && a != (T)0;
    if constexpr (MW == 0) {
      const TabReader<T> tab((const typename Vec4<T>::type*)nb.tab, N);
      int s0[EVAL_MAX_ROWS], s1[EVAL_MAX_ROWS];
      quad_runs((float)(xr * k.inv_eh), (float)(yr * k.inv_eh), part, nb.eg, nb.estart, s0, s1);
      for_candidates<T, true>(xr * k.ks, yr * k.ks, tab, s0, s1, part, k.rc2s,
                              [&](const typename Vec4<T>::type& c, T dx, T dy, T e) {
                          const T we = c.z * e;
                          sx = fma_t(we, dx, sx);
                          sy = fma_t(we, dy, sy);
                          if (scatter && e != (T)0) {
                            if (PLANES)
                              atomicAdd(&hw[bits_idx(c.w)], (double)(a * e));
                            else
                              atomicAdd(&d_w[bits_idx(c.w)], (double)(a * e));
                          }
                        });
      sx = quad_sum(sx);
      sy = quad_sum(sy);
    } else {
      const MeshReader<T> wt((const T*)nb.tab, N);
      adjoint_point_mesh<T, MW>(xr, yr, part, wt, nb.mg, k, a, scatter, hw, sx, sy);
    }
    const T fx = sx * k.gscale, fy = sy * k.gscale;
    const T dx0 = a * fx, dx1 = a * fy, dx2 = gr;
    if (POSE) {
      const T q0 = k.R[0] * dx0 + k.R[3] * dx1 + k.R[6] * dx2;
      const T q1 = k.R[1] * dx0 + k.R[4] * dx1 + k.R[7] * dx2;
      const T q2 = k.R[2] * dx0 + k.R[5] * dx1 + k.R[8] * dx2;
      if (part == 0) {  // one lane of the quad writes and adds the point
        if (d_pts) {
          d_pts[3 * i] = q0;
          d_pts[3 * i + 1] = q1;
          d_pts[3 * i + 2] = q2;
        }
        acc[0] += (double)(py * q2 - pz * q1);
        acc[1] += (double)(pz * q0 - px * q2);
        acc[2] += (double)(px * q1 - py * q0);
        acc[3] += (double)dx0;
        acc[4] += (double)dx1;
        acc[5] += (double)dx2;
      }
    } else if (d_pts && part == 0) {
      d_pts[2 * i] = dx0;
      d_pts[2 * i + 1] = dx1;
    }
  };
  int64_t i = (int64_t)blockIdx.x * PPB + threadIdx.x / LPP;
  if constexpr (PLANES) {
    const int64_t share = (Q + gridDim.x - 1) / gridDim.x;
    const int64_t end = min((blockIdx.x + 1) * share, Q);
    for (int e = threadIdx.x; e < N; e += NT) hw[e] = 0.0;
    __syncthreads();
    for (i = blockIdx.x * share + threadIdx.x / LPP; i < end; i += PPB) point(i);
  } else if (i < Q) {
    // no loop: the sums of the pose's gradient kept across one cost 16 registers
    // and a wavefront per SIMD (FP64, 72,900 points, 1.5 m apart: 35 -> 31 us)
    point(i);
  }
  if (POSE && d_pose) {
    __shared__ double red[6][NT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      double v = acc[c];
      for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
      if (lane == 0) red[c][wave] = v;
    }
    __syncthreads();
    if (threadIdx.x < 6) {
      double v = red[threadIdx.x][0];
      for (int q = 1; q < NT / 64; ++q) v += red[threadIdx.x][q];
      atomicAdd(&d_pose[threadIdx.x], v);
    }
  }
  if (PLANES) {
    __syncthreads();
    for (int e = threadIdx.x; e < N; e += NT) d_w[blockIdx.x * N + e] = hw[e];
  }
}

// d_w += the planes: 64 centers per workgroup, 16 waves over the planes. map:
// the center of each of the N nodes (mesh form), or null.
__global__ void __launch_bounds__(1024) k_adjoint_sum(const double* __restrict__ plane,
                                                      int planes, int64_t N,
                                                      const int32_t* __restrict__ map,
                                                      double* __restrict__ d_w) {
  __shared__ double s[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + lane;
  double v = 0.0;
  if (e < N)
    for (int q = w; q < planes; q += 16) v += plane[q * N + e];
  s[w][lane] = v;
  __syncthreads();
  if (w != 0 || e >= N) return;
  for (int q = 1; q < 16; ++q) v += s[q][lane];
  const int64_t c = map ? map[e] : e;
  if (c >= 0 && v != 0.0) atomicAdd(&d_w[c], v);  // other calls may add to d_w at the same time
}

// ---- pose increments on SO(3) x R^3 (differentiation form)
//
// R = R0 Exp(dtheta), t = t0 + dt, and the right Jacobian J_r(dtheta)
// (Exp(v + e) = Exp(v) Exp(J_r(v) e) to first order), from the closed forms
// of the exponential map of SO(3) (Rodrigues' formula):
//   Exp(v) = I + a K + b K^2,   J_r(v) = I - b K + c K^2,
//   K = [v]_x, th = |v|, a = sin th / th, b = (1 - cos th) / th^2,
//   c = (th - sin th) / th^3,
// with 1 - cos th = 2 sin^2(th/2) and Taylor series of a, b, c for small th
// (no cancellation). Out: pose[12] (R row-major, t), jr[9] row-major.
__global__ void k_pose_exp(Pose0 p0, const double* __restrict__ delta, double* __restrict__ out) {
  if (threadIdx.x != 0) return;
  const double v0 = delta[0], v1 = delta[1], v2 = delta[2];
  const double t2 = v0 * v0 + v1 * v1 + v2 * v2, th = sqrt(t2);
  double a, b, c;
  if (th < 1e-2) {
    a = 1.0 - t2 / 6.0 * (1.0 - t2 / 20.0 * (1.0 - t2 / 42.0));
    b = 0.5 * (1.0 - t2 / 12.0 * (1.0 - t2 / 30.0 * (1.0 - t2 / 56.0)));
  } else {
    const double sh = sin(0.5 * th);
    a = sin(th) / th;
    b = 2.0 * sh * sh / t2;
  }
  if (th < 1e-1)
    c = (1.0 - t2 / 20.0 * (1.0 - t2 / 42.0 * (1.0 - t2 / 72.0 * (1.0 - t2 / 110.0)))) / 6.0;
  else
    c = (th - sin(th)) / (t2 * th);
  const double K[9] = {0.0, -v2, v1, v2, 0.0, -v0, -v1, v0, 0.0};
  double K2[9];
  for (int r = 0; r < 3; ++r)
    for (int q = 0; q < 3; ++q)
      K2[3 * r + q] = K[3 * r] * K[q] + K[3 * r + 1] * K[3 + q] + K[3 * r + 2] * K[6 + q];
  double E[9];
  for (int e = 0; e < 9; ++e) {
    const double id = (e % 4 == 0) ? 1.0 : 0.0;
    E[e] = id + a * K[e] + b * K2[e];
    out[12 + e] = id - b * K[e] + c * K2[e];
  }
  for (int r = 0; r < 3; ++r)
    for (int q = 0; q < 3; ++q)
      out[3 * r + q] =
          p0.v[3 * r] * E[q] + p0.v[3 * r + 1] * E[3 + q] + p0.v[3 * r + 2] * E[6 + q];
  for (int q = 0; q < 3; ++q) out[9 + q] = p0.v[9 + q] + delta[3 + q];
}

// d_delta[0:3] += J_r^T g[0:3] (g: the gradient w.r.t. the right
// perturbation of R), d_delta[3:6] += g[3:6].
__global__ void k_pose_back(const double* __restrict__ jr, const double* __restrict__ gpose,
                            double* __restrict__ d_delta) {
  const int q = threadIdx.x;
  if (q < 3)
    d_delta[q] += jr[q] * gpose[0] + jr[3 + q] * gpose[1] + jr[6 + q] * gpose[2];
  else if (q < 6)
    d_delta[q] += gpose[q];
}

// ---- host side

static double coord_scale(const rbf_params* p, bool fp32) {
  // exp(-d^2/(2 sigma^2)) = exp(-(ks d)^2) with ks = 1/(sqrt(2) sigma);
  // = exp2(-(ks d)^2) with ks = sqrt(log2(e)/2)/sigma
  const double l2e = 1.4426950408889634;
  return fp32 ? std::sqrt(0.5 * l2e) / p->sigma : std::sqrt(0.5) / p->sigma;
}

// Coordinates are taken relative to the grid origin (binned form) or to
// the mesh origin (mesh form).
template <typename T>
static EvalK<T> make_consts(const rbf_params* p, const rbf_grid* g, const double* pose,
                            double z_off, bool mesh = false) {
  EvalK<T> k;
  const double ks = coord_scale(p, sizeof(T) == 4);
  const double rcs = p->cutoff * p->sigma * ks;
  k.x0 = (T)(mesh ? g->mx0 : g->x0);
  k.y0 = (T)(mesh ? g->my0 : g->y0);
  k.ks = (T)ks;
  k.rc2s = (T)(rcs * rcs);
  k.gscale = (T)(-1.0 / (ks * p->sigma * p->sigma));
  k.inv_eh = (T)g->inv_eh;
  for (int q = 0; q < 9; ++q) k.R[q] = pose ? (T)pose[q] : (T)0;
  for (int q = 0; q < 3; ++q) k.t[q] = pose ? (T)pose[9 + q] : (T)0;
  k.z_off = (T)z_off;
  return k;
}

static EGeom egeom(const rbf_params* p, const rbf_grid* g) {
  EGeom e;
  const double rb = p->cutoff * p->sigma * g->inv_eh;
  e.pad = EVAL_PAD;
  e.rbp = (float)(rb + EVAL_PAD);
  const double rbe = rb * (1.0 + 1e-5);
  e.rb2 = (float)(rbe * rbe);
  e.nbx = g->enbx;
  e.nby = g->enby;
  return e;
}

template <typename T>
static MGeom<T> mgeom(const rbf_params* p, const rbf_grid* g) {
  MGeom<T> m;
  m.hs = (T)(g->mres * coord_scale(p, sizeof(T) == 4));
  m.inv_res = (T)(1.0 / g->mres);
  m.rp = (float)(p->cutoff * p->sigma / g->mres + MESH_PAD);
  m.ilo = g->imin - g->mesh_w;
  m.ihi = g->imin + g->mnx;
  m.jlo = g->jmin - g->mesh_w;
  m.jhi = g->jmin + g->mny;
  m.ioff = g->mesh_w - g->imin;
  m.joff = g->mesh_w - g->jmin;
  m.pw = g->mpw;
  return m;
}

// Bytes of the evaluation table of grid g in precision T: the packed
// center table, or the dense node weights of the mesh form.
template <typename T>
static size_t table_bytes(const rbf_grid* g, bool mesh) {
  return mesh ? sizeof(T) * (size_t)g->mpw * (size_t)g->mph
              : sizeof(typename Vec4<T>::type) * (size_t)(g->N > 0 ? g->N : 1);
}

static rbf_status check_eval_args(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                                  const double* w, const void* pts, int64_t Q, int32_t dim,
                                  const double* pose, rbf_prec prec, const char* who) {
  if (!p || !g || !w) return fail(ctx, RBF_E_INVALID_ARG, "%s: null params/grid/w", who);
  if (Q < 0 || (Q > 0 && !pts)) return fail(ctx, RBF_E_INVALID_ARG, "%s: bad pts/Q", who);
  if (dim != 2 && dim != 3) return fail(ctx, RBF_E_INVALID_ARG, "%s: dim must be 2 or 3", who);
  if ((dim == 3) != (pose != nullptr))
    return fail(ctx, RBF_E_INVALID_ARG, "%s: pose required iff dim == 3", who);
  if (prec != RBF_F64 && prec != RBF_F32)
    return fail(ctx, RBF_E_INVALID_ARG, "%s: prec must be F64 or F32", who);
  if (!(p->sigma > 0) || !(p->cutoff > 0) || p->sigma != g->sigma || p->cutoff != g->cutoff)
    return fail(ctx, RBF_E_INVALID_ARG,
                "%s: sigma/cutoff differ from the grid's (rebuild the grid)", who);
  if (g->device != ctx->device)
    return fail(ctx, RBF_E_INVALID_ARG, "%s: grid on another device", who);
  if (g->N > ((int64_t)1 << 26))  // table offsets are 32-bit byte offsets
    return fail(ctx, RBF_E_INVALID_ARG, "%s: more than 2^26 centers", who);
  const uintptr_t two = prec == RBF_F64 ? 16 : 8;  // two elements
  if (dim == 2 && ((uintptr_t)pts % two) != 0)
    return fail(ctx, RBF_E_INVALID_ARG, "%s: xy points must be aligned to two elements", who);
  if (pose)
    for (int q = 0; q < 12; ++q)
      if (!std::isfinite(pose[q])) return fail(ctx, RBF_E_NONFINITE, "%s: non-finite pose", who);
  return RBF_OK;
}

static rbf_status check_eval_out(rbf_ctx* ctx, rbf_prec prec, const void* grad, const void* jac,
                                 const char* who) {
  const uintptr_t two = prec == RBF_F64 ? 16 : 8;
  if (((uintptr_t)grad % two) != 0 || ((uintptr_t)jac % two) != 0)
    return fail(ctx, RBF_E_INVALID_ARG, "%s: grad and jac must be aligned to two elements",
                who);
  return RBF_OK;
}

// Pack the evaluation table of grid g with weights w into tab (N entries).
template <typename T>
static rbf_status pack_into(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                            const double* w, typename Vec4<T>::type* tab) {
  k_pack_centers<T><<<ceil_div(g->N, 256), 256, 0, ctx->stream>>>(
      g->d_ecxy, g->d_eidx, w, g->N, g->x0, g->y0, coord_scale(p, sizeof(T) == 4), tab);
  RBF_LAUNCHED(ctx, "k_pack_centers");
  return RBF_OK;
}

rbf_status eval_workspace(rbf_ctx* ctx, const rbf_grid* g) {
  rbf_status st;
  size_t bytes = table_bytes<double>(g, false);
  if (g->mesh_w && table_bytes<double>(g, true) > bytes) bytes = table_bytes<double>(g, true);
  if (!ws_get(ctx, WS_TMP2, bytes, &st)) return st;
  return RBF_OK;
}

// Binned calls of few points read the grid's arrays as they are. That saves a
// launch, and forming the candidates anew for each point costs as much at some
// number of points times candidates (about half of max_cand), less in FP32, whose
// packed entries are half as large. Whole calls on 100 x 100 centers, so and packed
// (waited for): 0.5 m apart FP32 1000 points 21 and 25 us, 32,000 23.5 and 25,
// 50,000 27 and 26, FP64 64,000 29 and 30; 0.3 m apart FP32 16,000 25.6 and 27.5,
// 32,000 28.9 and 27.3, 65,000 38.7 and 29.5, FP64 32,000 30 and 31, 50,000 38
// and 36; 0.15 m apart FP32 1000 41 and 45, 4000 42 and 41, 65,000 92 and 44, FP64
// 16,000 46 and 44.
constexpr int64_t EVAL_RAW_Q = 65536;
template <typename T>
static bool raw_form(const rbf_grid* g, int64_t Q, bool mesh) {
  constexpr int64_t lim = sizeof(T) == 8 ? 7000000 : 3800000;
  return !mesh && Q <= EVAL_RAW_Q && (Q + 2000) * (int64_t)g->max_cand <= lim;
}

// The table of one call in `tab`: the mesh form's node weights if mesh,
// else the packed (x', y', w, index) of the eval-sorted centers.
template <typename T>
static rbf_status pack_nbr(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                           const double* w, void* tab, bool mesh, bool raw, Nbr<T>* nb) {
  nb->tab = tab;
  nb->estart = g->d_estart;
  if (raw) {
    nb->n = g->N;
    nb->eg = egeom(p, g);
    nb->ecxy = g->d_ecxy;
    nb->eidx = g->d_eidx;
    nb->w = w;
    nb->x0 = g->x0;
    nb->y0 = g->y0;
    nb->ks = coord_scale(p, sizeof(T) == 4);
    return RBF_OK;
  }
  if (mesh) {
    nb->n = (int64_t)g->mpw * g->mph;
    nb->mg = mgeom<T>(p, g);
    k_pack_mesh<T><<<ceil_div(nb->n, 256), 256, 0, ctx->stream>>>(g->d_mesh_map, w, nb->n,
                                                                  (T*)tab);
    RBF_LAUNCHED(ctx, "k_pack_mesh");
  } else {
    nb->n = g->N;
    nb->eg = egeom(p, g);
    RBF_TRY(pack_into<T>(ctx, p, g, w, (typename Vec4<T>::type*)tab));
  }
  return RBF_OK;
}

template <typename T, int MW>
static void launch_eval(rbf_ctx* ctx, unsigned blocks, int32_t dim, const void* pts, int64_t Q,
                        const Nbr<T>& nb, const EvalK<T>& k, const double* dpose, void* f,
                        void* grad, void* resid, void* jac) {
  if (dim == 3)
    k_eval<T, true, MW><<<blocks, 256, 0, ctx->stream>>>((const T*)pts, Q, nb, k, dpose, (T*)f,
                                                         (T*)grad, (T*)resid, (T*)jac);
  else
    k_eval<T, false, MW><<<blocks, 256, 0, ctx->stream>>>((const T*)pts, Q, nb, k, nullptr,
                                                          (T*)f, (T*)grad, nullptr, nullptr);
}

// Whether a call takes the LDS mesh form, and its table. The node array has to
// fit, and the registers of a window leave a workgroup of 12-node FP64 windows
// 256 threads only (200,000 points 34.8 us against the quads' 32.2). Whole
// calls on 100 x 100 centers otherwise, LDS and quads: FP32 1000 points 17.0
// and 20.2 us, 200,000 17.1 and 19.7, 1,000,000 26 and 42; FP64 16.9 and 19.3,
// 18.9 and 20.8, 51 and 74. (The kernels of 200,000 FP64 points: 17.7 us, with a
// second pass that few lanes take, against 15.1 + 2.9 for the packing. Waited for,
// from one point to 700,000, the LDS form is ahead or equal at every size.)
template <typename T>
static bool mesh_lds(const rbf_params* p, const rbf_grid* g, const double* w, bool mesh,
                     MeshTab<T>* mt) {
  if (!mesh || g->N <= 0 || (int64_t)table_bytes<T>(g, true) > MESH_LDS_BYTES) return false;
  if (sizeof(T) == 8 && g->mesh_w > 8) return false;
  mt->map = g->d_mesh_map;
  mt->w = w;
  mt->n = g->mpw * g->mph;
  mt->mg = mgeom<T>(p, g);
  return true;
}

template <typename T, int MW>
static void launch_eval_lds(rbf_ctx* ctx, int32_t dim, const void* pts, int64_t Q,
                            const MeshTab<T>& mt, const EvalK<T>& k, const double* dpose, void* f,
                            void* grad, void* resid, void* jac) {
  const int64_t share = mesh_share(Q);
  const unsigned wgs = (unsigned)ceil_div(Q, share);
  const size_t lds = sizeof(T) * (size_t)mt.n;
  if (dim == 3)
    k_eval_lds<T, true, MW><<<wgs, mesh_threads<T, MW>(), lds, ctx->stream>>>(
        (const T*)pts, Q, share, mt, k, dpose, (T*)f, (T*)grad, (T*)resid, (T*)jac);
  else
    k_eval_lds<T, false, MW><<<wgs, mesh_threads<T, MW>(), lds, ctx->stream>>>(
        (const T*)pts, Q, share, mt, k, nullptr, (T*)f, (T*)grad, nullptr, nullptr);
}

template <typename T, int MW>
static void launch_gn_lds(rbf_ctx* ctx, const void* pts, int64_t Q, const MeshTab<T>& mt,
                          const EvalK<T>& k, double* part) {
  const int64_t share = mesh_share(Q);
  constexpr int NT = GN_LDS_NT;
  const size_t lds = std::max(sizeof(T) * (size_t)mt.n, sizeof(double) * GN_TERMS * NT);
  k_gn_lds<T, MW><<<(unsigned)ceil_div(Q, share), NT, lds, ctx->stream>>>(
      (const T*)pts, Q, share, mt, k, part);
}

// Evaluation: the call's table in `tab` (table_bytes<T>(g, mesh) bytes),
// then one k_eval launch.
template <typename T>
static rbf_status eval_direct(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                              const double* w, const void* pts, int64_t Q, int32_t dim,
                              const double* pose, double z_off, void* f, void* grad,
                              void* resid, void* jac, void* tab, bool mesh,
                              const double* dpose = nullptr) {
  const EvalK<T> k = make_consts<T>(p, g, pose, z_off, mesh);
  MeshTab<T> mt;
  if (mesh_lds<T>(p, g, w, mesh, &mt)) {
    prof_begin(ctx, RBF_PROF_EVAL);
    switch (g->mesh_w) {
      case 4: launch_eval_lds<T, 4>(ctx, dim, pts, Q, mt, k, dpose, f, grad, resid, jac); break;
      case 8: launch_eval_lds<T, 8>(ctx, dim, pts, Q, mt, k, dpose, f, grad, resid, jac); break;
      default:
        if constexpr (sizeof(T) == 4)
          launch_eval_lds<T, 12>(ctx, dim, pts, Q, mt, k, dpose, f, grad, resid, jac);
        break;
    }
    RBF_LAUNCHED(ctx, "k_eval_lds");
    prof_end(ctx, RBF_PROF_EVAL);
    return RBF_OK;
  }
  const bool raw = raw_form<T>(g, Q, mesh);
  Nbr<T> nb;
  RBF_TRY(pack_nbr<T>(ctx, p, g, w, tab, mesh, raw, &nb));
  const unsigned blocks = (unsigned)ceil_div(Q * LPP, 256);
  prof_begin(ctx, RBF_PROF_EVAL);
  switch (mesh ? g->mesh_w : raw ? -1 : 0) {
    case -1: launch_eval<T, -1>(ctx, blocks, dim, pts, Q, nb, k, dpose, f, grad, resid, jac); break;
    case 0: launch_eval<T, 0>(ctx, blocks, dim, pts, Q, nb, k, dpose, f, grad, resid, jac); break;
    case 4: launch_eval<T, 4>(ctx, blocks, dim, pts, Q, nb, k, dpose, f, grad, resid, jac); break;
    case 8: launch_eval<T, 8>(ctx, blocks, dim, pts, Q, nb, k, dpose, f, grad, resid, jac); break;
    default:
      launch_eval<T, 12>(ctx, blocks, dim, pts, Q, nb, k, dpose, f, grad, resid, jac);
      break;
  }
  RBF_LAUNCHED(ctx, "k_eval");
  prof_end(ctx, RBF_PROF_EVAL);
  return RBF_OK;
}

// The call's table in the context's workspace.
template <typename T>
static rbf_status eval_ws(rbf_ctx* ctx, const rbf_grid* g, bool mesh, void** tab) {
  rbf_status st;
  *tab = ws_get(ctx, WS_TMP2, table_bytes<T>(g, mesh), &st);
  return *tab ? RBF_OK : st;
}

template <typename T>
static rbf_status eval_t(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g, const double* w,
                         const void* pts, int64_t Q, int32_t dim, const double* pose,
                         double z_off, void* f, void* grad, void* resid, void* jac,
                         const double* dpose = nullptr) {
  const bool mesh = g->mesh_w != 0;
  void* tab;
  RBF_TRY(eval_ws<T>(ctx, g, mesh, &tab));
  return eval_direct<T>(ctx, p, g, w, pts, Q, dim, pose, z_off, f, grad, resid, jac, tab, mesh,
                        dpose);
}

template <typename T>
static rbf_status gn_t(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g, const double* w,
                       const void* pts, int64_t Q, const double* pose, double z_off,
                       double* JtJ, double* Jtr, double* rtr) {
  const bool mesh = g->mesh_w != 0;
  void* tab;
  RBF_TRY(eval_ws<T>(ctx, g, mesh, &tab));
  const EvalK<T> k = make_consts<T>(p, g, pose, z_off, mesh);
  MeshTab<T> mt;
  // Not for the registers of 12-node windows (512 threads, 200,000 points 24.7 us
  // against the quads' 22.5). Else, LDS and quads on 10,000 centers: FP32 1000
  // points 16.5 and 18.2 us, 200,000 16.5 and 20.0, 1,000,000 30 and 38; FP64
  // 16 and 18, 20.4 and 21.4, 51 and 63.
  if (g->mesh_w <= 8 && mesh_lds<T>(p, g, w, mesh, &mt)) {
    rbf_status st;
    const int64_t wgs = ceil_div(Q, mesh_share(Q));
    double* part = (double*)ws_get(ctx, WS_TMP3, sizeof(double) * GN_TERMS * (size_t)wgs, &st);
    if (!part) return st;
    switch (g->mesh_w) {
      case 4: launch_gn_lds<T, 4>(ctx, pts, Q, mt, k, part); break;
      default: launch_gn_lds<T, 8>(ctx, pts, Q, mt, k, part); break;
    }
    RBF_LAUNCHED(ctx, "k_gn_lds");
    k_eval_gn_sum<<<GN_TERMS, GN_SUM_T, 0, ctx->stream>>>(
        part, wgs, JtJ, Jtr, rtr);
    RBF_LAUNCHED(ctx, "k_eval_gn_sum");
    return RBF_OK;
  }
  const bool raw = raw_form<T>(g, Q, mesh);
  Nbr<T> nb;
  RBF_TRY(pack_nbr<T>(ctx, p, g, w, tab, mesh, raw, &nb));
  int64_t blocks = ceil_div(Q * LPP, 256);
  if (blocks > GN_MAX_BLOCKS) blocks = GN_MAX_BLOCKS;
  rbf_status st;
  double* part = (double*)ws_get(ctx, WS_TMP3, sizeof(double) * GN_TERMS * (size_t)blocks, &st);
  if (!part) return st;
  const dim3 gr((unsigned)blocks);
  switch (mesh ? g->mesh_w : raw ? -1 : 0) {
    case -1: k_eval_gn<T, -1><<<gr, 256, 0, ctx->stream>>>((const T*)pts, Q, nb, k, part); break;
    case 0: k_eval_gn<T, 0><<<gr, 256, 0, ctx->stream>>>((const T*)pts, Q, nb, k, part); break;
    case 4: k_eval_gn<T, 4><<<gr, 256, 0, ctx->stream>>>((const T*)pts, Q, nb, k, part); break;
    case 8: k_eval_gn<T, 8><<<gr, 256, 0, ctx->stream>>>((const T*)pts, Q, nb, k, part); break;
    default: k_eval_gn<T, 12><<<gr, 256, 0, ctx->stream>>>((const T*)pts, Q, nb, k, part); break;
  }
  RBF_LAUNCHED(ctx, "k_eval_gn");
  k_eval_gn_sum<<<GN_TERMS, GN_SUM_T, 0, ctx->stream>>>(part, blocks, JtJ, Jtr, rtr);
  RBF_LAUNCHED(ctx, "k_eval_gn_sum");
  return RBF_OK;
}

template <typename T>
static rbf_status adjoint_t(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                            const double* w, const void* pts, int64_t Q, int32_t dim,
                            const double* pose, const void* gf, const void* gr, void* d_pts,
                            double* d_w, double* d_pose, const double* dpose = nullptr) {
  // Planes when the sums fit the LDS and the additions, about pi N / (bins with
  // centers) for a point, outweigh clearing, writing and adding up N sums per plane and a launch.
  // Few centers meet where more atomics fall on each of them, many where the
  // planes' traffic is covered. Whole calls by planes and by atomics, centers 0.5 m
  // and 1 m apart at a support of 1.5 m (28 and 7 additions): N = 400, 4096 points
  // 19 and 28 us, at 1 m 18 and 17; N = 3600, 10,800 20 and 18, 21,600 21 and 25;
  // N = 10,000, 20,000 points 21 and 24, at 1 m 20 and 16, 90,000 32 and 41;
  // N = 17,956, 53,868 points 34 and 47, at 1 m 33 and 27. Of 630 such pairs (3 to
  // 113 additions, 0.25 m to 1.5 m apart) none is slower by this rule than by
  // atomics by more than the runs differ.
  // The buffer's size depends on the grid and the type alone, as the table's; not
  // taken if it would grow during a capture.
  const int64_t planes = std::min<int64_t>(ADJ_PLANES, Q / 256);
  const int64_t nodes = (int64_t)g->mpw * g->mph;
  // In FP64 on a mesh with windows of up to 8 nodes (the registers of a 12-node
  // window do not fit 1024 threads) also by the mesh form: 200,000 points on
  // 10,000 centers 40 -> 30 us. FP32 keeps the binned terms.
  const bool mesh = sizeof(T) == 8 && g->mesh_w > 0 && g->mesh_w <= 8 && nodes <= ADJ_LDS_N;
  const int64_t n = mesh ? nodes : g->N;
  double* plane = nullptr;  // the planes, and behind them the mesh form's node weights
  const double adds =  // and the point itself; the outer bins hold no centers
      (double)Q * (1.0 + 3.14 * (double)g->N / ((double)(g->nbx - 2) * (g->nby - 2)));
  const bool enough =
      Q >= 2 * g->N && adds >= std::min(140.0 * g->N, 250e3 + 30.0 * g->N);
  if (d_w && n <= ADJ_LDS_N && planes >= ADJ_MIN_PLANES && enough)
    plane = (double*)ws_try(ctx, WS_ADJ, sizeof(double) * (ADJ_PLANES + 1) * n);
  const int form = plane && mesh ? g->mesh_w : 0;
  void* tab = plane ? plane + ADJ_PLANES * n : nullptr;
  if (!form) RBF_TRY(eval_ws<T>(ctx, g, false, &tab));
  Nbr<T> nb;
  RBF_TRY(pack_nbr<T>(ctx, p, g, w, tab, form != 0, false, &nb));
  const EvalK<T> k = make_consts<T>(p, g, pose, 0.0, form != 0);
  const auto launch = [&](auto kern, unsigned blocks, int nt, size_t lds, double* out) {
    kern<<<blocks, nt, lds, ctx->stream>>>((const T*)pts, Q, nb, k, dim == 3 ? dpose : nullptr,
                                           (const T*)gf, dim == 3 ? (const T*)gr : nullptr,
                                           (T*)d_pts, out, dim == 3 ? d_pose : nullptr);
  };
  if (plane) {
    const size_t lds = sizeof(double) * (size_t)n;
    const bool p3 = dim == 3;
    if constexpr (sizeof(T) == 8) {
      if (form == 4)
        launch(p3 ? k_eval_adjoint<T, true, true, 4> : k_eval_adjoint<T, false, true, 4>,
               (unsigned)planes, adj_threads<4>(), lds, plane);
      else if (form == 8)
        launch(p3 ? k_eval_adjoint<T, true, true, 8> : k_eval_adjoint<T, false, true, 8>,
               (unsigned)planes, adj_threads<8>(), lds, plane);
    }
    if (form == 0)
      launch(p3 ? k_eval_adjoint<T, true, true, 0> : k_eval_adjoint<T, false, true, 0>,
             (unsigned)planes, adj_threads<0>(), lds, plane);
    RBF_LAUNCHED(ctx, "k_eval_adjoint");
    k_adjoint_sum<<<ceil_div(n, 64), 1024, 0, ctx->stream>>>(
        plane, (int)planes, n, form ? g->d_mesh_map : nullptr, d_w);
    RBF_LAUNCHED(ctx, "k_adjoint_sum");
    return RBF_OK;
  }
  launch(dim == 3 ? k_eval_adjoint<T, true, false, 0> : k_eval_adjoint<T, false, false, 0>,
         (unsigned)ceil_div(Q * LPP, 256), 256, 0, d_w);
  RBF_LAUNCHED(ctx, "k_eval_adjoint");
  return RBF_OK;
}

// Pose (12) and right Jacobian (9) of the increment form in the context's
// workspace, followed by 6 doubles for the pose gradient.
static rbf_status pose_at(rbf_ctx* ctx, const double* pose0, const double* delta,
                          double** out) {
  rbf_status st;
  double* buf = (double*)ws_get(ctx, WS_POSE, sizeof(double) * 32, &st);
  if (!buf) return st;
  Pose0 p0;
  for (int q = 0; q < 12; ++q) p0.v[q] = pose0[q];
  k_pose_exp<<<1, 64, 0, ctx->stream>>>(p0, delta, buf);
  RBF_LAUNCHED(ctx, "k_pose_exp");
  *out = buf;
  return RBF_OK;
}

// ---- allocation-free evaluation (rbf_eval_noalloc)
//
// The packed center table of rbf_eval_noalloc lives in this device array
// instead of the context's workspace, so that entry point allocates
// nothing. Each GPU the library runs on holds its own copy at its own
// address until the process ends. In host code the array's name is only a
// host-side stand-in, never a device address: eval_scratch_init looks the
// device address up once per device (from rbf_ctx_create, with the device
// current) and kernels receive that pointer.
static __device__ __align__(256) double4 scratch[RBF_EVAL_NOALLOC_MAX_CENTERS];

constexpr int SCRATCH_MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[SCRATCH_MAX_DEVICES] = {};

rbf_status eval_scratch_init(int device) {
  if (device < 0 || device >= SCRATCH_MAX_DEVICES) return RBF_E_INVALID_ARG;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return RBF_OK;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    (void)hipGetLastError();
    return RBF_E_HIP;
  }
  g_scratch_ptr[device] = ptr;
  return RBF_OK;
}

static void* eval_scratch(int device) {
  if (device < 0 || device >= SCRATCH_MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}

}  // namespace rbf

using namespace rbf;

extern "C" {

rbf_status rbf_eval_noalloc(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                            const double* w, const void* pts, int64_t Q, int32_t dim,
                            const double* pose, double z_off, rbf_prec prec, void* f,
                            void* grad, void* resid, void* jac) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_eval_args(ctx, p, g, w, pts, Q, dim, pose, prec, "rbf_eval_noalloc"));
  RBF_TRY(check_eval_out(ctx, prec, grad, jac, "rbf_eval_noalloc"));
  if (Q > 0 && !f) return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval_noalloc: f is required");
  if (dim == 2 && (resid || jac))
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval_noalloc: resid/jac need dim == 3");
  // the mesh form when its node weights fit the scratch array (else the
  // binned form, which rbf_eval would not take)
  const size_t cap = sizeof(double4) * (size_t)RBF_EVAL_NOALLOC_MAX_CENTERS;
  const bool mesh = g->mesh_w != 0 && (prec == RBF_F64 ? table_bytes<double>(g, true)
                                                       : table_bytes<float>(g, true)) <= cap;
  if (g->mesh_w && !mesh)
    return fail(ctx, RBF_E_CAPACITY,
                "rbf_eval_noalloc: the mesh's %lld nodes exceed the scratch array (use "
                "rbf_eval)", (long long)g->mpw * g->mph);
  if (!mesh && g->N > RBF_EVAL_NOALLOC_MAX_CENTERS)
    return fail(ctx, RBF_E_CAPACITY,
                "rbf_eval_noalloc: %lld centers exceed the maximum of %d (use rbf_eval)",
                (long long)g->N, (int)RBF_EVAL_NOALLOC_MAX_CENTERS);
  if (Q == 0) return RBF_OK;
  RBF_TRY(set_device(ctx));
  void* tab = eval_scratch(ctx->device);
  if (!tab)
    return fail(ctx, RBF_E_HIP, "rbf_eval_noalloc: no device address of the scratch table");
  if (prec == RBF_F64)
    return eval_direct<double>(ctx, p, g, w, pts, Q, dim, pose, z_off, f, grad, resid, jac,
                               tab, mesh);
  return eval_direct<float>(ctx, p, g, w, pts, Q, dim, pose, z_off, f, grad, resid, jac, tab,
                            mesh);
}

rbf_status rbf_eval(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g, const double* w,
                    const void* pts, int64_t Q, int32_t dim, const double* pose, double z_off,
                    rbf_prec prec, void* f, void* grad, void* resid, void* jac) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_eval_args(ctx, p, g, w, pts, Q, dim, pose, prec, "rbf_eval"));
  RBF_TRY(check_eval_out(ctx, prec, grad, jac, "rbf_eval"));
  if (Q > 0 && !f) return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval: f is required");
  if (dim == 2 && (resid || jac))
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval: resid/jac need dim == 3");
  if (Q == 0) return RBF_OK;
  RBF_TRY(set_device(ctx));
  if (prec == RBF_F64) return eval_t<double>(ctx, p, g, w, pts, Q, dim, pose, z_off, f, grad,
                                             resid, jac);
  return eval_t<float>(ctx, p, g, w, pts, Q, dim, pose, z_off, f, grad, resid, jac);
}

rbf_status rbf_eval_at(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g, const double* w,
                       const void* pts, int64_t Q, const double* pose0, const double* delta,
                       double z_off, rbf_prec prec, void* f, void* grad, void* resid,
                       void* jac) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_eval_args(ctx, p, g, w, pts, Q, 3, pose0, prec, "rbf_eval_at"));
  RBF_TRY(check_eval_out(ctx, prec, grad, jac, "rbf_eval_at"));
  if (!delta) return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval_at: delta is required");
  if (Q > 0 && !f) return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval_at: f is required");
  if (Q == 0) return RBF_OK;
  RBF_TRY(set_device(ctx));
  double* buf;
  RBF_TRY(pose_at(ctx, pose0, delta, &buf));
  if (prec == RBF_F64)
    return eval_t<double>(ctx, p, g, w, pts, Q, 3, pose0, z_off, f, grad, resid, jac, buf);
  return eval_t<float>(ctx, p, g, w, pts, Q, 3, pose0, z_off, f, grad, resid, jac, buf);
}

rbf_status rbf_eval_adjoint_at(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                               const double* w, const void* pts, int64_t Q, const double* pose0,
                               const double* delta, rbf_prec prec, const void* gbar_f,
                               const void* gbar_r, void* d_pts, double* d_w, double* d_delta) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_eval_args(ctx, p, g, w, pts, Q, 3, pose0, prec, "rbf_eval_adjoint_at"));
  if (!delta) return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval_adjoint_at: delta is required");
  if (Q == 0) return RBF_OK;
  RBF_TRY(set_device(ctx));
  double* buf;
  RBF_TRY(pose_at(ctx, pose0, delta, &buf));
  double* gpose = d_delta ? buf + 24 : nullptr;
  if (gpose) RBF_TRY(fill_zero(ctx, gpose, 6 * sizeof(double)));
  if (prec == RBF_F64)
    RBF_TRY(adjoint_t<double>(ctx, p, g, w, pts, Q, 3, pose0, gbar_f, gbar_r, d_pts, d_w, gpose,
                              buf));
  else
    RBF_TRY(adjoint_t<float>(ctx, p, g, w, pts, Q, 3, pose0, gbar_f, gbar_r, d_pts, d_w, gpose,
                             buf));
  if (gpose) {
    k_pose_back<<<1, 64, 0, ctx->stream>>>(buf + 12, gpose, d_delta);
    RBF_LAUNCHED(ctx, "k_pose_back");
  }
  return RBF_OK;
}

rbf_status rbf_eval_gn(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g, const double* w,
                       const void* pts, int64_t Q, const double* pose, double z_off,
                       rbf_prec prec, double* JtJ, double* Jtr, double* rtr) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_eval_args(ctx, p, g, w, pts, Q, 3, pose, prec, "rbf_eval_gn"));
  if (!JtJ || !Jtr) return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval_gn: JtJ and Jtr required");
  RBF_TRY(set_device(ctx));
  if (Q == 0) {
    RBF_TRY(fill_zero(ctx, JtJ, 36 * sizeof(double)));
    RBF_TRY(fill_zero(ctx, Jtr, 6 * sizeof(double)));
    if (rtr) RBF_TRY(fill_zero(ctx, rtr, sizeof(double)));
    return RBF_OK;
  }
  if (prec == RBF_F64) return gn_t<double>(ctx, p, g, w, pts, Q, pose, z_off, JtJ, Jtr, rtr);
  return gn_t<float>(ctx, p, g, w, pts, Q, pose, z_off, JtJ, Jtr, rtr);
}

rbf_status rbf_eval_adjoint(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                            const double* w, const void* pts, int64_t Q, int32_t dim,
                            const double* pose, rbf_prec prec, const void* gbar_f,
                            const void* gbar_r, void* d_pts, double* d_w, double* d_pose) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_eval_args(ctx, p, g, w, pts, Q, dim, pose, prec, "rbf_eval_adjoint"));
  if (dim == 2 && (gbar_r || d_pose))
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_eval_adjoint: gbar_r/d_pose need dim == 3");
  if (Q == 0) return RBF_OK;
  RBF_TRY(set_device(ctx));
  if (prec == RBF_F64)
    return adjoint_t<double>(ctx, p, g, w, pts, Q, dim, pose, gbar_f, gbar_r, d_pts, d_w,
                             d_pose);
  return adjoint_t<float>(ctx, p, g, w, pts, Q, dim, pose, gbar_f, gbar_r, d_pts, d_w, d_pose);
}

}  // extern "C"

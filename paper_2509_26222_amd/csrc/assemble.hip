// Regressor rows (ELL) and the ridge information matrix (CSR).
//
// m(x, c) = s_m exp(-d^2 / (2 sigma_t^2)) for d <= cutoff sigma_t, else 0,
// with sigma_t^2 = sigma^2 + sigma_eps^2 and s_m = sigma^2 / sigma_t^2
// (moment regressor of the ridge-regression subsection; eq. rbf_kernel is
// the matrix of these rows for one scan). calH = lambda I + sum_i m_i m_i^T
// and b = sum_i m_i z_i (eq. RBF_estimator with the ridge term).
//
// The support test d^2 <= rc^2 decides the sparsity pattern, so it is done
// with separately rounded products (no fused multiply-add) to be exactly the
// plain definition's decision.
#include <algorithm>
#include <cmath>

#include "internal.hpp"

namespace rbf {

struct RegK {
  double rc2;    // (cutoff sigma_t)^2
  double den;    // 2 sigma_t^2, formed as (2 sigma_t) sigma_t
  double scale;  // s_m
};

static RegK reg_consts(const rbf_params* p) {
  RegK k;
  const double st = std::sqrt(p->sigma * p->sigma + p->sigma_eps * p->sigma_eps);
  const double rc = p->cutoff * st;
  k.rc2 = rc * rc;
  k.den = 2.0 * st * st;
  k.scale = (p->sigma * p->sigma) / (st * st);
  return k;
}

__device__ inline double sq_d(double px, double py, double cx, double cy) {
  const double dx = __dsub_rn(px, cx), dy = __dsub_rn(py, cy);
  return __dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy));
}

__device__ inline double reg_val(double d2, const RegK& k) {
  return k.scale * exp(-d2 / k.den);
}

// ---------------------------------------------------------------- ELL rows

// Sixteen lanes per point: the lanes test the candidates of a bin row 16 at
// a time, and a ballot with a popcount prefix gives each hit its slot in
// candidate order (the order of a serial scan); the row's padding is then
// written 16 slots at a time. The 16 lanes of a point share its loop bounds,
// so they stay together through every ballot.
template <typename T>
__global__ void __launch_bounds__(256) k_assemble_phi(const double* __restrict__ xy, int64_t M,
                                                      const double* __restrict__ cxy,
                                                      const int32_t* __restrict__ idx,
                                                      const int32_t* __restrict__ start,
                                                      GridGeom g, RegK k, int32_t kmax,
                                                      T* __restrict__ vals,
                                                      int32_t* __restrict__ cols,
                                                      int32_t* __restrict__ nnz,
                                                      int32_t* __restrict__ status) {
  const int tid = threadIdx.x, l = tid & 15, gshift = tid & 48;
  const int64_t i = (int64_t)blockIdx.x * 16 + (tid >> 4);
  if (i >= M) return;  // whole groups of 16 lanes leave together
  const double x = xy[2 * i], y = xy[2 * i + 1];
  T* vrow = vals + i * kmax;
  int32_t* crow = cols + i * kmax;
  int n = 0;
  int bx0, bx1, by0, by1;
  if (bin_range(x, g.x0, g.inv_h, g.nbx, &bx0, &bx1) &&
      bin_range(y, g.y0, g.inv_h, g.nby, &by0, &by1)) {
    for (int by = by0; by <= by1; ++by) {
      const int row = by * g.nbx;
      const int s0 = start[row + bx0], s1 = start[row + bx1 + 1];
      for (int base = s0; base < s1; base += 16) {
        const int s = base + l;
        double d2 = 0.0;
        bool ok = false;
        if (s < s1) {
          d2 = sq_d(x, y, cxy[2 * s], cxy[2 * s + 1]);
          ok = d2 <= k.rc2;
        }
        const uint32_t gm = (uint32_t)(__ballot(ok) >> gshift) & 0xFFFFu;
        const int pos = n + __popc(gm & ((1u << l) - 1u));
        if (ok && pos < kmax) {
          vrow[pos] = (T)reg_val(d2, k);
          crow[pos] = idx[s];
        }
        n += __popc(gm);
      }
    }
  }
  if (l == 0 && n > kmax) set_status(status, RBF_E_CAPACITY, i);
  const int w = n < kmax ? n : kmax;
  for (int q = w + l; q < kmax; q += 16) {
    vrow[q] = (T)0;
    crow[q] = 0;
  }
  if (l == 0) nnz[i] = w;
}

// ---------------------------------------------------------- Gram pattern

// Row of center j: centers within 2 cutoff sigma_t, found in the 5x5 bins
// around j (bin side > cutoff sigma_t). count pass then fill pass.
__global__ void __launch_bounds__(256) k_gram_count(const double* __restrict__ cxy, int64_t N,
                                                    const int32_t* __restrict__ idx,
                                                    const int32_t* __restrict__ start, GridGeom g,
                                                    double r2, int64_t* __restrict__ rowcnt) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= N) return;
  const double x = cxy[2 * s], y = cxy[2 * s + 1];
  const int bx = bin_of(x, g.x0, g.inv_h, g.nbx), by = bin_of(y, g.y0, g.inv_h, g.nby);
  int64_t n = 0;
  for (int yy = (by > 1 ? by - 2 : 0); yy <= (by + 2 < g.nby ? by + 2 : g.nby - 1); ++yy) {
    const int row = yy * g.nbx;
    const int s0 = start[row + (bx > 1 ? bx - 2 : 0)];
    const int s1 = start[row + (bx + 2 < g.nbx ? bx + 2 : g.nbx - 1) + 1];
    for (int t = s0; t < s1; ++t) n += sq_d(x, y, cxy[2 * t], cxy[2 * t + 1]) <= r2;
  }
  rowcnt[idx[s]] = n;
}

__global__ void __launch_bounds__(256) k_gram_fill(const double* __restrict__ cxy, int64_t N,
                                                   const int32_t* __restrict__ idx,
                                                   const int32_t* __restrict__ start, GridGeom g,
                                                   double r2, const int64_t* __restrict__ rowptr,
                                                   int32_t* __restrict__ colidx, int64_t cap) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= N) return;
  const int64_t j = idx[s];
  const int64_t a = rowptr[j], e = rowptr[j + 1];
  if (e > cap) return;  // capacity error reported by the host
  const double x = cxy[2 * s], y = cxy[2 * s + 1];
  const int bx = bin_of(x, g.x0, g.inv_h, g.nbx), by = bin_of(y, g.y0, g.inv_h, g.nby);
  int64_t n = a;
  for (int yy = (by > 1 ? by - 2 : 0); yy <= (by + 2 < g.nby ? by + 2 : g.nby - 1); ++yy) {
    const int row = yy * g.nbx;
    const int s0 = start[row + (bx > 1 ? bx - 2 : 0)];
    const int s1 = start[row + (bx + 2 < g.nbx ? bx + 2 : g.nbx - 1) + 1];
    for (int t = s0; t < s1; ++t) {
      if (sq_d(x, y, cxy[2 * t], cxy[2 * t + 1]) <= r2 && n < e) {
        // insertion into the ascending run colidx[a, n)
        const int32_t c = idx[t];
        int64_t q = n;
        while (q > a && colidx[q - 1] > c) {
          colidx[q] = colidx[q - 1];
          --q;
        }
        colidx[q] = c;
        ++n;
      }
    }
  }
}

// ------------------------------------------------------------ Gram values
//
// calH gains sum_i m_i m_i^T. The points of one bin support centers of the 3x3
// bins around it only, so their part is a dense product: with Phi the bin's
// points against its R candidate centers (R <= the grid's max_cand, 81 on a
// regular mesh of three centers per support radius), G_bin = Phi^T Phi on
// FP64 MFMA (k_gram_bins), and an entry (j, k) of calH is the sum of its
// elements of the at most nine bins next to both centers (k_gram_gather), in
// the order of the bins. Each regressor value is formed once per point and
// candidate; the row-wise kernel below forms the 28 values of a point again
// for every one of the 28 rows it belongs to, two passes per row. 800,000
// points on 40,000 centers: 10.4 -> 0.85 ms; 10,007 on 5,041: 224 -> 53 us.
// What bounds it now is the FP64 exponentials of the candidates (81 formed
// for 28 in the support).
//
// The bins' blocks are kept dense (both triangles, leading dimension ld =
// max_cand rounded up to 16) in a workspace of at most GRAM_WS bytes; larger
// grids go through it in strips of bins.
constexpr int GRAM_NT = 512;            // threads of k_gram_bins (8 waves)
constexpr int GRAM_PTS = 32;            // points per LDS chunk
constexpr int GRAM_RMAX = 256;          // candidates per bin
constexpr int GRAM_BLK = 5;             // 16x16 blocks per wave and pass
constexpr size_t GRAM_WS = (size_t)128 << 20;

typedef double v4d __attribute__((ext_vector_type(4)));

// Candidate runs of bin (bx, by): in the sorted centers, row y of the 3x3 bins
// is the run [s0, s1), and its centers take the local indices from base on.
struct BinRuns {
  int s0[3], s1[3], base[4];
};
__device__ __forceinline__ BinRuns bin_runs(int bx, int by, const GridGeom& g,
                                            const int32_t* __restrict__ start) {
  BinRuns r;
  r.base[0] = 0;
  const int x0 = bx > 0 ? bx - 1 : 0, x1 = bx + 1 < g.nbx ? bx + 1 : g.nbx - 1;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int y = by + d - 1;
    const bool in = y >= 0 && y < g.nby;
    r.s0[d] = in ? start[y * g.nbx + x0] : 0;
    r.s1[d] = in ? start[y * g.nbx + x1 + 1] : 0;
    r.base[d + 1] = r.base[d] + r.s1[d] - r.s0[d];
  }
  return r;
}

// Workgroup: bin bin0 + blockIdx.x. G[local][local'] and B[local] = sum m z of
// its points, and off[bin][d] with local index = sorted position + off of the
// center's bin row (d = row - by + 1); off[bin][3] = 0 if the bin has no
// points (then nothing else is written).
// RMAX: 128 or GRAM_RMAX candidates (LDS for four or two workgroups per CU).
template <int RMAX>
__global__ void __launch_bounds__(GRAM_NT) k_gram_bins(
    const double* __restrict__ cxy, const int32_t* __restrict__ start,
    const double* __restrict__ pxy, const double* __restrict__ pz,
    const int32_t* __restrict__ pstart, GridGeom g, RegK k, int32_t bin0, int32_t ld,
    double* __restrict__ G, double* __restrict__ B, int32_t* __restrict__ off) {
  __shared__ double Phi[GRAM_PTS][RMAX + 4];
  __shared__ double cx[RMAX], cy[RMAX];
  __shared__ double px[GRAM_PTS], py[GRAM_PTS], pzs[GRAM_PTS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, kq = lane >> 4;
  const int bin = bin0 + blockIdx.x;
  const int bx = bin % g.nbx, by = bin / g.nbx;
  const int p0 = pstart[bin], np = pstart[bin + 1] - p0;
  const BinRuns r = bin_runs(bx, by, g, start);
  const int R = r.base[3];
  const bool any = np > 0 && R > 0;
  const int o0 = r.base[0] - r.s0[0], o1 = r.base[1] - r.s0[1], o2 = r.base[2] - r.s0[2];
  if (tid < 4)
    off[4 * (int64_t)blockIdx.x + tid] = tid == 0 ? o0 : tid == 1 ? o1 : tid == 2 ? o2 : any;
  if (!any) return;  // uniform
  for (int e = tid; e < R; e += GRAM_NT) {
    const int64_t s = e - (e < r.base[1] ? o0 : e < r.base[2] ? o1 : o2);
    cx[e] = cxy[2 * s];
    cy[e] = cxy[2 * s + 1];
  }
  const int nb = (R + 15) / 16, Rp = 16 * nb, nblk = nb * (nb + 1) / 2;
  const int kk0 = tid / Rp, e0 = tid % Rp, dk = GRAM_NT / Rp, de = GRAM_NT % Rp;
  double* Gb = G + (int64_t)blockIdx.x * ld * ld;
  for (int pass = 0; pass * GRAM_BLK * 8 < nblk; ++pass) {
    int bi[GRAM_BLK], bj[GRAM_BLK];
    v4d acc[GRAM_BLK];
    int nq = 0;  // this wave's blocks: idx = first + wave, + 8, ...
#pragma unroll
    for (int q = 0; q < GRAM_BLK; ++q) {
      const int idx = pass * GRAM_BLK * 8 + wave + 8 * q;
      int i = 0;
      while ((i + 1) * (i + 2) / 2 <= idx) ++i;
      bi[q] = i;
      bj[q] = idx - i * (i + 1) / 2;
      acc[q] = (v4d){0.0, 0.0, 0.0, 0.0};
      if (idx < nblk) nq = q + 1;
    }
    double bsum = 0.0;
    // a chunk's points are loaded while the chunk before is multiplied
    double nx = 0.0, ny = 0.0, nz = 0.0;
    auto fetch = [&](int c0) {
      if (tid < min(GRAM_PTS, np - c0)) {
        const int64_t p = p0 + c0 + tid;
        nx = pxy[2 * p];
        ny = pxy[2 * p + 1];
        nz = pz[p];
      }
    };
    fetch(0);
    for (int c0 = 0; c0 < np; c0 += GRAM_PTS) {
      const int cnt = min(GRAM_PTS, np - c0);
      __syncthreads();  // the chunk before is read (and, first, cx / cy written)
      if (tid < cnt) {
        px[tid] = nx;
        py[tid] = ny;
        pzs[tid] = nz;
      }
      __syncthreads();
      const int cnt4 = (cnt + 3) & ~3;
      // all lanes take entries of the cnt4 x Rp block, row by row
      for (int kk = kk0, e = e0; kk < cnt4;) {
        double m = 0.0;
        if (kk < cnt && e < R) {
          const double d2 = sq_d(px[kk], py[kk], cx[e], cy[e]);
          if (d2 <= k.rc2) m = reg_val(d2, k);
        }
        Phi[kk][e] = m;
        kk += dk;
        e += de;
        if (e >= Rp) {
          e -= Rp;
          ++kk;
        }
      }
      __syncthreads();
      if (c0 + GRAM_PTS < np) fetch(c0 + GRAM_PTS);
      for (int kk = 0; kk < cnt4; kk += 4) {
#pragma unroll
        for (int q = 0; q < GRAM_BLK; ++q)
          if (q < nq)
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(Phi[kk + kq][16 * bi[q] + li],
                                                          Phi[kk + kq][16 * bj[q] + li], acc[q],
                                                          0, 0, 0);
      }
      if (pass == 0 && tid < R) {
        for (int kk = 0; kk < cnt; kk += 8) {
          double m[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) m[u] = Phi[min(kk + u, cnt - 1)][tid];
#pragma unroll
          for (int u = 0; u < 8; ++u)  // a non-finite height stays with its support
            if (kk + u < cnt && m[u] != 0.0) bsum += m[u] * pzs[kk + u];
        }
      }
    }
    if (pass == 0 && tid < R) B[(int64_t)blockIdx.x * ld + tid] = bsum;
#pragma unroll
    for (int q = 0; q < GRAM_BLK; ++q)
      if (q < nq)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = 16 * bi[q] + 4 * v + kq, j = 16 * bj[q] + li;
          Gb[(int64_t)i * ld + j] = acc[q][v];
          if (bi[q] != bj[q]) Gb[(int64_t)j * ld + i] = acc[q][v];
        }
  }
}

// Workgroup: bin first + blockIdx.x; a wavefront per row j of calH whose center
// is in the bin, lanes on its entries: vals += the entry's elements of the bins
// [bin0, bin0 + nbins) next to both centers, b += the row's, and lambda on the
// diagonal with the bin itself. A row next to no points is not touched.
__global__ void __launch_bounds__(256) k_gram_gather(
    const double* __restrict__ cxy, const int32_t* __restrict__ start,
    const int32_t* __restrict__ rank, const int32_t* __restrict__ idx, GridGeom g, int32_t first,
    int32_t bin0, int32_t nbins, int32_t ld, const double* __restrict__ G,
    const double* __restrict__ B, const int32_t* __restrict__ off,
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx, double lambda,
    double* __restrict__ vals, double* __restrict__ b) {
  const int lane = threadIdx.x & 63;
  const int own = first + blockIdx.x;
  const int bx = own % g.nbx, by = own / g.nbx;
  const int32_t* ob[9];  // local index = sorted position + ob[q][row], null: no points in bin q
  bool any = false;
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    const int x = bx + q % 3 - 1, y = by + q / 3 - 1;
    const int bin = y * g.nbx + x - bin0;
    ob[q] = nullptr;
    if (x < 0 || x >= g.nbx || y < 0 || y >= g.nby || bin < 0 || bin >= nbins) continue;
    if (off[4 * (int64_t)bin + 3] == 0) continue;
    ob[q] = off + 4 * (int64_t)bin;
    any = true;
  }
  const double diag = own >= bin0 && own < bin0 + nbins ? lambda : 0.0;
  if (!any && diag == 0.0) return;  // uniform
  for (int s = start[own] + (threadIdx.x >> 6); s < start[own + 1]; s += 4) {
    const int64_t j = idx[s];
    int64_t at[9];  // element (j, 0) of bin q's block
    double bj = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      if (!ob[q]) continue;
      const int64_t bin = by * g.nbx + bx + (q / 3 - 1) * g.nbx + q % 3 - 1 - bin0;
      const int64_t jl = s + ob[q][2 - q / 3];
      at[q] = (bin * ld + jl) * ld;
      bj += B[bin * ld + jl];
    }
    const int64_t e = rowptr[j + 1];
    for (int64_t ent = rowptr[j] + lane; ent < e; ent += 64) {
      const int32_t kk = colidx[ent];
      const int64_t sk = rank[kk];
      const int kx = bin_of(cxy[2 * sk], g.x0, g.inv_h, g.nbx) - bx;
      const int ky = bin_of(cxy[2 * sk + 1], g.y0, g.inv_h, g.nby) - by;
      double acc = 0.0;
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const int dx = kx - (q % 3 - 1), dy = ky - (q / 3 - 1);  // center k's bin from bin q
        if (ob[q] && dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1)
          acc += G[at[q] + sk + ob[q][dy + 1]];
      }
      if (kk == j) acc += diag;
      vals[ent] += acc;
    }
    if (lane == 0) b[j] += bj;
  }
}

// Row-wise form, for grids with more candidates per bin than k_gram_bins holds
// and for few points on many centers.
// One wavefront per row j. The points within the support of c_j are read as
// three contiguous runs of the bin-sorted point table (uniform across the
// wave); lane e handles row entry e (center c_k) and accumulates
// m(x_i, c_j) m(x_i, c_k) in point order, so the sums are deterministic.
__global__ void __launch_bounds__(256) k_gram_values(
    const double* __restrict__ cxy, const int32_t* __restrict__ rank, int64_t N,
    const int32_t* __restrict__ idx, const double* __restrict__ pxy,
    const double* __restrict__ pz, const int32_t* __restrict__ pstart, GridGeom g, RegK k,
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx, double lambda,
    double* __restrict__ vals, double* __restrict__ b) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s >= N) return;
  const int64_t j = idx[s];
  const double cjx = cxy[2 * s], cjy = cxy[2 * s + 1];
  const int bx = bin_of(cjx, g.x0, g.inv_h, g.nbx), by = bin_of(cjy, g.y0, g.inv_h, g.nby);
  const int bx0 = bx > 0 ? bx - 1 : 0, bx1 = bx + 1 < g.nbx ? bx + 1 : g.nbx - 1;
  const int by0 = by > 0 ? by - 1 : 0, by1 = by + 1 < g.nby ? by + 1 : g.nby - 1;
  const int64_t a = rowptr[j], e = rowptr[j + 1];
  double bj = 0.0;
  for (int64_t base = a; base < e; base += 64) {
    const int64_t ent = base + lane;
    const bool act = ent < e;
    int32_t kk = act ? colidx[ent] : (int32_t)j;
    const int64_t sk = rank[kk];
    const double ckx = cxy[2 * sk], cky = cxy[2 * sk + 1];
    double acc = 0.0;
    for (int yy = by0; yy <= by1; ++yy) {
      const int row = yy * g.nbx;
      const int p0 = pstart[row + bx0], p1 = pstart[row + bx1 + 1];
      for (int p = p0; p < p1; ++p) {
        const double px = pxy[2 * p], py = pxy[2 * p + 1];
        const double dj = sq_d(px, py, cjx, cjy);
        if (dj <= k.rc2) {  // uniform across the wave
          const double mj = reg_val(dj, k);
          if (base == a) bj += mj * pz[p];
          const double dk = sq_d(px, py, ckx, cky);
          if (dk <= k.rc2) acc += mj * reg_val(dk, k);
        }
      }
    }
    if (act) {
      if (kk == j) acc += lambda;
      vals[ent] += acc;
    }
  }
  if (lane == 0) b[j] += bj;
}

}  // namespace rbf

using namespace rbf;

static rbf_status check_grid(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                             const char* who) {
  if (!p || !g) return fail(ctx, RBF_E_INVALID_ARG, "%s: null params or grid", who);
  if (g->device != ctx->device)
    return fail(ctx, RBF_E_INVALID_ARG, "%s: grid on another device", who);
  if (p->sigma != g->sigma || p->cutoff != g->cutoff || p->sigma_eps != g->sigma_eps)
    return fail(ctx, RBF_E_INVALID_ARG, "%s: params differ from the grid's", who);
  return RBF_OK;
}

// Whether the information matrix is formed by blocks: estimates of what each form
// takes beyond the parts they share. The row-wise kernel pays for each row, and for the
// points in the bins around it, once per 64 of its entries (about 1.2 max_cand); a small
// map's rows are on the chip at once and wait for one row's points. The blocks pay for
// bins, rows, the blocks' memory and, least, points, and for the launches of every strip.
// The constants (one unit is near 2 us) are those that choose best, by the time lost to
// the other form, over whole calls of both on 75 lattices of 100 to 193,600 centers,
// 0.25 m to 1.4 m apart and down to one center wide, with 0.76 to 8 points per center,
// at a support of 1.5 m: of 409 calls 4 take more than 1.08 times the faster form, at
// most 1.17. Row-wise and by blocks, us: 100 x 100 centers 0.5 m apart, 7600 points 154
// and 108, at 1 m 50 and 112, 40,000 points 132 and 141, 80,000 218 and 159; 60 x 60 at
// 0.75 m, 5400 points 58 and 65, 14,400 104 and 72; 16,000 x 1 at 0.5 m, 12,160 points 59
// and 172, 128,000 245 and 248; 10 x 10, 100 points 66 and 60.
// More bins than centers (scattered ones) are mostly empty blocks; below 100 points
// in all (77 on 10 x 10 centers: 52 and 60) and 3 / 4 per center the rows are ahead.
static bool gram_by_blocks(const rbf_grid* g, int64_t M, int64_t ld, int64_t strips) {
  const double N = (double)g->N, bins = (double)g->nbx * g->nby;
  const double bx = g->nbx - 2, by = g->nby - 2;  // bins with centers
  const double near = (double)M / (bx * by) * (3.0 - 2.0 / bx) * (3.0 - 2.0 / by);
  const double read = near * std::ceil(g->max_cand / 56.0);
  double rows = std::max(1.4e-3 * N + 0.105e-3 * N * read, 3.0 + 0.22 * read);
  // a line of bins: rows of few entries leave most lanes without one
  if (bx < 2 || by < 2) rows *= g->max_cand <= 16 ? 1.6 : g->max_cand <= 32 ? 1.3 : 1.0;
  // each strip also gathers for the bins next to its own
  const double next = strips > 1 ? 2.0 * strips * g->nbx : 0.0;
  const double blocks = 9.0 * strips + 8.4e-3 * bins + 2.5e-3 * next + 1.1e-3 * N +
                        2.9e-6 * bx * by * ld * ld + 0.35e-3 * M;
  return rows > blocks;
}

extern "C" {

rbf_status rbf_assemble_phi(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                            const double* xy, int64_t M, rbf_prec prec, void* vals,
                            int32_t* cols, int32_t* nnz, int32_t kmax) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_grid(ctx, p, g, "rbf_assemble_phi"));
  if (M < 0 || kmax <= 0 || (M > 0 && (!xy || !vals || !cols || !nnz)))
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_assemble_phi: bad pointer, M or kmax");
  if (prec != RBF_F64 && prec != RBF_F32)
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_assemble_phi: prec must be F64 or F32");
  if (M == 0) return RBF_OK;
  RBF_TRY(set_device(ctx));
  RegK k = reg_consts(p);
  if (prec == RBF_F64)
    k_assemble_phi<double><<<ceil_div(M, 16), 256, 0, ctx->stream>>>(
        xy, M, g->d_cxy, g->d_idx, g->d_start, geom(g), k, kmax, (double*)vals, cols, nnz,
        ctx->d_status);
  else
    k_assemble_phi<float><<<ceil_div(M, 16), 256, 0, ctx->stream>>>(
        xy, M, g->d_cxy, g->d_idx, g->d_start, geom(g), k, kmax, (float*)vals, cols, nnz,
        ctx->d_status);
  RBF_LAUNCHED(ctx, "k_assemble_phi");
  return RBF_OK;
}

rbf_status rbf_gram_pattern(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                            int64_t* rowptr, int32_t* colidx, int64_t cap, int64_t* nnz_out) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_grid(ctx, p, g, "rbf_gram_pattern"));
  if (!rowptr || !nnz_out || cap < 0 || (cap > 0 && !colidx))
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_gram_pattern: bad pointer or cap");
  RBF_TRY(set_device(ctx));
  const double st = std::sqrt(p->sigma * p->sigma + p->sigma_eps * p->sigma_eps);
  const double r = 2.0 * p->cutoff * st;
  const int64_t N = g->N;
  k_gram_count<<<ceil_div(N, 256), 256, 0, ctx->stream>>>(g->d_cxy, N, g->d_idx, g->d_start,
                                                          geom(g), r * r, rowptr);
  RBF_LAUNCHED(ctx, "k_gram_count");
  k_scan_excl_i64<<<1, 1024, 0, ctx->stream>>>(rowptr, N);
  RBF_LAUNCHED(ctx, "k_scan_excl_i64");
  if (cap > 0) {
    k_gram_fill<<<ceil_div(N, 256), 256, 0, ctx->stream>>>(g->d_cxy, N, g->d_idx, g->d_start,
                                                           geom(g), r * r, rowptr, colidx, cap);
    RBF_LAUNCHED(ctx, "k_gram_fill");
  }
  int64_t nnz = 0;
  RBF_HIP(ctx, hipMemcpyAsync(&nnz, rowptr + N, sizeof(int64_t), hipMemcpyDeviceToHost,
                              ctx->stream));
  RBF_HIP(ctx, hipStreamSynchronize(ctx->stream));
  *nnz_out = nnz;
  if (nnz > cap)
    return fail(ctx, RBF_E_CAPACITY, "rbf_gram_pattern: nnz %lld > cap %lld",
                (long long)nnz, (long long)cap);
  return RBF_OK;
}

rbf_status rbf_assemble_gram(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g,
                             const double* xy, const double* z, int64_t M,
                             const int64_t* rowptr, const int32_t* colidx, double* vals,
                             double* b, int32_t add_lambda) {
  if (!ctx) return RBF_E_INVALID_ARG;
  RBF_TRY(check_grid(ctx, p, g, "rbf_assemble_gram"));
  if (M < 0 || M >= ((int64_t)1 << 31) || !rowptr || !colidx || !vals || !b ||
      (M > 0 && (!xy || !z)))
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_assemble_gram: bad pointer or M");
  if (add_lambda && !(p->lambda >= 0))
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_assemble_gram: lambda < 0");
  RBF_TRY(set_device(ctx));
  rbf_status st;
  const int64_t nbins = (int64_t)g->nbx * g->nby;
  const int64_t Mc = M > 0 ? M : 1;
  int32_t* keys = (int32_t*)ws_get(ctx, WS_SORT0, sizeof(int32_t) * Mc, &st);
  if (!keys) return st;
  int32_t* pstart = (int32_t*)ws_get(ctx, WS_SORT1, sizeof(int32_t) * (nbins + 1), &st);
  if (!pstart) return st;
  int32_t* perm = (int32_t*)ws_get(ctx, WS_TMP0, sizeof(int32_t) * Mc, &st);
  if (!perm) return st;
  double* pxy = (double*)ws_get(ctx, WS_TMP1, sizeof(double) * 2 * Mc, &st);
  if (!pxy) return st;
  double* pz = (double*)ws_get(ctx, WS_TMP3, sizeof(double) * Mc, &st);
  if (!pz) return st;
  RBF_TRY(rbf_sort_points(ctx, g, xy, z, M, pxy, pz, perm));
  if (M == 0) {
    // only the ridge term
    RBF_TRY(fill_zero(ctx, pstart, sizeof(int32_t) * (nbins + 1)));
  } else {
    // rbf_sort_points leaves the bin offsets of the sorted points in WS_SORT1
  }
  RegK k = reg_consts(p);
  const int64_t N = g->N;
  const double lambda = add_lambda ? p->lambda : 0.0;
  const int64_t ld = ceil_div(g->max_cand > 0 ? g->max_cand : 1, 16) * 16;
  const int64_t blk = sizeof(double) * ld * (ld + 1) + 4 * sizeof(int32_t);  // bytes per bin
  const int64_t strip = std::min<int64_t>(nbins, (int64_t)(GRAM_WS / blk));
  char* ws = nullptr;
  if (ld <= GRAM_RMAX && M >= 100 && 4 * M >= 3 * N && nbins <= N &&
      gram_by_blocks(g, M, ld, ceil_div(nbins, strip)))
    ws = (char*)ws_try(ctx, WS_GRAM, (size_t)(strip * blk));
  if (!ws) {  // or no room for the blocks
    k_gram_values<<<ceil_div(N, 4), 256, 0, ctx->stream>>>(
        g->d_cxy, g->d_rank, N, g->d_idx, pxy, pz, pstart, geom(g), k, rowptr, colidx, lambda,
        vals, b);
    RBF_LAUNCHED(ctx, "k_gram_values");
    return RBF_OK;
  }
  double* G = (double*)ws;
  double* B = G + strip * ld * ld;
  int32_t* off = (int32_t*)(B + strip * ld);
  for (int64_t b0 = 0; b0 < nbins; b0 += strip) {
    const int32_t nb = (int32_t)std::min(strip, nbins - b0);
    if (ld <= 128)
      k_gram_bins<128><<<(unsigned)nb, GRAM_NT, 0, ctx->stream>>>(
          g->d_cxy, g->d_start, pxy, pz, pstart, geom(g), k, (int32_t)b0, (int32_t)ld, G, B, off);
    else
      k_gram_bins<GRAM_RMAX><<<(unsigned)nb, GRAM_NT, 0, ctx->stream>>>(
          g->d_cxy, g->d_start, pxy, pz, pstart, geom(g), k, (int32_t)b0, (int32_t)ld, G, B, off);
    RBF_LAUNCHED(ctx, "k_gram_bins");
    // the bins next to the strip's
    const int64_t f = std::max<int64_t>(0, b0 - g->nbx - 1);
    const int64_t l = std::min<int64_t>(nbins, b0 + nb + g->nbx + 1);
    k_gram_gather<<<(unsigned)(l - f), 256, 0, ctx->stream>>>(
        g->d_cxy, g->d_start, g->d_rank, g->d_idx, geom(g), (int32_t)f, (int32_t)b0, nb,
        (int32_t)ld, G, B, off, rowptr, colidx, lambda, vals, b);
    RBF_LAUNCHED(ctx, "k_gram_gather");
  }
  return RBF_OK;
}

rbf_status rbf_assemble(rbf_ctx* ctx, const rbf_params* p, const rbf_grid* g, const double* xy,
                        const double* z, int64_t M, int32_t what, rbf_prec prec, void* phi_val,
                        int32_t* phi_col, int32_t* phi_nnz, int32_t kmax, rbf_csr* H, double* b,
                        int32_t add_lambda) {
  if (!ctx) return RBF_E_INVALID_ARG;
  if (what == 0 || (what & ~(RBF_ASSEMBLE_PHI | RBF_ASSEMBLE_GRAM)) != 0)
    return fail(ctx, RBF_E_INVALID_ARG, "rbf_assemble: what must be PHI and/or GRAM");
  if ((what & RBF_ASSEMBLE_GRAM) != 0) {
    if (prec != RBF_F64)
      return fail(ctx, RBF_E_INVALID_ARG, "rbf_assemble: the Gram matrix is FP64 only");
    if (!H || !g || H->n != g->N)
      return fail(ctx, RBF_E_INVALID_ARG, "rbf_assemble: H missing or H->n != N");
  }
  if ((what & RBF_ASSEMBLE_PHI) != 0)
    RBF_TRY(rbf_assemble_phi(ctx, p, g, xy, M, prec, phi_val, phi_col, phi_nnz, kmax));
  if ((what & RBF_ASSEMBLE_GRAM) != 0)
    RBF_TRY(rbf_assemble_gram(ctx, p, g, xy, z, M, H->rowptr, H->colidx, H->vals, b,
                              add_lambda));
  return RBF_OK;
}

}  // extern "C"

// Inverse of the Cholesky factor of one 64x64 SPD block, for a 256-thread
// workgroup (included by update.hip inside namespace rbf, after its tile
// helpers).
//
// What bounds it is the dependent chain of 64 pivots (reciprocal, two FMAs,
// scaling, next column: about 56 cycles each), so the chain is kept free of
// everything else. FP64 products on the matrix pipe do not overlap FP64
// vector work of the same SIMD, so what is not on the chain has to be on
// another wave. Four 16-column panels, eliminated four columns at a time
// (group q = columns 4q .. 4q + 3), as L D L^T without square roots:
//   - Wave p is the chain of panel p. It holds the panel's 16x16 diagonal
//     block in the accumulator layout of v_mfma_f64_16x16x4 (element
//     (4v + l / 16, l % 16) in lane l, item v). The block is symmetric, so
//     item q is at the same time the group's four columns, row l % 16 and
//     column 4q + l / 16, which is the A and the B operand layout of the
//     group's rank-4 update. Only the four columns' exchange among a lane's
//     four row groups (lane swaps) moves data. The pivot comes from its lane
//     by a DPP row broadcast, and the later columns of the group take their
//     update as FMAs whose column entry is the FMA's own DPP source.
//   - After each group the chain publishes its columns and pivots in LDS.
//     Wave w > p follows one group behind with row block w of the panel (held
//     transposed, in the same layout), and adds each finished group to its
//     own diagonal block: after the last group of panel p wave p + 1 has its
//     diagonal block ready and goes on as the chain without waiting for
//     anyone.
//   - A wave that has been the chain (w <= p) carries row block w of the
//     identity through the same steps: the elimination turns [A; I] into
//     [L; L^{-T}], so these rows end as the rows of L^{-T}, scaled by
//     1 / sqrt(pivot) (v_rsq_f64 and two Newton-Raphson steps) when they are
//     stored. They run behind the chain and end about four groups after it.
// Pivots, panel rows and inverse rows are scaled by reciprocals within 11 ulp
// (rcp_nr); chol64_phased takes correctly rounded ones for the panel rows. All sums
// are FP64 in both.
// The waves wait for each other by progress words in LDS. A wave only ever
// waits for an earlier panel or an earlier wave of the same panel, the
// first chain waits for nothing, and all four waves of the workgroup are
// resident, so every wait ends.
//
// Phases of their own on four waves (16x16 factor, panel rows, trailing
// products, inverse) took 26.9k cycles per block, every wave doing the chain
// and one row block in step 19.2k; this form takes 14.6k. Cholesky step
// launches of a single update: 20.4 -> 16.0 us.
#pragma once

// Value of v in lane k of each row of 16 lanes: DPP row_newbcast (gfx90a
// and later), two 32-bit moves per double, no LDS and no scalar registers.
template <int K>
__device__ __forceinline__ double dpp_bcast16(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + K, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + K, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
// k must fold to a constant (unrolled loops), which leaves one case.
__device__ __forceinline__ double row_bcast16(double v, int k) {
  switch (k) {
    case 0: return dpp_bcast16<0>(v);
    case 1: return dpp_bcast16<1>(v);
    case 2: return dpp_bcast16<2>(v);
    case 3: return dpp_bcast16<3>(v);
    case 4: return dpp_bcast16<4>(v);
    case 5: return dpp_bcast16<5>(v);
    case 6: return dpp_bcast16<6>(v);
    case 7: return dpp_bcast16<7>(v);
    case 8: return dpp_bcast16<8>(v);
    case 9: return dpp_bcast16<9>(v);
    case 10: return dpp_bcast16<10>(v);
    case 11: return dpp_bcast16<11>(v);
    case 12: return dpp_bcast16<12>(v);
    case 13: return dpp_bcast16<13>(v);
    case 14: return dpp_bcast16<14>(v);
    default: return dpp_bcast16<15>(v);
  }
}

// a += v(lane k of its row of 16) * m as one v_fmac_f64 with a DPP
// row_newbcast source (the only DPP control 64-bit operands take), instead
// of two 32-bit broadcasts and an FMA. Same fused operation, so the same
// result. A DPP read needs two wait states after the VALU write of its
// source; the compiler pads its own DPP reads after inline asm, but not
// the DPP read inside this asm, so every source given to it here is either
// loaded from LDS or written several dependent instructions earlier (a
// listing check over the compiled kernels confirms it).
template <int K>
__device__ __forceinline__ void fmac_bcast16_k(double& a, double v, double m) {
  asm volatile("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
               : "+v"(a)
               : "v"(v), "v"(m), "i"(K));
}
// a -= v(lane K of its row of 16) * m, the same instruction with the
// multiplier negated by the operand modifier.
template <int K>
__device__ __forceinline__ void fnmac_bcast16_k(double& a, double v, double m) {
  asm volatile("v_fmac_f64_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
               : "+v"(a)
               : "v"(v), "v"(m), "i"(K));
}
// k must fold to a constant (unrolled loops), which leaves one case.
#define RBF_BCAST16_CASES(F, ...)                                     \
  switch (k) {                                                        \
    case 0: F<0>(__VA_ARGS__); break;                                 \
    case 1: F<1>(__VA_ARGS__); break;                                 \
    case 2: F<2>(__VA_ARGS__); break;                                 \
    case 3: F<3>(__VA_ARGS__); break;                                 \
    case 4: F<4>(__VA_ARGS__); break;                                 \
    case 5: F<5>(__VA_ARGS__); break;                                 \
    case 6: F<6>(__VA_ARGS__); break;                                 \
    case 7: F<7>(__VA_ARGS__); break;                                 \
    case 8: F<8>(__VA_ARGS__); break;                                 \
    case 9: F<9>(__VA_ARGS__); break;                                 \
    case 10: F<10>(__VA_ARGS__); break;                               \
    case 11: F<11>(__VA_ARGS__); break;                               \
    case 12: F<12>(__VA_ARGS__); break;                               \
    case 13: F<13>(__VA_ARGS__); break;                               \
    case 14: F<14>(__VA_ARGS__); break;                               \
    default: F<15>(__VA_ARGS__); break;                               \
  }
__device__ __forceinline__ void fmac_bcast16(double& a, double v, double m, int k) {
  RBF_BCAST16_CASES(fmac_bcast16_k, a, v, m)
}
__device__ __forceinline__ void fnmac_bcast16(double& a, double v, double m, int k) {
  RBF_BCAST16_CASES(fnmac_bcast16_k, a, v, m)
}
#undef RBF_BCAST16_CASES

// 1/p: the v_rcp_f64 estimate (about 24 correct bits) and one
// Newton-Raphson step r <- r + r (1 - p r), which doubles them: within 11
// ulp of 1/p (measured over random pivots), a relative error of the factor
// far below the rounding of its own sums. A second step (correctly rounded)
// costs two more dependent FMAs per pivot on the factor's critical path.
__device__ __forceinline__ double rcp_nr(double p) {
  double r = __builtin_amdgcn_rcp(p);
  r = fma(r, fma(-p, r, 1.0), r);
  return r;
}

// 1/sqrt(p): the v_rsq_f64 estimate and two Newton-Raphson steps (off the
// factor's dependent chain).
__device__ __forceinline__ double rsq_nr(double p) {
  double r = __builtin_amdgcn_rsq(p);
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double e = fma(-p * r, r, 1.0);
    r = fma(0.5 * r, e, r);
  }
  return r;
}

// Column exchange among the four 16-lane rows of a wave: o[k] in every lane
// = v of the lane with the same l % 16 in row k. v_permlane32_swap exchanges
// the upper half of its first with the lower half of its second operand,
// v_permlane16_swap the odd rows of the first with the even rows of the
// second; given the same value twice they return it spread over both.
__device__ __forceinline__ void row_exchange(double v, double (&o)[4]) {
  const auto l2 = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false,
                                                   false);
  const auto h2 = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false,
                                                   false);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto l = __builtin_amdgcn_permlane16_swap(l2[h], l2[h], false, false);
    const auto u = __builtin_amdgcn_permlane16_swap(h2[h], h2[h], false, false);
    o[2 * h] = __hiloint2double(u[0], l[0]);
    o[2 * h + 1] = __hiloint2double(u[1], l[1]);
  }
}

// o[k] with k = the lane's row of 16 (kq): the way back into operand layout.
// (Passed by value: a select between two array elements in memory would put
// the array there.)
__device__ __forceinline__ double row_pick(double o0, double o1, double o2, double o3, int kq) {
  const double lo = (kq & 1) ? o1 : o0, hi = (kq & 1) ? o3 : o2;
  return (kq & 2) ? hi : lo;
}


// Exchange buffers of one factor, laid over the input tile once it is read.
struct Chol64Lds {
  double c[4][256];     // panel p: column 4q + k, row i at 64 q + 16 k + i
  double x[3][3][256];  // row block r (at r - 1) after panel p, the same layout
  double rp[64];        // 1 / pivot
  double pv[64];        // pivot
};
static_assert(sizeof(Chol64Lds) <= sizeof(double) * NB * LDT, "fits the input tile");

// Progress words, written after the data they announce. LDS operations of one
// wave are carried out in order, so the words need no fence of their own;
// the clobbers keep the compiler to the same order. (Relaxed atomics rather
// than volatile accesses, which the compiler leaves as generic ones that
// wait for every global access as well.)
__device__ __forceinline__ void lds_post(int32_t* f, int32_t v) {
  asm volatile("" ::: "memory");
  __hip_atomic_store(f, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_wait(int32_t* f, int32_t v) {
  while (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < v) {
  }
  asm volatile("" ::: "memory");
}

// Chain: group Q of the panel whose diagonal block is dg. Rows already
// eliminated keep rounding residues that no later step reads. c: the panel's
// columns in LDS; rp, pv: its pivots.
template <int Q>
__device__ __forceinline__ void chain_group(v4d& dg, int lane, int kq, double* c_out,
                                            double* rp_out, double* pv_out,
                                            int32_t* prog) {
  double c[4], pv[4], rp[4];
  row_exchange(dg[Q], c);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    pv[k] = row_bcast16(c[k], 4 * Q + k);
    rp[k] = rcp_nr(pv[k]);
    const double t = c[k] * rp[k];
#pragma unroll
    for (int m = k + 1; m < 4; ++m)
      fnmac_bcast16(c[m], c[k], t, 4 * Q + m);  // c_m -= c_k[row of pivot m] t
  }
  const double da = row_pick(c[0], c[1], c[2], c[3], kq);
  const double r = row_pick(rp[0], rp[1], rp[2], rp[3], kq);
  c_out[64 * Q + lane] = da;
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      rp_out[4 * Q + k] = rp[k];
      pv_out[4 * Q + k] = pv[k];
    }
  }
  lds_post(prog, Q + 1);
  if (Q < 3) dg = __builtin_amdgcn_mfma_f64_16x16x4f64(da, -(da * r), dg, 0, 0, 0);
}

// Row block: group Q of a panel, once the chain has published it. blk: the
// wave's row block of the panel; xp: its finished columns (operand layout,
// unscaled), xb: times -1 / pivot.
template <int Q>
__device__ __forceinline__ void row_group(v4d& blk, int lane, int kq, const double* c_in,
                                          const double* rp_in, int32_t* prog,
                                          double& xp, double& xb) {
  double x[4];
  row_exchange(blk[Q], x);
  lds_wait(prog, Q + 1);
  double c[3], rp[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c[k] = c_in[64 * Q + 16 * k + (lane & 15)];
    rp[k] = rp_in[4 * Q + k];
  }
  const double rq = rp_in[4 * Q + kq], da = c_in[64 * Q + lane];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double u = x[k] * rp[k];
#pragma unroll
    for (int m = k + 1; m < 4; ++m) fnmac_bcast16(x[m], c[k], u, 4 * Q + m);
  }
  xp = row_pick(x[0], x[1], x[2], x[3], kq);
  xb = -(xp * rq);
  if (Q < 3) blk = __builtin_amdgcn_mfma_f64_16x16x4f64(da, xb, blk, 0, 0, 0);
}

// The wave's block of a later panel r takes panel p's columns: xr = row block
// r of panel p (LDS).
__device__ __forceinline__ void row_update(v4d& blk, const double* xr, int lane,
                                           const double (&xb)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q)
    blk = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[64 * q + lane], xb[q], blk, 0, 0, 0);
}

// T (LDS, lower triangle read; overwritten by the exchange): the block.
// Linv (64 x 64, row-major) receives L^{-1} (zero above the diagonal), and
// with LiT (leading dimension ldt, zero above the diagonal on entry) its
// transpose. A non-positive or non-finite pivot records RBF_E_NOT_SPD with
// `index` for launch group `seq` (the factor runs to its end; its output is
// then not used).
__device__ __forceinline__ void chol64(double (*T)[LDT], double* __restrict__ Linv,
                                       double* __restrict__ LiT, int64_t ldt, int32_t* status,
                                       int64_t index, int64_t seq) {
  __shared__ int32_t prog[4];      // groups of panel p published by its chain
  __shared__ int32_t xprog[4][3];  // row block r of panel p published
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, kq = lane >> 4;
  if (tid < 4) prog[tid] = 0;
  if (tid < 12) (&xprog[0][0])[tid] = 0;
  Chol64Lds& E = *reinterpret_cast<Chol64Lds*>(&T[0][0]);
  // blk[p]: the wave's row block of panel p, transposed (element (column i,
  // row li)): of the matrix for p < wave, of the identity from p = wave on
  v4d dg, blk[4];
  double a[3][4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = 4 * v + kq;
    dg[v] = T[16 * wave + max(i, li)][16 * wave + min(i, li)];
#pragma unroll
    for (int p = 0; p < 3; ++p) a[p][v] = T[16 * wave + li][16 * p + i];  // used if p < wave
  }
  // all loads issued, in bounds for any p: none behind a branch of its own
  asm volatile(""
               : "+v"(a[0][0]), "+v"(a[0][1]), "+v"(a[0][2]), "+v"(a[0][3]), "+v"(a[1][0]),
                 "+v"(a[1][1]), "+v"(a[1][2]), "+v"(a[1][3]), "+v"(a[2][0]), "+v"(a[2][1]),
                 "+v"(a[2][2]), "+v"(a[2][3]));
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      blk[p][v] = p < 3 && p < wave ? a[p < 3 ? p : 0][v]
                                    : ((p == wave && 4 * v + kq == li) ? 1.0 : 0.0);
  __syncthreads();  // T is read: it now serves the exchange
  if (wave > 0) {   // zeros above the diagonal, two 16x16 blocks per wave
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int z = 2 * (wave - 1) + e;  // (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
      const int pr = z < 3 ? 0 : z < 5 ? 1 : 2, pc = z < 3 ? z + 1 : z < 5 ? z - 1 : 3;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        Linv[(16 * pr + 4 * q + kq) * NB + 16 * pc + li] = 0.0;
    }
  }
  // ---- row block `wave` of the panels before the wave's own
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (p >= wave) break;
    double xp[4], xb[4];
#define RBF_ROW_GROUP(Q)                                                                     \
  row_group<Q>(blk[p], lane, kq, E.c[p], E.rp + 16 * p, &prog[p], xp[Q], xb[Q]);             \
  E.x[wave - 1][p][64 * Q + lane] = xp[Q];                                                   \
  dg = __builtin_amdgcn_mfma_f64_16x16x4f64(xp[Q], xb[Q], dg, 0, 0, 0);
    RBF_ROW_GROUP(0) RBF_ROW_GROUP(1) RBF_ROW_GROUP(2) RBF_ROW_GROUP(3)
#undef RBF_ROW_GROUP
    lds_post(&xprog[wave][p], 1);
#pragma unroll
    for (int r = 1; r < 3; ++r) {
      if (r <= p) continue;
      if (r >= wave) break;
      lds_wait(&xprog[r][p], 1);
      row_update(blk[r], E.x[r - 1][p], lane, xb);
    }
  }
  // ---- the chain of the wave's own panel
  {
    double* c = E.c[wave];
    double *rp = E.rp + 16 * wave, *pv = E.pv + 16 * wave;
    chain_group<0>(dg, lane, kq, c, rp, pv, &prog[wave]);
    chain_group<1>(dg, lane, kq, c, rp, pv, &prog[wave]);
    chain_group<2>(dg, lane, kq, c, rp, pv, &prog[wave]);
    chain_group<3>(dg, lane, kq, c, rp, pv, &prog[wave]);
  }
  // ---- row block `wave` of the identity, from the wave's own panel on
  bool good = true;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    if (p < wave) continue;
    double xp[4], xb[4];
    row_group<0>(blk[p], lane, kq, E.c[p], E.rp + 16 * p, &prog[p], xp[0], xb[0]);
    row_group<1>(blk[p], lane, kq, E.c[p], E.rp + 16 * p, &prog[p], xp[1], xb[1]);
    row_group<2>(blk[p], lane, kq, E.c[p], E.rp + 16 * p, &prog[p], xp[2], xb[2]);
    row_group<3>(blk[p], lane, kq, E.c[p], E.rp + 16 * p, &prog[p], xp[3], xb[3]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double pm = E.pv[16 * p + 4 * q + kq];
      good = good && pm > 0.0 && pm < INFINITY;
      const double lx = xp[q] * rsq_nr(pm);
      Linv[(16 * p + 4 * q + kq) * NB + 16 * wave + li] = lx;
      if (LiT) LiT[(int64_t)(16 * wave + li) * ldt + 16 * p + 4 * q + kq] = lx;
    }
#pragma unroll
    for (int r = 1; r < 4; ++r) {
      if (r <= p) continue;
      lds_wait(&xprog[r][p], 1);
      row_update(blk[r], E.x[r - 1][p], lane, xb);
    }
  }
  // wave 0 has seen every pivot
  if (wave == 0 && __ballot(!good) != 0 && lane == 0)
    set_status(status, RBF_E_NOT_SPD, index, seq);
}

// ------------------------------------------- the factor in four phases
//
// The form of the updates with FP32 or BF16 covariance products: Cholesky
// factor and inverse of T (in place, and in Ti). Those products round V, and
// a last bit of V moves a rounded operand now and then, after which the later
// batches' P differs by the products' own error (3.2e-5 relative at N = 5041,
// ten BF16x3 batches, between this form and the one above), so they keep
// this one and with it their results: 26.9k cycles per block against 14.6k.
// FP64 products have no such rounding (1.4e-11 between the two forms).
//
// Right-looking over four 16-column panels. For panel c0:
//   A. wave 0 factors the 16x16 diagonal block in registers, one row per lane
//      (lane g, g = lane % 16, holds row g); step j takes the pivot from its
//      lane with a DPP row broadcast and updates the later columns with
//      FP64 FMAs whose column entry comes from its lane through the FMA's
//      own DPP source (no LDS, no barrier), scaling by the pivot's
//      reciprocal only; after the 16 steps lane j takes the square root of
//      pivot j and its reciprocal, and broadcasts the reciprocal. It writes
//      L and 1 / L_jj;
//   B. the panel rows below, L_p D^T = A_p, by forward substitution in
//      registers (waves 1-3, one row per lane; lane g also holds row g of
//      the diagonal factor D, whose entries reach the other lanes the same
//      way);
//   C. the trailing lower blocks: A_rs -= L_r L_s^T (FP64 MFMA).
// Then the four diagonal 16x16 inverses, one per wave, by forward
// substitution (lane c holds column c, lane g row g of D), and the
// off-diagonal 16x16 blocks
// of the inverse by block diagonals:
//   Linv_ij = -Linv_ii sum_{j<=k<i} L_ik Linv_kj,
// where the f64 MFMA output layout (lane j + 16 (i % 4), item i / 4) is the
// B-operand layout of the next product's k-steps, so the two products chain
// in registers. No panel waits for an inverse. A non-positive or non-finite
// pivot records RBF_E_NOT_SPD with `index` for launch group `seq` (the
// factor runs to its end; its output is then not used).

// 16x16 product tile on FP64 MFMA: acc += A[r0.., a0..] * B where B[k][j] is
// B_t[b0 + j][bk0 + k] (i.e. the operand is read transposed from LDS).
__device__ __forceinline__ v4d mma16_nt(const double (*A)[LDT], int r0, int a0, const double (*Bt)[LDT],
                               int b0, int bk0, v4d acc) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int ks = 0; ks < 16; ks += 4) {
    const int kk = ks + (lane >> 4);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[r0 + (lane & 15)][a0 + kk],
                                               Bt[b0 + (lane & 15)][bk0 + kk], acc, 0, 0, 0);
  }
  return acc;
}

// Phase A for the diagonal block at (c0, c0): T gets L (zero above the
// diagonal), dinv[c0 + j] = 1 / L_jj; returns false if a pivot was not
// positive and finite. Wave 0 only.
// Step j works on the unscaled column c (c_g = a[g][j], pivot p_j = c_j):
// a[g][k] -= c_g c_k / p_j for j < k, so the square roots are off the
// dependent chain; afterwards L[g][j] = c_g / sqrt(p_j).
__device__ __forceinline__ bool chol16_factor(double (*T)[LDT], double* dinv, int c0) {
  const int lane = threadIdx.x & 63;
  const int g = lane & 15;
  double a[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) a[k] = T[c0 + g][c0 + k];
  int nbad = 0;  // counted without branches: the 16 steps stay one block
  double mypiv = 1.0;  // lane g keeps pivot g
  // The pivot test stays off the dependent chain of the steps: a pivot that
  // is not positive and finite is counted (the batch is then discarded
  // through the status word) and the factor goes on with it. Each step
  // updates the next pivot column first and broadcasts the next pivot.
  double pj = row_bcast16(a[0], 0);
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    nbad += 1 - ((int)(pj > 0.0) & (int)(pj < INFINITY));
    mypiv = (g == j) ? pj : mypiv;
    const double negt = -(a[j] * rcp_nr(pj));
    // entries above the diagonal (lanes g < k) receive unused values
    if (j + 1 < 16) {
      fmac_bcast16(a[j + 1], a[j], negt, j + 1);
      pj = row_bcast16(a[j + 1], j + 1);
    }
#pragma unroll
    for (int k = j + 2; k < 16; ++k) fmac_bcast16(a[k], a[j], negt, k);
  }
  __builtin_amdgcn_sched_barrier(0);
  // each lane takes the root and reciprocal of its own pivot (one square
  // root and one division per lane rather than sixteen) and the others
  // receive the reciprocals by broadcast. The broadcasts are statements of
  // their own: inside an arm of the select below they would make it a
  // branch, with the source lane switched off while they read it.
  const double mine_d = sqrt(mypiv);
  const double mine = 1.0 / mine_d;
  double rinv[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) rinv[j] = row_bcast16(mine, j);
#pragma unroll
  for (int j = 0; j < 16; ++j) a[j] = (g == j) ? mine_d : a[j] * rinv[j];
  __builtin_amdgcn_sched_barrier(0);
  if (lane < 16) {
#pragma unroll
    for (int k = 0; k < 16; ++k) T[c0 + g][c0 + k] = (k <= g) ? a[k] : 0.0;
    dinv[c0 + g] = mine;
  }
  return nbad == 0;
}

// Phase B for panel c0: row r (one per lane of waves 1..3, g = lane % 16)
// solves l D^T = a for its 16 entries, D = the panel's diagonal factor.
// Lane g also holds row g of D and 1 / D_gg, so D_kj and 1 / D_jj reach
// every lane by DPP broadcast from lane k (resp. j) rather than as LDS
// reads; the DPP sources come from LDS loads, never from a VALU write.
__device__ __forceinline__ void panel_rows(double (*T)[LDT], const double* dinv, int c0, int r) {
  const int lane = threadIdx.x & 63;
  const int g = lane & 15;
  double x[16], d[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) x[k] = T[r][c0 + k];
#pragma unroll
  for (int k = 0; k < 16; ++k) d[k] = T[c0 + g][c0 + k];
  const double dv = dinv[c0 + g];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    x[j] *= row_bcast16(dv, j);
#pragma unroll
    for (int k = j + 1; k < 16; ++k) fnmac_bcast16(x[k], d[j], x[j], k);  // x_k -= D_kj x_j
  }
  if (lane < 16) {
#pragma unroll
    for (int k = 0; k < 16; ++k) T[r][c0 + k] = x[k];
  }
}

// Inverse of the 16x16 diagonal factor block at (b0, b0) into Ti (lane c of
// the wave computes column c by forward substitution). Lane g holds row g
// of D and 1 / D_gg, broadcast by DPP as in panel_rows. The substitution is
// right-looking: once x_j is known, every later s_k takes its term at once,
// so the dependent chain is two operations per row (x_j, then s_{j+1})
// rather than a sum of up to 15 terms per row.
__device__ __forceinline__ void diag_inverse(const double (*T)[LDT], double (*Ti)[LDT],
                                             const double* dinv, int b0) {
  const int lane = threadIdx.x & 63;
  const int g = lane & 15;
  double x[16], d[16], s[16], dvb[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) d[k] = T[b0 + g][b0 + k];
  const double dv = dinv[b0 + g];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    s[k] = (g == k) ? 1.0 : 0.0;
    dvb[k] = row_bcast16(dv, k);
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    x[j] = s[j] * dvb[j];
#pragma unroll
    for (int k = j + 1; k < 16; ++k) fnmac_bcast16(s[k], d[j], x[j], k);  // s_k -= D_kj x_j
  }
  if (lane < 16) {
#pragma unroll
    for (int k = 0; k < 16; ++k) Ti[b0 + k][b0 + g] = (k >= g) ? x[k] : 0.0;
  }
}

__device__ __forceinline__ void chol64_phased(double (*T)[LDT], double (*Ti)[LDT],
                                              int32_t* status, int64_t index, int64_t seq) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ int bad;
  __shared__ double dinv[NB];
  if (tid == 0) bad = 0;
  for (int c0 = 0; c0 < NB; c0 += 16) {
    // ---- A: 16x16 diagonal block (wave 0, registers)
    if (wave == 0) {
      const bool ok = chol16_factor(T, dinv, c0);
      if (lane == 0 && !ok) bad = 1;
    } else if (c0 == 0) {
      // meanwhile waves 1-3 clear the strictly upper 16x16 blocks of L and
      // of its inverse: no phase reads them, and the inverse's diagonal and
      // lower blocks are all written below
      for (int e = tid - 64; e < NB * NB; e += 192)
        if (((e & 63) >> 4) > (e >> 10)) {
          T[e >> 6][e & 63] = 0.0;
          Ti[e >> 6][e & 63] = 0.0;
        }
    }
    __syncthreads();
    const int nrb = (NB - c0 - 16) / 16;  // row blocks below the panel
    if (nrb == 0) break;
    // ---- B: panel rows below, L_p D^T = A_p
    if (wave >= 1 && wave <= nrb) panel_rows(T, dinv, c0, c0 + 16 * wave + (lane & 15));
    __syncthreads();
    // ---- C: trailing lower blocks A_rs -= L_r L_s^T
    const int nblocks = nrb * (nrb + 1) / 2;
    for (int bidx = wave; bidx < nblocks; bidx += 4) {
      int rb = 0;
      while ((rb + 1) * (rb + 2) / 2 <= bidx) ++rb;
      const int sb = bidx - rb * (rb + 1) / 2;
      const int r0 = c0 + 16 + 16 * rb, s0 = c0 + 16 + 16 * sb;
      v4d acc = (v4d){0.0, 0.0, 0.0, 0.0};
      acc = mma16_nt(T, r0, c0, T, s0, c0, acc);
#pragma unroll
      for (int v = 0; v < 4; ++v) T[r0 + 4 * v + (lane >> 4)][s0 + (lane & 15)] -= acc[v];
    }
    __syncthreads();
  }
  // ---- the four diagonal inverses, one per wave
  diag_inverse(T, Ti, dinv, 16 * wave);
  __syncthreads();
  // ---- off-diagonal blocks of the inverse, by block diagonals d = i - j
  for (int d = 1; d < 4; ++d) {
    const int nb = 4 - d;
    if (wave < nb) {
      const int i = wave + d, j = wave;
      v4d t = (v4d){0.0, 0.0, 0.0, 0.0};
      for (int k = j; k < i; ++k) {
        // t += L_ik Linv_kj: B[kk][col] = Linv[16k + kk][16j + col]
#pragma unroll
        for (int ks = 0; ks < 16; ks += 4) {
          const int kk = ks + (lane >> 4);
          t = __builtin_amdgcn_mfma_f64_16x16x4f64(T[16 * i + (lane & 15)][16 * k + kk],
                                                   Ti[16 * k + kk][16 * j + (lane & 15)], t, 0,
                                                   0, 0);
        }
      }
      // result = -Linv_ii t; t (output layout) is the B operand, item = k-step
      v4d res = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int kk = 4 * s + (lane >> 4);
        res = __builtin_amdgcn_mfma_f64_16x16x4f64(Ti[16 * i + (lane & 15)][16 * i + kk], t[s],
                                                   res, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v)
        Ti[16 * i + 4 * v + (lane >> 4)][16 * j + (lane & 15)] = -res[v];
    }
    __syncthreads();
  }
  if (tid == 0 && bad) set_status(status, RBF_E_NOT_SPD, index, seq);
}


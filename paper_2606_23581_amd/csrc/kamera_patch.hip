// gfx950 kernels of the compile-side patch forming (App. A compile step):
// the top-m singular triplets of each deficit Delta (n x d) as the stored
// patch, W = V_m^T and U = Delta V_m (the singular values folded in).
//
// By default W comes from form_tri_kernel (kamera_tridiag.hip).  Here are
// block Jacobi -- the solver on request (sweeps > 0), and for the units that
// kernel could not finish -- and form_u_kernel, which forms U = Delta W^T from
// the stored W.
//
// form_patch_kernel: one 1024-thread workgroup per (chunk, layer, head) unit,
// everything in LDS (d is padded to dp, a multiple of 16, with zero rows and
// columns):
//   1. Gram matrix G = Delta^T Delta at fp32 accuracy on bf16 MFMA (16x16x32):
//      Delta split exactly into three bf16 parts, six products per tile,
//      streamed in 64-row tiles with the next tile's loads in flight during
//      the products;
//   2. block Jacobi on G: the indices form dp/8 blocks of 8; each step pairs
//      the blocks round-robin (circle method) into dp/16 groups of 16
//      indices; one wave per group runs one cyclic Jacobi sweep on the
//      group's 16x16 principal submatrix, accumulating its rotation Q; then
//      G <- J^T G J and V <- V J with J = diag(Q_group) as 16x16 tile
//      products on fp32 MFMA.  Sweeps stop once the off-diagonal mass is
//      negligible against the diagonal;
//   3. rank the eigenvalues (diag G) of the real indices, keep the m largest;
//   4. W[k] = V[:, order[k]]^T, rounded to bf16, and sigma.
// With an orbit (Sec. 5, reorder) Delta is the mean of the members' deficits,
// formed on the fly wherever Delta is read.
// The eigenvalues of G are the squared singular values of Delta and its
// eigenvectors the right singular vectors, so U W is the rank-m truncation.
// Padded indices keep zero rows and columns: every rotation that touches
// one is the identity, so they never mix with the real spectrum.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "kamera.h"
#include "kamera_form.h"
#include "kamera_launch.h"

namespace kamera {

namespace {

constexpr int kFormThreads = 1024;
constexpr int kWaves = kFormThreads / 64;
constexpr int kGramRows = 64;          // Delta rows per staged tile of the Gram product
constexpr int kBlk = 8;                // block-Jacobi block width
constexpr int kGrp = 2 * kBlk;         // indices of one rotated group (two blocks)
constexpr int kLdQ = kGrp + 1;         // padded row stride of a group's 16x16 scratch
constexpr int kFormFallbackSweeps = 12; // Jacobi limit after a failed tridiagonal solve

__host__ __device__ inline int pad16(int d) { return (d + 15) & ~15; }
// bf16 offset of rows 8 j .. 8 j + 7 of column c in a staged Gram part:
// columns of kGramRows rows, their 16-byte pieces permuted by (c >> 1) & 7,
// so that the 32 lanes of a half wave reading 8-row pieces of 16 consecutive
// columns (two pieces each), and 16 lanes storing one piece of consecutive
// columns, touch distinct banks (16-byte reads are served per half wave over
// 512 bytes of banks, 16-byte stores per quarter wave over 256 bytes)
__device__ __forceinline__ int gram_slot(int c, int j) { return c * kGramRows + 8 * (j ^ ((c >> 1) & 7)); }
// row stride of G and V: == 2 (mod 32), so an MFMA operand load of 16 rows
// x 2 columns (half a wave) and a 16-row tile's row pieces fall on distinct banks
__host__ __device__ inline int gv_ld(int dp) { return dp + ((2 - dp) % 32 + 32) % 32; }

// circle method over `n` items at `step`: the (smaller, larger) members of pair k
__device__ __forceinline__ void circle_pair(int n, int step, int k, int& a, int& b) {
  const int pa = k == 0 ? 0 : 1 + (k - 1 + step) % (n - 1);
  const int pb = 1 + (n - 2 - k + step) % (n - 1);
  a = pa < pb ? pa : pb;
  b = pa < pb ? pb : pa;
}

// global index of local index r (0..15) of the group made of blocks (bi, bj)
__device__ __forceinline__ int group_index(int bi, int bj, int r) {
  return r < kBlk ? kBlk * bi + r : kBlk * bj + (r - kBlk);
}

__device__ __forceinline__ f32x4v mfma4(float a, float b, f32x4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float block_sum(float v, float* red) {
  // wave reduction, then across the 16 waves through LDS
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kFormThreads / 64; ++w) s += red[w];
  return s;
}

// The workgroup's dynamic LDS (one unit's working set).
extern __shared__ __align__(16) float form_lds[];

// Rotation (c, s) = (cos, sin) and t = tan that zero a[p][q] of the 2x2
// symmetric block [[app, apq], [apq, aqq]]: t is the smaller root of
// t^2 + 2 theta t - 1 = 0 with theta = (aqq - app) / (2 apq); no rotation
// when apq is negligible.  Hardware reciprocal and (reciprocal) square root:
// c^2 + s^2 = 1 to a few ulp, which is all the iteration needs.  Branch free.
__device__ __forceinline__ void rotation(float app, float aqq, float apq, float& c, float& s, float& t) {
  const bool act = fabsf(apq) > 1e-30f;
  const float theta = (aqq - app) * __builtin_amdgcn_rcpf(2.f * (act ? apq : 1.f));
  const float tt = (theta >= 0.f ? 1.f : -1.f) *
                   __builtin_amdgcn_rcpf(fabsf(theta) + __builtin_amdgcn_sqrtf(fmaf(theta, theta, 1.f)));
  t = act ? tt : 0.f;
  c = __builtin_amdgcn_rsqf(fmaf(t, t, 1.f));
  s = t * c;
}

// One cyclic Jacobi sweep, by one wave, on a group's 16x16 symmetric matrix S
// (at form_lds + so, row stride kLdQ); Q (at form_lds + qo, identity on entry)
// accumulates the rotations, so that on exit S = Q^T S_in Q.  Lane (kr, kc) =
// (lane / 8, lane % 8) owns the 2x2 block of S on the rows of pair kr and the
// columns of pair kc, and rows kr and kr + 8 of Q on the columns of pair kc;
// it derives both pairs' rotations itself from the values it reads, so a
// step is one round of reads followed by one round of writes.  The wave's LDS
// accesses are performed in program order, so no barrier is needed.
__device__ __forceinline__ void group_sweep(int so, int qo, int lane, float* G, int ld, int bi, int bj) {
  const int kr = lane >> 3, kc = lane & 7;
  // circle positions of both pairs at step 0; every step moves positions
  // 1..15 on by one (position 0 stays)
  int ra = kr, rb = 15 - kr;
  int ca = kc, cb = 15 - kc;
  int p = 0, q = 0, p2 = 0, q2 = 0;
  float na = 0.f, nb = 0.f, ne = 0.f, nf = 0.f;
#pragma unroll 3
  for (int st = 0; st < kGrp - 1; ++st) {
    p = min(ra, rb);
    q = max(ra, rb);
    p2 = min(ca, cb);
    q2 = max(ca, cb);
    const float rpp = form_lds[so + p * kLdQ + p], rqq = form_lds[so + q * kLdQ + q];
    const float rpq = form_lds[so + p * kLdQ + q];
    const float cpp = form_lds[so + p2 * kLdQ + p2], cqq = form_lds[so + q2 * kLdQ + q2];
    const float cpq = form_lds[so + p2 * kLdQ + q2];
    const float a0 = form_lds[so + p * kLdQ + p2], b0 = form_lds[so + p * kLdQ + q2];
    const float e0 = form_lds[so + q * kLdQ + p2], f0 = form_lds[so + q * kLdQ + q2];
    const float qp0 = form_lds[qo + kr * kLdQ + p2], qq0 = form_lds[qo + kr * kLdQ + q2];
    const float qp1 = form_lds[qo + (kr + 8) * kLdQ + p2], qq1 = form_lds[qo + (kr + 8) * kLdQ + q2];
    float c1, s1, t1, c2, s2, t2;
    rotation(rpp, rqq, rpq, c1, s1, t1);
    rotation(cpp, cqq, cpq, c2, s2, t2);
    const float a1 = c1 * a0 - s1 * e0, e1 = s1 * a0 + c1 * e0;
    const float b1 = c1 * b0 - s1 * f0, f1 = s1 * b0 + c1 * f0;
    na = c2 * a1 - s2 * b1;
    nb = s2 * a1 + c2 * b1;
    ne = c2 * e1 - s2 * f1;
    nf = s2 * e1 + c2 * f1;
    if (kr == kc) {
      // the pivot block (same four addresses): exact diagonal update,
      // off-diagonal zeroed
      na = a0 - t1 * b0;
      nf = f0 + t1 * b0;
      nb = 0.f;
      ne = 0.f;
    }
    form_lds[so + p * kLdQ + p2] = na;
    form_lds[so + p * kLdQ + q2] = nb;
    form_lds[so + q * kLdQ + p2] = ne;
    form_lds[so + q * kLdQ + q2] = nf;
    form_lds[qo + kr * kLdQ + p2] = c2 * qp0 - s2 * qq0;
    form_lds[qo + kr * kLdQ + q2] = s2 * qp0 + c2 * qq0;
    form_lds[qo + (kr + 8) * kLdQ + p2] = c2 * qp1 - s2 * qq1;
    form_lds[qo + (kr + 8) * kLdQ + q2] = s2 * qp1 + c2 * qq1;
    __builtin_amdgcn_wave_barrier();
    ra = ra == 0 ? 0 : (ra == 15 ? 1 : ra + 1);
    rb = rb == 15 ? 1 : rb + 1;
    ca = ca == 0 ? 0 : (ca == 15 ? 1 : ca + 1);
    cb = cb == 15 ? 1 : cb + 1;
  }
  // The last step wrote every entry of S = Q^T G_gg Q: the group's diagonal
  // tile of the rotated G.  Lanes on and above the pair diagonal store their
  // 2x2 block with its mirror, so G stays exactly symmetric.
  if (kr <= kc) {
    const int gp = group_index(bi, bj, p), gq = group_index(bi, bj, q);
    const int gp2 = group_index(bi, bj, p2), gq2 = group_index(bi, bj, q2);
    G[gp * ld + gp2] = na;
    G[gp * ld + gq2] = nb;
    G[gq * ld + gp2] = ne;
    G[gq * ld + gq2] = nf;
    G[gp2 * ld + gp] = na;
    G[gq2 * ld + gp] = nb;
    G[gp2 * ld + gq] = ne;
    G[gq2 * ld + gq] = nf;
  }
}

// Rows i0 .. i0 + 7 of column j of the (orbit-mean) deficit (zero past n
// rows or d columns); a wave's lanes take consecutive columns, so each row's
// loads are one contiguous piece.  Orbit members are read two at a time, all
// their loads issued before the sums, which keep the members' order.
__device__ __forceinline__ void load_col8(const FormParams& P, const float* delta, int i0, int j, int n, int d,
                                          float (&x)[8]) {
  const float* v = delta + (int64_t)i0 * P.delta_s[3] + j;
  bool ok[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ok[e] = j < d && i0 + e < n;
    x[e] = ok[e] ? v[(int64_t)e * P.delta_s[3]] : 0.f;
  }
  if (P.n_orbit > 1) {
    for (int o = 1; o < P.n_orbit; o += 2) {
      const bool two = o + 1 < P.n_orbit;
      const float* v1 = v + (int64_t)o * P.orbit_s;
      const float* v2 = two ? v1 + P.orbit_s : v1;
      float y[8], z[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        y[e] = ok[e] ? v1[(int64_t)e * P.delta_s[3]] : 0.f;
        z[e] = ok[e] && two ? v2[(int64_t)e * P.delta_s[3]] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = (x[e] + y[e]) + z[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] *= P.inv_orbit;
  }
}

// V <- V J for one block-Jacobi step: the 16-row tile rt of group b's
// columns becomes V_tile Q_b (Q at form_lds + qo, group blocks in grp).  The
// (dp / 16) x ng tiles are spread over waves [w0, w0 + nw), four at a time
// with their MFMA chains interleaved; tiles are disjoint, so each is updated
// in place by its wave.
__device__ __forceinline__ void apply_v(float* V, int ld, int qo, const int* grp, const int* ident, int ng, int dp,
                                        int w0, int nw, int wave, int lj, int lr) {
  const int ntile = (dp / 16) * ng;
  const uint32_t ng_magic = (65536u + ng - 1) / ng;
  for (int t0 = wave - w0; t0 < ntile; t0 += 4 * nw) {
    bool ok[4];
    int rtile[4], gb[4], qb[4];
    float vv[4][4], qv[4][4];
    f32x4v vt[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + u * nw;
      ok[u] = t < ntile;
      const int rt = ok[u] ? (int)(((uint32_t)t * ng_magic) >> 16) : 0, b = ok[u] ? t - rt * ng : 0;
      ok[u] = ok[u] && !ident[b];            // Q_b = I leaves the tile as it is
      rtile[u] = rt;
      gb[u] = grp[b];
      qb[u] = qo + b * kGrp * kLdQ;
      const int bi = gb[u] & 0xff, bj = gb[u] >> 8;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        const int k = 4 * kb + lj;
        vv[u][kb] = ok[u] ? V[(16 * rt + lr) * ld + group_index(bi, bj, k)] : 0.f;
        qv[u][kb] = form_lds[qb[u] + k * kLdQ + lr];
      }
      vt[u] = (f32x4v){0.f, 0.f, 0.f, 0.f};
    }
    if (!ok[0] && !ok[1] && !ok[2] && !ok[3]) continue;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int u = 0; u < 4; ++u) vt[u] = mfma4(vv[u][kb], qv[u][kb], vt[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (ok[u]) {
        const int bi = gb[u] & 0xff, bj = gb[u] >> 8;
        const int gcol = group_index(bi, bj, lr);
#pragma unroll
        for (int i = 0; i < 4; ++i) V[(16 * rtile[u] + 4 * lj + i) * ld + gcol] = vt[u][i];
      }
    }
  }
}

}  // namespace

// The Gram tiles (I, J), I <= J, of nt x nt blocks of 16 go in sets of at
// most three consecutive tiles of one block row (row I's nt - I tiles split
// evenly), so a set's products share their A operand.  The sets are dealt
// largest first, in row order, each to the SIMD (wave mod 4) with the least
// work so far that still has a wave free.  Returns this wave's tile count
// (0: none) with its block row I and first block column J0; nt <= 8 makes at
// most 15 sets.
__device__ __forceinline__ int gram_set(int nt, int wave, int& I0, int& J0) {
  int l0 = 0, l1 = 0, l2 = 0, l3 = 0, u0 = 0, u1 = 0, u2 = 0, u3 = 0;
  for (int sz = 3; sz >= 1; --sz) {
    for (int I = 0; I < nt; ++I) {
      const int k = nt - I, ns = (k + 2) / 3, base = k / ns, extra = k - base * ns;
      int J = I;
      for (int s = 0; s < ns; ++s) {
        const int z = base + (s < extra ? 1 : 0);
        if (z == sz) {
          int q = -1, bl = 1 << 30;
          if (u0 < 4 && l0 < bl) { q = 0; bl = l0; }
          if (u1 < 4 && l1 < bl) { q = 1; bl = l1; }
          if (u2 < 4 && l2 < bl) { q = 2; bl = l2; }
          if (u3 < 4 && l3 < bl) { q = 3; bl = l3; }
          const int used = q == 0 ? u0 : q == 1 ? u1 : q == 2 ? u2 : u3;
          if (q + 4 * used == wave) {
            I0 = I;
            J0 = J;
            return z;
          }
          if (q == 0) { ++u0; l0 += z; }
          else if (q == 1) { ++u1; l1 += z; }
          else if (q == 2) { ++u2; l2 += z; }
          else { ++u3; l3 += z; }
        }
        J += z;
      }
    }
  }
  I0 = J0 = 0;
  return 0;
}

// The NS tiles (I, J0 + u) of a set on the staged rows: lane (kg, t) reads
// 8 consecutive rows of one column from each bf16 part (parts at Tb, part
// stride `part`), and a tile takes the six products of the parts that are
// not below 2^-27 relative.  A's three parts are loaded first; then B's parts
// one at a time, each used at once by the products that need it (hi: mid hi,
// lo hi, hi hi; mid: mid mid, hi mid; lo: hi lo), round the tiles, so
// consecutive MFMAs update different accumulators and only one B part per
// tile is held.  A diagonal first tile takes A's parts as its B.
template <int NS, bool DIAG>
__device__ __forceinline__ void gram_steps(const uint16_t* Tb, int part, int I, int J0, int kg, int t,
                                           f32x4v (&acc)[3]) {
#pragma unroll
  for (int ks = 0; ks < kGramRows / 32; ++ks) {
    const int kj = 4 * ks + kg;                // this lane's 8-row piece
    bf16x8v a[3];
    const uint16_t* pa = Tb + gram_slot(16 * I + t, kj);
#pragma unroll
    for (int q = 0; q < 3; ++q) a[q] = *reinterpret_cast<const bf16x8v*>(pa + q * part);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      bf16x8v b[NS];
#pragma unroll
      for (int u = 0; u < NS; ++u)
        b[u] = (DIAG && u == 0) ? a[q]
                                : *reinterpret_cast<const bf16x8v*>(Tb + gram_slot(16 * (J0 + u) + t, kj) + q * part);
      constexpr int kCount[3] = {3, 2, 1};   // A parts 1, 2, 0 | 1, 0 | 0
#pragma unroll
      for (int r = 0; r < kCount[q]; ++r) {
        const int ia = q == 0 ? (r == 0 ? 1 : r == 1 ? 2 : 0) : q == 1 ? (r == 0 ? 1 : 0) : 0;
#pragma unroll
        for (int u = 0; u < NS; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ia], b[u], acc[u], 0, 0, 0);
      }
    }
  }
}

// One unit: its Gram matrix, block Jacobi, W and sigma.
__device__ __forceinline__ void jacobi_unit(const FormParams& P, int unit, int sweeps) {
  float* const lds_f = form_lds;
  __shared__ int s_order[128];
  __shared__ float s_red[kWaves];
  __shared__ int s_grp[2][kFormMaxDim / (2 * kBlk)];   // blocks (bi | bj << 8) of each group, this and last step
  __shared__ int s_ident[2][kFormMaxDim / (2 * kBlk)]; // group kept Q = I, this and last step

  const int h = unit % P.n_heads;
  const int l = (unit / P.n_heads) % P.n_layers;
  const int c = unit / (P.n_heads * P.n_layers);
  const int d = P.dim, n = P.n_tokens, m = P.m;
  const int dp = pad16(d);                   // padded size (zero rows/columns beyond d)
  const int ld = gv_ld(dp);                  // padded LDS row stride of G and V
  const int nb = dp / kBlk;                  // Jacobi blocks (even)
  const int ng = nb / 2;                     // groups rotated per step
  float* G = lds_f;                          // [dp][ld]
  float* V = lds_f + dp * ld;                // [dp][ld]; holds Delta tiles in phase 1
  float* Ss = V + dp * ld;                   // [ng][16][kLdQ] group matrices
  float* Qs2 = Ss + ng * kGrp * kLdQ;        // [2][ng][16][kLdQ] group rotations of this and the last step
  const float* delta = P.delta + (int64_t)c * P.delta_s[0] + (int64_t)l * P.delta_s[1] + (int64_t)h * P.delta_s[2];
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int lj = lane >> 4, lr = lane & 15;  // MFMA operand slot (k within a step) and row/column

  // ---- 1. G = Delta^T Delta on MFMA: a wave owns up to 3 tiles of one block row ----
  {
    const int nt = dp / 16;
    uint16_t* Tb = reinterpret_cast<uint16_t*>(V);   // staged parts hi, mid, lo: [3][dp][kGramRows] bf16
    const int part = dp * kGramRows;
    // this wave's tiles (gI, gJ + u), u < my: the same on every lane
    int gI, gJ;
    const int my = __builtin_amdgcn_readfirstlane(gram_set(nt, wave, gI, gJ));
    gI = __builtin_amdgcn_readfirstlane(gI);
    gJ = __builtin_amdgcn_readfirstlane(gJ);
    const bool gdiag = gI == gJ;
    f32x4v acc[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) acc[u] = (f32x4v){0.f, 0.f, 0.f, 0.f};
    // thread (sg, sc) stages rows 8 sg .. 8 sg + 7 of column sc of each
    // kGramRows-row tile, split into three bf16 parts, as one 16-byte piece
    // per part; the next tile's loads are in flight during the products on
    // the current one
    const bool stager = tid < (kGramRows / 8) * dp;
    const int sg = stager ? tid / dp : 0, sc = stager ? tid - sg * dp : 0;
    float x[8];
    load_col8(P, delta, 8 * sg, stager ? sc : d, n, d, x);
    for (int t0 = 0; t0 < n; t0 += kGramRows) {
      __syncthreads();
      if (stager) {
        u32x4v hi, mid, lo;
        split3_bf16x8(x, hi, mid, lo);
        uint16_t* q = Tb + gram_slot(sc, sg);
        *reinterpret_cast<u32x4v*>(q) = hi;
        *reinterpret_cast<u32x4v*>(q + part) = mid;
        *reinterpret_cast<u32x4v*>(q + 2 * part) = lo;
      }
      __syncthreads();
      if (t0 + kGramRows < n) load_col8(P, delta, t0 + kGramRows + 8 * sg, stager ? sc : d, n, d, x);
      // the set is the same on every lane: one scalar branch picks a loop
      // without branches; rows past n are staged as zeros, so every tile
      // takes all k-steps
      if (gdiag) {
        if (my == 3) gram_steps<3, true>(Tb, part, gI, gJ, lj, lr, acc);
        else if (my == 2) gram_steps<2, true>(Tb, part, gI, gJ, lj, lr, acc);
        else if (my == 1) gram_steps<1, true>(Tb, part, gI, gJ, lj, lr, acc);
      } else {
        if (my == 3) gram_steps<3, false>(Tb, part, gI, gJ, lj, lr, acc);
        else if (my == 2) gram_steps<2, false>(Tb, part, gI, gJ, lj, lr, acc);
        else if (my == 1) gram_steps<1, false>(Tb, part, gI, gJ, lj, lr, acc);
      }
    }
    // lane (lj, lr) holds G[16 gI + 4 lj + i][16 (gJ + u) + lr]; store it and its mirror
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      if (u < my) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * gI + 4 * lj + i, col = 16 * (gJ + u) + lr;
          if (gI < gJ + u || row <= col) {
            G[row * ld + col] = acc[u][i];
            G[col * ld + row] = acc[u][i];
          }
        }
      }
    }
    __syncthreads();
    // V = I (the staged tile is no longer needed)
    for (int e = tid; e < dp * dp; e += kFormThreads) V[(e / dp) * ld + e % dp] = (e / dp == e % dp) ? 1.f : 0.f;
    __syncthreads();
  }

  // ---- 2. block Jacobi ----
  // Each step's V <- V J is deferred to the next step's first phase, where the
  // waves without a group to solve apply it while the others run their inner
  // sweeps; the Q buffers and group lists alternate between steps.
  int sweeps_run = 0;
  int cur = 0;                                 // buffer of the step being formed
  bool pending = false;                        // V still owes the previous step's rotation
  for (int sweep = 0; sweep < sweeps; ++sweep) {
    // stop once the off-diagonal mass is negligible against the diagonal
    float off = 0.f, dia = 0.f;
    for (int e = tid; e < d * d; e += kFormThreads) {
      const int i = e / d, j = e % d;
      const float g = G[i * ld + j];
      if (i == j) dia += g * g; else off += g * g;
    }
    off = block_sum(off, s_red);
    dia = block_sum(dia, s_red);
    if (off <= 1e-9f * dia) break;             // ~(d * 4 eps)^2: the fp32 floor
    ++sweeps_run;
    for (int step = 0; step < nb - 1; ++step) {
      float* Qs = Qs2 + cur * ng * kGrp * kLdQ;
      const int* grp = s_grp[cur];
      // (a) one wave per group: a Jacobi sweep on the group's principal
      // submatrix; the remaining waves apply the previous step to V
      if (wave < ng) {
        int bi, bj;
        circle_pair(nb, step, wave, bi, bj);
        if (lane == 0) s_grp[cur][wave] = bi | (bj << 8);
        const int so = (int)(Ss - lds_f) + wave * kGrp * kLdQ;
        const int qo = (int)(Qs - lds_f) + wave * kGrp * kLdQ;
        float goff = 0.f;
#pragma unroll
        for (int u = 0; u < kGrp * kGrp / 64; ++u) {
          const int e = lane + 64 * u, r = e >> 4, cc = e & 15;
          const float g = G[group_index(bi, bj, r) * ld + group_index(bi, bj, cc)];
          lds_f[so + r * kLdQ + cc] = g;
          lds_f[qo + r * kLdQ + cc] = r == cc ? 1.f : 0.f;
          if (r != cc) goff += g * g;
        }
        for (int o = 32; o > 0; o >>= 1) goff += __shfl_xor(goff, o, 64);
        // a group whose block is already diagonal to well below the
        // convergence test (at most 120 such groups per sweep stay under it)
        // keeps Q = I, and the tile products it would leave unchanged are skipped
        const bool skip = goff <= 1e-12f * dia;
        if (lane == 0) s_ident[cur][wave] = skip ? 1 : 0;
        __builtin_amdgcn_wave_barrier();
        if (!skip) group_sweep(so, qo, lane, G, ld, bi, bj);
      } else if (pending) {
        apply_v(V, ld, (int)(Qs2 - lds_f) + (cur ^ 1) * ng * kGrp * kLdQ, s_grp[cur ^ 1], s_ident[cur ^ 1], ng, dp,
                ng, kWaves - ng, wave, lj, lr);
      }
      __syncthreads();
      // (b) G <- J^T G J.  The diagonal tiles (a, a) are the groups' rotated
      // blocks Q_a^T G_aa Q_a, written by their inner sweeps.  An off-diagonal
      // tile (a < b) becomes Q_a^T G_ab Q_b on MFMA and is stored with its
      // mirror, so G stays exactly symmetric: at most ng (ng - 1) / 2 = 28 of
      // them, two per wave, their loads issued together and their MFMA chains
      // interleaved.
      {
        const int ntile = ng * (ng - 1) / 2;
        bool ok[2];
        int rowa[2], ga[2], gb[2];
        float gv[2][4], qv[2][4];
        f32x4v mt[2], tt[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          int t = wave + u * kWaves, a = 0;
          ok[u] = t < ntile;
          if (ok[u]) {
            while (t >= ng - 1 - a) {        // row a of the strict upper triangle holds ng - 1 - a tiles
              t -= ng - 1 - a;
              ++a;
            }
          }
          const int b = ok[u] ? a + 1 + t : 0;
          ok[u] = ok[u] && !(s_ident[cur][a] && s_ident[cur][b]);   // both sides kept Q = I
          ga[u] = grp[a];
          gb[u] = grp[b];
          rowa[u] = a;
          const int ai = ga[u] & 0xff, aj = ga[u] >> 8, bi = gb[u] & 0xff, bj = gb[u] >> 8;
          const float* Qb = Qs + b * kGrp * kLdQ;
          const int grow = group_index(ai, aj, lr);
#pragma unroll
          for (int kb = 0; kb < 4; ++kb) {
            const int k = 4 * kb + lj;
            gv[u][kb] = G[grow * ld + group_index(bi, bj, k)];
            qv[u][kb] = Qb[k * kLdQ + lr];
          }
          mt[u] = (f32x4v){0.f, 0.f, 0.f, 0.f};
          tt[u] = (f32x4v){0.f, 0.f, 0.f, 0.f};
        }
        if (ok[0] || ok[1]) {
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int u = 0; u < 2; ++u) mt[u] = mfma4(gv[u][kb], qv[u][kb], mt[u]);
          // T = Q_a^T M: step i sums k = 4 lj + i, whose M row this lane already holds
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const float* Qa = Qs + rowa[u] * kGrp * kLdQ;
#pragma unroll
            for (int i = 0; i < 4; ++i) qv[u][i] = Qa[(4 * lj + i) * kLdQ + lr];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int u = 0; u < 2; ++u) tt[u] = mfma4(qv[u][i], mt[u][i], tt[u]);
          // lane (lj, lr) holds T[4 lj + i][lr]: row of group a, column of group b
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            if (ok[u]) {
              const int ai = ga[u] & 0xff, aj = ga[u] >> 8, bi = gb[u] & 0xff, bj = gb[u] >> 8;
              const int gcol = group_index(bi, bj, lr);
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int grw = group_index(ai, aj, 4 * lj + i);
                G[grw * ld + gcol] = tt[u][i];
                G[gcol * ld + grw] = tt[u][i];
              }
            }
          }
        }
      }
      __syncthreads();
      pending = true;
      cur ^= 1;
    }
  }
  if (pending) {
    // the last step's rotation of V
    apply_v(V, ld, (int)(Qs2 - lds_f) + (cur ^ 1) * ng * kGrp * kLdQ, s_grp[cur ^ 1], s_ident[cur ^ 1], ng, dp, 0,
            kWaves, wave, lj, lr);
    __syncthreads();
  }
  if (P.sweeps_done != nullptr && tid == 0) P.sweeps_done[unit] = sweeps_run;

  // ---- 3. the m largest eigenvalues (ties by index; NaN counts as the least, so
  // that every rank is taken) ----
  if (tid < d) {
    const float li = fmaxf(G[tid * ld + tid], -__builtin_inff());
    int rank = 0;
    for (int j = 0; j < d; ++j) {
      const float lk = fmaxf(G[j * ld + j], -__builtin_inff());
      rank += (lk > li) || (lk == li && j < tid);
    }
    if (rank < m) s_order[rank] = tid;
  }
  __syncthreads();

  // ---- 4. W = V_m^T and sigma (U = Delta W^T follows in form_u_kernel) ----
  uint16_t* Wout = P.W + (int64_t)c * P.w_s[0] + (int64_t)l * P.w_s[1] + (int64_t)h * P.w_s[2];
  for (int e = tid; e < m * d; e += kFormThreads) {
    const int k = e / d, j = e % d;
    Wout[(int64_t)k * P.w_s[3] + j] = to_bf16_rne(V[j * ld + s_order[k]]);
  }
  if (P.sigma != nullptr && tid < m) {
    const float lam = G[s_order[tid] * ld + s_order[tid]];
    P.sigma[(int64_t)c * P.sigma_s[0] + (int64_t)l * P.sigma_s[1] + (int64_t)h * P.sigma_s[2] + tid] =
        sqrtf(lam > 0.f ? lam : 0.f);
  }
}

// FALLBACK = false: unit blockIdx.x, P.sweeps sweeps at most.  FALLBACK = true
// (after form_tri_kernel): a workgroup looks at its unit of every row of
// gridDim.x units (form_fallback_unit) and forms those whose W carries
// kFormFailMark.  Almost none does, so the grid is small and a workgroup reads
// 1024 marks at once: the kernel then costs its launch.
template <bool FALLBACK>
__global__ __launch_bounds__(kFormThreads) void form_patch_kernel(const FormParams /*by value, read in place*/) {
  const FormParams& P = *static_cast<const FormParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
  if constexpr (!FALLBACK) {
    jacobi_unit(P, blockIdx.x, P.sweeps);
  } else {
    __shared__ int s_todo;
    const uint32_t n_rows = ((uint32_t)P.n_units + gridDim.x - 1) / gridDim.x;   // (n_units < 2^22)
    for (uint32_t row0 = 0; row0 < n_rows; row0 += kFormThreads) {
      const int64_t unit = form_fallback_unit(row0 + threadIdx.x, blockIdx.x, gridDim.x);
      bool failed = false;
      if (unit < P.n_units) {
        const int64_t h = unit % P.n_heads, l = (unit / P.n_heads) % P.n_layers,
                      c = unit / ((int64_t)P.n_heads * P.n_layers);
        failed = P.W[c * P.w_s[0] + l * P.w_s[1] + h * P.w_s[2]] == kFormFailMark;
      }
      // the failed units one after the other, lowest thread first
      int from = 0;
      for (;;) {
        if (threadIdx.x == 0) s_todo = kFormThreads;
        __syncthreads();
        if (failed && (int)threadIdx.x >= from) atomicMin(&s_todo, (int)threadIdx.x);
        __syncthreads();
        const int t = s_todo;
        __syncthreads();                       // read before the next round resets it
        if (t >= kFormThreads) break;
        jacobi_unit(P, (int)form_fallback_unit(row0 + t, blockIdx.x, gridDim.x), kFormFallbackSweeps);
        from = t + 1;
      }
    }
  }
}

// LDS floats: phase 1 G [dp][gv_ld] and the staged parts [3][dp][kGramRows] bf16;
// phase 2 G and V [dp][gv_ld] each, the groups' S [16][17] and two sets of
// their Q [16][17]
size_t form_lds_bytes(int dim, int /*m*/) {
  const size_t dp = (size_t)pad16(dim), ld = (size_t)gv_ld((int)dp), ng = dp / (2 * kBlk);
  const size_t f1 = dp * ld + 3 * dp * kGramRows / 2;
  const size_t f2 = 2 * dp * ld + 3 * ng * kGrp * kLdQ;
  return (f1 > f2 ? f1 : f2) * sizeof(float);
}

// ---------------------------------------------------------------------------
// U = Delta W^T, the factor's token side, from the W that the solver has stored
// (so U W is formed from exactly the kept W).  A wave takes ROWS
// token rows of one unit, as 16-row tiles, and the ranks 64 at a time (the
// workgroup's four waves share those 64 W rows, staged once in LDS); the
// products are 16x16x32 bf16 MFMAs with fp32 accumulation.  Delta is read in
// fp32 and split into hi = bf16(Delta) and lo = bf16(Delta - hi), and both
// parts are multiplied, so Delta enters to ~2^-16 relative.  Lane (kg, t)
// holds row t of a tile on k-slots 8 kg .. 8 kg + 7 (A operand), rank t on
// the same slots (B operand), and rows 4 kg .. 4 kg + 3 of rank t of the
// product.  With an orbit the members' rows are averaged in fp32 first.
// ---------------------------------------------------------------------------
// token rows per wave: 64, so that the W rows a workgroup stages serve 256
// token rows; 16 while the launch then has fewer than 512 workgroups (two per
// CU).  Whole calls of 1024 rows, rank 64, with 16 and with 64: 8 units 200 and
// 209 us, 100 units 214 and 216, 128 (512 workgroups) 217 and 217, 256 239 and 233
constexpr int kURowsMany = 64, kURowsFew = 16;
constexpr int kUThreads = 256;
constexpr int kUWLd = 144;            // bf16 per staged W row: 288 bytes, so the B-operand reads
                                      // of a half wave (16 rows x 2 pieces) fall on distinct banks

template <int ROWS>
__global__ __launch_bounds__(kUThreads) void form_u_kernel(const FormParams /*by value, read in place*/) {
  const FormParams& P = *static_cast<const FormParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = lane & 15, kg = lane >> 4;
  const int n = P.n_tokens, d = P.dim, m = P.m;
  constexpr int kRowsPerBlock = ROWS * (kUThreads / 64);
  const uint32_t bpu = (uint32_t)((n + kRowsPerBlock - 1) / kRowsPerBlock);   // blocks per unit
  // workgroups go to the 8 XCDs in turn: block b takes the place
  // (b mod 8) * (grid / 8) + b / 8, so that the blocks of one unit share an
  // XCD and read its W from that XCD's L2 (the grid is a multiple of 8)
  const uint32_t place = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const uint32_t unit = place / bpu;
  if ((int)unit >= P.n_units) return;
  const int h = (int)(unit % (uint32_t)P.n_heads);
  const int l = (int)((unit / (uint32_t)P.n_heads) % (uint32_t)P.n_layers);
  const int c = (int)(unit / ((uint32_t)P.n_heads * (uint32_t)P.n_layers));
  const int row0 = (int)(place - unit * bpu) * kRowsPerBlock + wave * ROWS;
  // (a wave past the unit's rows still takes part in the W staging)
  __shared__ __align__(16) uint16_t s_w[64 * kUWLd];
  const float* delta = P.delta + (int64_t)c * P.delta_s[0] + (int64_t)l * P.delta_s[1] + (int64_t)h * P.delta_s[2];
  const uint16_t* Wu = P.W + (int64_t)c * P.w_s[0] + (int64_t)l * P.w_s[1] + (int64_t)h * P.w_s[2];
  uint16_t* Uu = P.U + (int64_t)c * P.u_s[0] + (int64_t)l * P.u_s[1] + (int64_t)h * P.u_s[2];
  const int ks = (d + 31) / 32;                // k-steps of 32 dims (<= 4)
  // Delta row i, dims [8 kg + 32 s, +8) as fp32 (zero past n or d; d is a multiple of 4)
  auto load_rows = [&](int i, float (&x)[4][8]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const int j = 32 * s + 8 * kg + 4 * hf;
        f32x4v v = {0.f, 0.f, 0.f, 0.f};
        if (s < ks && i < n && j < d) {
          const float* row = delta + (int64_t)i * P.delta_s[3] + j;
          v = *reinterpret_cast<const f32x4v*>(row);
          if (P.n_orbit > 1) {
            for (int o = 1; o < P.n_orbit; ++o) v += *reinterpret_cast<const f32x4v*>(row + (int64_t)o * P.orbit_s);
            v *= P.inv_orbit;
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) x[s][4 * hf + e] = v[e];
      }
  };
  for (int r0 = 0; r0 < m; r0 += 64) {
    // W rows r0 .. r0 + 63 into LDS, 16-byte pieces (zero past m or d), once
    // for the workgroup's four waves
    __syncthreads();                           // the previous ranks' W is consumed
#pragma unroll
    for (int q = 0; q < 64 * 16 / kUThreads; ++q) {
      const int e = threadIdx.x + q * kUThreads, rr = e >> 4, j0 = 8 * (e & 15);
      const int r = r0 + rr;
      u32x4v v = {0u, 0u, 0u, 0u};
      if (r < m && j0 < d) {
        const uint16_t* wr = Wu + (int64_t)r * P.w_s[3] + j0;
        if (P.w_vec && j0 + 8 <= d) {
          v = *reinterpret_cast<const u32x4v*>(wr);
        } else {
#pragma unroll
          for (int e2 = 0; e2 < 8; ++e2)
            if (j0 + e2 < d) v[e2 >> 1] |= (uint32_t)wr[e2] << (16 * (e2 & 1));
        }
      }
      *reinterpret_cast<u32x4v*>(s_w + rr * kUWLd + j0) = v;
    }
    __syncthreads();
    // B operands: W rows r0 + 16 ct + t, dims [8 kg + 32 s, +8)
    auto wb = [&](int ct, int s) {
      return *reinterpret_cast<const u32x4v*>(s_w + (16 * ct + t) * kUWLd + 32 * s + 8 * kg);
    };
    for (int rt = 0; rt < ROWS / 16; ++rt) {
      const int i0 = row0 + 16 * rt;
      if (i0 >= n) break;                      // uniform in the wave (no barrier inside)
      float x[4][8];
      load_rows(i0 + t, x);
      f32x4v acc[4];
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) acc[ct] = (f32x4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (s < ks) {
          float lo[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) lo[e] = x[s][e] - __uint_as_float((uint32_t)to_bf16_rne(x[s][e]) << 16);
          const bf16x8v ahi = __builtin_bit_cast(bf16x8v, pack_bf16x8(x[s]));
          const bf16x8v alo = __builtin_bit_cast(bf16x8v, pack_bf16x8(lo));
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) {
            const bf16x8v b = __builtin_bit_cast(bf16x8v, wb(ct, s));
            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, b, acc[ct], 0, 0, 0);
            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, b, acc[ct], 0, 0, 0);
          }
        }
      }
      if (P.u_pair) {
        // ranks t and t ^ 1 meet by a DPP swap; the even lane stores both
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          const int r = r0 + 16 * ct + t;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float nb = dpp_f<0xB1>(acc[ct][q]);
            const int i = i0 + 4 * kg + q;
            if ((t & 1) == 0 && r < m && i < n) {
              uint16_t* dst = Uu + (int64_t)i * P.u_s[3] + r;
              if (r + 1 < m)
                *reinterpret_cast<uint32_t*>(dst) = (uint32_t)to_bf16_rne(acc[ct][q]) | ((uint32_t)to_bf16_rne(nb) << 16);
              else
                *dst = to_bf16_rne(acc[ct][q]);
            }
          }
        }
      } else {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          const int r = r0 + 16 * ct + t;
          if (r < m) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int i = i0 + 4 * kg + q;
              if (i < n) Uu[(int64_t)i * P.u_s[3] + r] = to_bf16_rne(acc[ct][q]);
            }
          }
        }
      }
    }
  }
}

template <bool FALLBACK>
static hipError_t launch_jacobi(const FormParams& p, uint32_t grid, hipStream_t s) {
  static std::atomic<bool> lds_set[kMaxDevices];
  const hipError_t e = ensure_lds_limit((const void*)form_patch_kernel<FALLBACK>,
                                        (int)form_lds_bytes(kFormMaxDim, kFormMaxDim), lds_set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((form_patch_kernel<FALLBACK>), dim3(grid), dim3(kFormThreads), form_lds_bytes(p.dim, p.m), s, p);
  return hipGetLastError();
}

template <int ROWS>
static hipError_t launch_u(const FormParams& p, hipStream_t s) {
  constexpr int kRowsPerBlock = ROWS * (kUThreads / 64);
  const int64_t bpu = (p.n_tokens + kRowsPerBlock - 1) / kRowsPerBlock;
  const int64_t blocks = (bpu * p.n_units + 7) / 8 * 8;   // the places past the units return at once
  hipLaunchKernelGGL((form_u_kernel<ROWS>), dim3((uint32_t)blocks), dim3(kUThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_form_patch(const FormParams& p, hipStream_t s) {
  hipError_t e;
  if (p.sweeps > 0) {
    e = launch_jacobi<false>(p, (uint32_t)p.n_units, s);
  } else {
    e = launch_form_tridiag(p, s);
    if (e != hipSuccess) return e;
    e = launch_jacobi<true>(p, std::min((uint32_t)p.n_units, kFormFallbackGrid), s);
  }
  if (e != hipSuccess) return e;
  // U from the stored W, on the same stream: after the W of every unit
  return (p.n_tokens + 255) / 256 * (int64_t)p.n_units < 512 ? launch_u<kURowsFew>(p, s) : launch_u<kURowsMany>(p, s);
}

}  // namespace kamera

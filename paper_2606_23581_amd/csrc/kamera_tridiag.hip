// gfx950 kernel of the compile step's default solver: the top-m eigenpairs of
// each unit's Gram matrix G = Delta^T Delta by Householder tridiagonalisation.
//
// form_tri_kernel<NB>: one 256-thread workgroup (four waves) per (chunk, layer,
// head) unit, the d columns (d <= 32 NB) in NB blocks of 32, one block per wave
// ("role" J).  Wave J holds G's columns 32 J .. 32 J + 31, all rows, as NB
// accumulators of 32x32 MFMA tiles: lane l, element r of tile I is row
// 32 I + 8 (r / 4) + 4 (l / 32) + r % 4, column 32 J + l % 32.
//   1. G at fp32 accuracy on bf16 MFMA (32x32x16): Delta split exactly into
//      three bf16 parts h + m + l, the six products above 2^-27 relative,
//      straight into those accumulators; where a unit has a CU to itself, by
//      two groups of four waves (S = 2).
//   2. Householder reduction in the same registers (tri_reduce).
//   3. Eigenvalues by multisection on Sturm counts, eigenvectors of T by
//      twisted factorisation, close ones orthogonalised, checks.
//   4. Back-transformation, W = V_m^T (bf16) and sigma.
// A unit that fails its checks (exactly multiple eigenvalues make twisted
// vectors coincide) stores kFormFailMark in W and is formed again by the
// Jacobi kernel that follows on the stream.
//
// What bounds it: the phases of one unit are serial chains (126 dependent
// reflectors, recurrences of length d), none of which fills a CU.  So a unit
// takes a quarter of a CU -- 128 registers and 40 KiB of LDS at m <= 64 --
// and four units per CU fill each other's latencies; what is left is VALU
// throughput.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "kamera.h"
#include "kamera_form.h"
#include "kamera_launch.h"

namespace kamera {

namespace {

constexpr int kTriThreads = 256;
constexpr int kTriRows = 16;           // Delta rows per stage of the Gram product

// LDS, in floats.  The Z area holds the staged Gram tiles, then the reduction's
// vectors, then the eigenvectors of T in groups of 32 columns (row stride 33,
// so that lanes on consecutive columns and lanes on consecutive rows both fall
// on distinct banks; groups 32 banks apart), then blocks of 32 reflectors.
constexpr int kZLd = 33;
constexpr int kZGroup = 128 * kZLd + 32;
constexpr int kVLd = 132;              // staged reflector: 4-byte reads of 16 entries of 4 reflectors
                                       // (4 apart) fall on distinct banks
constexpr int kTriVec = 11 * 128 + 16; // a, b, beta, b2, b2s, lam, cs, r2[4]; lo, hi, fail

constexpr int tri_lds_floats(int zgroups) { return zgroups * kZGroup + kTriVec; }
static_assert(32 * (kVLd + 36) <= 2 * kZGroup, "a staged block of reflectors fits two groups of Z");
static_assert(2 * 3 * 128 * kTriRows * 2 <= 2 * kZGroup * 4, "the staged Gram parts fit two groups of Z");

__device__ __forceinline__ float* zcol(float* Z, int k) { return Z + (k >> 5) * kZGroup + (k & 31); }

// One eigenvector of T (diagonal a, subdiagonal b, b2[i] = b_i^2 and
// b2s[i] = b_{i-1}^2, both floored at FLT_MIN, 0 where b does not exist) for
// the eigenvalue lam by twisted factorisation, into z[i * ldz].  D- is kept
// in the column while D+ is recomputed where it is needed: the twist search
// runs D+ forward beside it, then D+ overwrites D- above the twist (where D-
// is no longer read) for the upward recurrence.  The pivot recurrences run in
// IEEE arithmetic as the Sturm counts do, from an infinite pivot beyond the
// first row; in the vector's recurrences a zero pivot is replaced by 1e-30.
// The twist is the rank-th least |gamma_i| (ties: lower index).  Every loop
// runs over aligned groups of four rows (d is a multiple of 4) with the
// shared operands read as 16-byte vectors, the next group loaded ahead.
__device__ __forceinline__ void twisted_vector(const float* __restrict__ a, const float* __restrict__ b,
                                               const float* __restrict__ b2, const float* __restrict__ b2s,
                                               float* __restrict__ z, int ldz, int d, float lam, int rank) {
  const float tiny = 1e-30f;
  const int ng = d >> 2;
  {                                            // backward pivots D-, bottom up
    float dmv = __builtin_inff();
    f32x4v an = ld4(a + d - 4), bn = ld4(b2 + d - 4);
    for (int g = ng - 1; g >= 0; --g) {
      const f32x4v ac = an, bc = bn;
      if (g > 0) {
        an = ld4(a + 4 * g - 4);
        bn = ld4(b2 + 4 * g - 4);
      }
#pragma unroll
      for (int u = 3; u >= 0; --u) {
        dmv = (ac[u] - lam) - bc[u] * __builtin_amdgcn_rcpf(dmv);
        z[(4 * g + u) * ldz] = dmv;
      }
    }
  }
  int r = 0;
  float prev = -1.f;
  int prev_i = -1;
  for (int s2 = 0; s2 <= rank; ++s2) {         // twist search, D+ top down beside D-
    float best = 3.4e38f, dpv = __builtin_inff();
    int bi = 0;
    f32x4v an = ld4(a), bn = ld4(b2s);
    float zn[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) zn[u] = z[u * ldz];
    for (int g = 0; g < ng; ++g) {
      const f32x4v ac = an, bc = bn;
      float zc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) zc[u] = zn[u];
      if (g + 1 < ng) {
        an = ld4(a + 4 * g + 4);
        bn = ld4(b2s + 4 * g + 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) zn[u] = z[(4 * g + 4 + u) * ldz];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = 4 * g + u;
        const float al = ac[u] - lam;
        dpv = al - bc[u] * __builtin_amdgcn_rcpf(dpv);
        const float gm = fabsf(dpv + zc[u] - al);
        // (bitwise, so that the selection compiles to selects, not branches)
        const bool take = ((gm > prev) | ((gm == prev) & (i > prev_i))) & (gm < best);
        best = take ? gm : best;
        bi = take ? i : bi;
      }
    }
    prev = best;
    prev_i = bi;
    r = bi;
  }
  {                                            // D+ above the twist
    float dpv = __builtin_inff();
    for (int g = 0; 4 * g < r; ++g) {
      const f32x4v ac = ld4(a + 4 * g), bc = ld4(b2s + 4 * g);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        dpv = (ac[u] - lam) - bc[u] * __builtin_amdgcn_rcpf(dpv);
        if (4 * g + u < r) z[(4 * g + u) * ldz] = dpv;
      }
    }
  }
  // the vector from the twist outwards; the pivots of a group are read
  // before any of its rows is overwritten, the next group's during this one.
  // Every row of a visited group is stored: rows outside the pass get back
  // the value just read (D- below the twist, the vector above it), so the
  // steps are selects and not branches.
  float up = 0.f, down = 0.f, x = 1.f;        // sums of squares (added as the two-lane form adds them)
  if (r > 0) {
    int g = (r - 1) >> 2;
    float qn[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) qn[u] = z[(4 * g + u) * ldz];
    f32x4v bn = ld4(b + 4 * g);
    for (; g >= 0; --g) {
      float q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) q[u] = qn[u];
      const f32x4v bc = bn;
      if (g > 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) qn[u] = z[(4 * g - 4 + u) * ldz];
        bn = ld4(b + 4 * g - 4);
      }
#pragma unroll
      for (int u = 3; u >= 0; --u) {
        const int i = 4 * g + u;
        const bool in = i < r;
        const float xn = -bc[u] * __builtin_amdgcn_rcpf(q[u] != 0.f ? q[u] : tiny) * x;
        x = in ? xn : x;
        up += in ? xn * xn : 0.f;
        z[i * ldz] = in ? xn : q[u];
      }
    }
  }
  z[r * ldz] = 1.f;
  x = 1.f;
  {
    int g = (r + 1) >> 2;
    float qn[4], bbn[4];
    auto load_group = [&](int gg) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = 4 * gg + u;
        qn[u] = z[i * ldz];
        bbn[u] = i > 0 ? b[i - 1] : 0.f;
      }
    };
    if (4 * g < d) load_group(g);
    for (; 4 * g < d; ++g) {
      float q[4], bb[4];                       // pivots D- and b_{i-1} of the group
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        q[u] = qn[u];
        bb[u] = bbn[u];
      }
      if (4 * g + 4 < d) load_group(g + 1);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = 4 * g + u;
        const bool in = i > r;
        const float xn = -bb[u] * __builtin_amdgcn_rcpf(q[u] != 0.f ? q[u] : tiny) * x;
        x = in ? xn : x;
        down += in ? xn * xn : 0.f;
        z[i * ldz] = in ? xn : q[u];
      }
    }
  }
  const float inv = 1.f / sqrtf(1.f + up + down);
  for (int g = 0; g < ng; ++g) {
#pragma unroll
    for (int u = 0; u < 4; ++u) z[(4 * g + u) * ldz] *= inv;
  }
}

// The same vector with two lanes per eigenvalue, on two waves, where Z has a
// spare column per eigenvalue (2 m <= ldz): the lane pair's pivots D- (into
// the vector's column zm) and D+ (into the spare column zp) run at once; the
// twist is then a scan over both stored columns; the vector above the twist
// (from D+, written into zm) and below it (from D-, in place) again run at
// once, each pass writing only its own rows.  Same recurrences, same
// arithmetic as twisted_vector.
__device__ __forceinline__ void tw_pivots(const float* __restrict__ a, const float* __restrict__ b2,
                                          const float* __restrict__ b2s, float* __restrict__ z, int ldz, int d,
                                          float lam, bool backward) {
  const int ng = d >> 2;
  float pv = __builtin_inff();
  if (backward) {                              // D-, bottom up
    f32x4v an = ld4(a + d - 4), bn = ld4(b2 + d - 4);
    for (int g = ng - 1; g >= 0; --g) {
      const f32x4v ac = an, bc = bn;
      if (g > 0) {
        an = ld4(a + 4 * g - 4);
        bn = ld4(b2 + 4 * g - 4);
      }
#pragma unroll
      for (int u = 3; u >= 0; --u) {
        pv = (ac[u] - lam) - bc[u] * __builtin_amdgcn_rcpf(pv);
        z[(4 * g + u) * ldz] = pv;
      }
    }
  } else {                                     // D+, top down
    f32x4v an = ld4(a), bn = ld4(b2s);
    for (int g = 0; g < ng; ++g) {
      const f32x4v ac = an, bc = bn;
      if (g + 1 < ng) {
        an = ld4(a + 4 * g + 4);
        bn = ld4(b2s + 4 * g + 4);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        pv = (ac[u] - lam) - bc[u] * __builtin_amdgcn_rcpf(pv);
        z[(4 * g + u) * ldz] = pv;
      }
    }
  }
}

// the twist from the stored pivots: the rank-th least |gamma_i|,
// gamma_i = D+_i + D-_i - (a_i - lam) (ties: lower index)
__device__ __forceinline__ int tw_twist(const float* __restrict__ a, const float* __restrict__ zm,
                                        const float* __restrict__ zp, int ldz, int d, float lam, int rank) {
  const int ng = d >> 2;
  float prev = -1.f;
  int prev_i = -1, r = 0;
  for (int s2 = 0; s2 <= rank; ++s2) {
    float best = 3.4e38f;
    int bi = 0;
    for (int g = 0; g < ng; ++g) {
      const f32x4v ac = ld4(a + 4 * g);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = 4 * g + u;
        const float al = ac[u] - lam;
        const float gm = fabsf(zp[i * ldz] + zm[i * ldz] - al);
        const bool take = ((gm > prev) | ((gm == prev) & (i > prev_i))) & (gm < best);
        best = take ? gm : best;
        bi = take ? i : bi;
      }
    }
    prev = best;
    prev_i = bi;
    r = bi;
  }
  return r;
}

// rows r-1 .. 0 of the vector (x_r = 1) from D+ (column zp) into column zm;
// returns their sum of squares
__device__ __forceinline__ float tw_up(const float* __restrict__ b, const float* __restrict__ zp,
                                       float* __restrict__ zm, int ldz, int r) {
  const float tiny = 1e-30f;
  float n2 = 0.f, x = 1.f;
  if (r > 0) {
    int g = (r - 1) >> 2;
    float qn[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) qn[u] = zp[(4 * g + u) * ldz];
    f32x4v bn = ld4(b + 4 * g);
    for (; g >= 0; --g) {
      float q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) q[u] = qn[u];
      const f32x4v bc = bn;
      if (g > 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) qn[u] = zp[(4 * g - 4 + u) * ldz];
        bn = ld4(b + 4 * g - 4);
      }
#pragma unroll
      for (int u = 3; u >= 0; --u) {
        const int i = 4 * g + u;
        const bool in = i < r;
        const float xn = -bc[u] * __builtin_amdgcn_rcpf(q[u] != 0.f ? q[u] : tiny) * x;
        x = in ? xn : x;
        n2 += in ? xn * xn : 0.f;
        if (in) zm[i * ldz] = xn;
      }
    }
  }
  return n2;
}

// rows r+1 .. d-1 of the vector (x_r = 1) from D- (column zm, in place);
// returns their sum of squares
__device__ __forceinline__ float tw_down(const float* __restrict__ b, float* __restrict__ zm, int ldz, int d,
                                         int r) {
  const float tiny = 1e-30f;
  float n2 = 0.f, x = 1.f;
  int g = (r + 1) >> 2;
  float qn[4], bbn[4];
  auto load_group = [&](int gg) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = 4 * gg + u;
      qn[u] = zm[i * ldz];
      bbn[u] = i > 0 ? b[i - 1] : 0.f;
    }
  };
  if (4 * g < d) load_group(g);
  for (; 4 * g < d; ++g) {
    float q[4], bb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      q[u] = qn[u];
      bb[u] = bbn[u];
    }
    if (4 * g + 4 < d) load_group(g + 1);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = 4 * g + u;
      const bool in = i > r;
      const float xn = -bb[u] * __builtin_amdgcn_rcpf(q[u] != 0.f ? q[u] : tiny) * x;
      x = in ? xn : x;
      n2 += in ? xn * xn : 0.f;
      if (in) zm[i * ldz] = xn;
    }
  }
  return n2;
}

// bf16 offset of rows 8 p .. 8 p + 7 of column c in a staged Gram part:
// columns of kTriRows rows, their two 16-byte pieces swapped so that 32 lanes
// reading one piece of 32 consecutive columns (16-byte reads are served per
// half wave over 512 bytes of banks) and 16 lanes storing one piece of
// consecutive columns (stores: per quarter wave over 256 bytes) touch distinct
// banks
__device__ __forceinline__ int tri_slot(int c, int p) { return c * kTriRows + 8 * (p ^ (((c >> 3) ^ (c >> 4)) & 1)); }

// One deficit through a buffer descriptor: rows past n and lanes without a
// column read zeros by its bounds check, and a row's address is one scalar
// addition (64-bit row pointers took 123 scalar instructions a stage).  For
// rows that do not overlap and a unit's rows within 2^31 bytes.
struct TriRows {
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t col;            // byte offset of the lane's column (past the end: none)
  int32_t row;             // bytes of a row
  int32_t end;             // the descriptor's bytes: a row's offset stops there, where no lane is in range

  __device__ __forceinline__ void load8(int i0, float (&x)[8]) const {
    int32_t at = i0 * row;
#pragma unroll
    for (int e = 0; e < 8; ++e, at += row)
      x[e] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)col, min(at, end), 0));
  }
};

// The general form, also the mean of an orbit's members: 64-bit row pointers.
// A row past n is read at row n - 1, so that every call issues the same loads
// (a load behind a branch would make the compiler wait for all the loads in
// flight).  Orbit members are read two at a time, all their loads issued before
// the sums, which keep the members' order.
struct TriOrbit {
  const FormParams& P;
  const float* delta;
  uint32_t j;

  __device__ __forceinline__ void load8(int i0, float (&x)[8]) const {
    const int64_t s3 = P.delta_s[3];
    const int n = P.n_tokens;
    const float* row[8];
    row[0] = delta + (int64_t)min(i0, n - 1) * s3;
#pragma unroll
    for (int e = 1; e < 8; ++e) row[e] = row[e - 1] + (i0 + e < n ? s3 : 0);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = row[e][j];
    for (int o = 1; o < P.n_orbit; o += 2) {
      const bool two = o + 1 < P.n_orbit;
      const int64_t o1 = (int64_t)o * P.orbit_s, o2 = two ? o1 + P.orbit_s : o1;
      float y[8], z[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        y[e] = (row[e] + o1)[j];
        z[e] = (row[e] + o2)[j];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = two ? (x[e] + y[e]) + z[e] : x[e] + y[e];
    }
    if (P.n_orbit > 1) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] *= P.inv_orbit;
    }
  }
};

// ---- 1. G = Delta^T Delta: tiles (I, J), I < NB, into acc ----
// src: TriRows (ZEROS: it reads zeros past n rows or d columns) or TriOrbit.
// Stages of S x kTriRows = 16 S rows (S MFMA k-steps) in two LDS buffers, one
// barrier each: thread (sg, c) splits rows 8 sg .. 8 sg + 7 of column c of
// stage s + 1 into three bf16 parts while stage s is multiplied; its loads are
// issued kTriAhead stages before.  One wave per SIMD issues the split, the
// products and the waits for LDS and memory in turn; with four units on the CU
// they overlap, and for a unit alone there S = 2 brings a second wave per SIMD:
// group g of four waves forms tiles g NB / S .. (g + 1) NB / S - 1 of each column,
// from all rows, so that a tile is the same sum in the same order whatever S is.
// (With the rows split between the groups, and four products a tile for six by
// adding the transpose, a call of 8 units of 1024 x 128 took 192 us for 200, but
// a unit's patch then depended on how many shared its call.)
constexpr int kTriAhead = 3;
constexpr int kTriGramBytes = 2 * 3 * 128 * kTriRows * 2;   // two staged buffers of kTriRows rows

template <int NB, int S, bool ZEROS, typename SRC>
__device__ __forceinline__ void tri_gram(const SRC& src, int n, int d, int J, int g, uint16_t* Tb,
                                         f32x16v (&acc)[NB / S]) {
  constexpr int kPart = 32 * NB * kTriRows, NT = NB / S;
  const int tid = threadIdx.x, lane = tid & 63;
  const int sc = tid & 127, sg = __builtin_amdgcn_readfirstlane(tid >> 7) & (2 * S - 1);
  auto row0 = [&](int s) { return kTriRows * S * s + 8 * sg; };   // first row of the thread's piece of stage s
  const bool cin = sc < d;
#pragma unroll
  for (int u = 0; u < NT; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[u][r] = 0.f;
  const int ns = (n + kTriRows * S - 1) / (kTriRows * S);
  float x[kTriAhead][8];
#pragma unroll
  for (int a = 0; a < kTriAhead; ++a) src.load8(row0(a), x[a]);
  uint16_t* const mine = Tb + (sg >> 1) * 3 * kPart + tri_slot(sc, sg & 1);
  auto put = [&](float (&y)[8], int s, int buf) {
    if (!ZEROS && (kTriRows * S * (s + 1) > n || 32 * NB > d)) {   // zeros past n rows or d columns
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = row0(s) + e < n && cin ? y[e] : 0.f;
    }
    u32x4v hi, mid, lo;
    split3_bf16x8(y, hi, mid, lo);
    uint16_t* q = mine + buf * S * 3 * kPart;
    if (NB == 4 || sc < 32 * NB) {
      *reinterpret_cast<u32x4v*>(q) = hi;
      *reinterpret_cast<u32x4v*>(q + kPart) = mid;
      *reinterpret_cast<u32x4v*>(q + 2 * kPart) = lo;
    }
  };
  put(x[0], 0, 0);
  src.load8(row0(kTriAhead), x[0]);
  // stage s: y holds stage s + 1, split into the other buffer between the
  // products (past the last stage: zeros, never read), then takes the loads of
  // stage s + 1 + kTriAhead.  The buffer it writes was read in stage s - 1, before
  // the barrier.
  auto stage = [&](int s, float (&y)[8]) {
    const int buf = s & 1;
    __syncthreads();
    const int p = lane >> 5, c = lane & 31;
    if (NB == 4 || J < NB) {
#pragma unroll
      for (int k = 0; k < S; ++k) {
        const uint16_t* const Ts = Tb + (buf * S + k) * 3 * kPart;
        auto part = [&](int q, int col) { return *reinterpret_cast<const bf16x8v*>(Ts + q * kPart + tri_slot(col + c, p)); };
        bf16x8v b[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) b[q] = part(q, 32 * J);
        // the tiles' chains of products alternate (a product waits about twice its
        // own 32 cycles for the one before it in its chain): lo hi; mid mid, mid
        // hi; hi lo, hi mid, hi hi, one part of A at a time
#pragma unroll
        for (int q = 2; q >= 0; --q) {
          bf16x8v av[NT];
#pragma unroll
          for (int u = 0; u < NT; ++u) av[u] = part(q, 32 * (NT * g + u));
#pragma unroll
          for (int t = 2 - q; t >= 0; --t)
#pragma unroll
            for (int u = 0; u < NT; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[u], b[t], acc[u], 0, 0, 0);
        }
        if (k == 0 && NB == 4) put(y, s + 1, buf ^ 1);
      }
    }
    if (NB < 4) put(y, s + 1, buf ^ 1);
    src.load8(row0(s + 1 + kTriAhead), y);
    __builtin_amdgcn_sched_barrier(0);
  };
  // (whole groups of kTriAhead stages, the last ones of zeros: no branch between them)
  for (int s = 0; s < ns; s += kTriAhead) {
#pragma unroll
    for (int a = 0; a < kTriAhead; ++a) stage(s + a, x[(a + 1) % kTriAhead]);
  }
}

// sum over the wave, the same on every lane: three DPP adds per 8 lanes, the
// other half of each row of 16, then row_bcast:15 and row_bcast:31 carry the
// row sums into lane 63 (-0 is the sum's identity, so each step is one add)
__device__ __forceinline__ float tri_wave_sum(float v) {
  constexpr int kZero = (int)0x80000000;
  v = sum8(v);
  v += dpp_f<0x140>(v);
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(kZero, __builtin_bit_cast(int, v), 0x142, 0xa, 0xf, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(kZero, __builtin_bit_cast(int, v), 0x143, 0xc, 0xf, false));
  return lane_f(v, 63);
}

// swaps a's upper 32 lanes with b's lower 32: a = [a.lo | b.lo], b = [a.hi | b.hi]
__device__ __forceinline__ void half_swap(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// ---- 2. Householder reduction T = Q^T G Q, Q = H_0 ... H_{d-3},
// H_j = I - beta_j v_j v_j^T ----
// Step j takes row j right of the diagonal, x = A[j, j+1..]: alpha =
// -sign(x_0) |x|, v = x - alpha e_0, beta = 2 / v^T v; the trailing block
// becomes A - v w^T - w v^T with p = beta A v, w = p - (beta / 2)(p^T v) v.
// alpha is T's subdiagonal b_j, A[j][j] its diagonal a_j.
// A step has one barrier.  Before it each wave takes p = A v_j on its own 32
// columns (fp32 on the VALU, v_j broadcast from LDS) and, by symmetry, its
// columns of row j + 1; both go through LDS.  After it every wave still in the
// trailing block forms w_j for itself, starts the rank-2 update of its tiles
// (one v_mfma_f32_32x32x2_f32 each: K = 2 is exactly the two outer products,
// and its operands are lane-per-index vectors, a permlane32 swap each), and
// while the matrix pipe runs forms the updated row j + 1 and the next
// reflector, so nothing waits for an owner.
// No column is touched once it is reduced (v and w are zero there); after the
// last step of its block its wave puts v_j in place of x_j, for the
// back-transformation.  It has to be the step's own v: the matrix is symmetric to
// rounding only (the six products of a tile and of its transpose are added in
// different orders, as are the two outer products of an update), so where |x_j|
// is itself rounding the column holds another vector than the row that v_j came
// from, and a Q made of such vectors is not the one that T came from.
// alpha, v's first entry and beta of the reflector of (x0, x) with |x|^2 = sq.
// (hardware square root and reciprocal, 1 ulp each: beta is formed from the v
// that is kept, so H is orthogonal to rounding; sq = 0: already reduced, H = I)
__device__ __forceinline__ void tri_scales(float x0, float sq, float& alpha, float& v0, float& beta) {
  const float nrm = __builtin_amdgcn_sqrtf(fmaf(x0, x0, sq));
  alpha = sq != 0.f ? (x0 >= 0.f ? -nrm : nrm) : x0;
  v0 = x0 - alpha;
  beta = sq != 0.f ? 2.f * __builtin_amdgcn_rcpf(fmaf(v0, v0, sq)) : 0.f;
}

template <int V>
struct IntC {
  static constexpr int value = V;
};

struct TriVec {
  float v0, v1;          // v_j, entries lane and 64 + lane (v0 unused once j + 1 >= 64)
  float beta;
};

// entry i of a vector held as (lane, 64 + lane)
__device__ __forceinline__ float tri_at(float x0, float x1, int i) { return lane_f(i < 64 ? x0 : x1, i & 63); }

// scr: [2] x (p[128], row[128]) of alternate steps; the last 32 steps' v, written
// by the wave that runs every step, in rows of kVLd; a copy of the last one for
// each of the others, so that none waits for it
constexpr int kTriScr = 512 + 32 * kVLd + 3 * 128;
static_assert(kTriScr <= 2 * kZGroup, "the reduction's vectors fit two groups of Z");

// The reflector of column jn <= d - 2 from its updated row (r0, r1), x0 =
// row[jn + 1]; the wave's v_jn goes to its own vbuf, alpha and beta to s_b
// and s_beta.  mid1 and mid2 are run
// inside the dependent chain (work for the matrix pipe, which issues in order
// with it).
template <int NB, typename F1, typename F2>
__device__ __forceinline__ void tri_reflect(TriVec& S, int jn, float r0, float r1, float x0, float* vbuf, float* s_b,
                                            float* s_beta, int J, F1 mid1, F2 mid2) {
  const int lane = threadIdx.x & 63;
  const float q0 = lane > jn + 1 ? r0 : 0.f;
  const float q1 = lane + 64 > jn + 1 ? r1 : 0.f;
  const float part = NB > 2 ? fmaf(q0, q0, q1 * q1) : q0 * q0;
  mid1();
  const float sq = tri_wave_sum(part);
  float v0, alpha;
  tri_scales(x0, sq, alpha, v0, S.beta);
  mid2();
  if (J == NB - 1 && lane == 0) {              // (the wave that runs every step)
    s_b[jn] = alpha;
    s_beta[jn] = S.beta;
  }
  S.v0 = lane == jn + 1 ? v0 : q0;
  vbuf[lane] = S.v0;
  if (NB > 2) {
    S.v1 = lane + 64 == jn + 1 ? v0 : q1;
    vbuf[64 + lane] = S.v1;
  }
}

// Steps 0 .. d - 3.  A wave runs those of its own and earlier blocks, then
// clears its p in both buffers and only keeps the barriers.
template <int NB>
__device__ __forceinline__ void tri_steps(f32x16v (&acc)[NB], TriVec& S, int J, int d, float* scr, float* s_b,
                                          float* s_beta) {
  const int lane = threadIdx.x & 63;
  const int col = 32 * J + (lane & 31);
  float* const ring = scr + 512;
  float* const vbase = J == NB - 1 ? ring : ring + 32 * kVLd + 128 * J;
  const int vmask = J == NB - 1 ? 31 : 0;
  const int j_own = J < NB ? min(32 * J + 31, d - 2) : 0;
  for (int j = 0; j < j_own; ++j) {
    float* const pb = scr + 256 * (j & 1);
    const int ib = (j + 1) >> 5;               // first block of the trailing rows
    const float* const vrow = vbase + kVLd * (j & vmask) + 4 * (lane >> 5);
    {
      float s[4] = {0.f, 0.f, 0.f, 0.f};
      // row j + 1 within its block: an element of one lane half, which writes
      // it while the other half writes p
      const int rr = (j + 1) & 31, re = ((rr >> 3) << 2) | (rr & 3);
      float row = 0.f;
      f32x4v vn[4];                            // a block's share of v, the next block's read ahead
#pragma unroll
      for (int g = 0; g < 4; ++g) vn[g] = ld4(vrow + 8 * g);
#pragma unroll
      for (int I = 0; I < NB; ++I) {
        f32x4v v[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          v[g] = vn[g];
          if (I + 1 < NB) vn[g] = ld4(vrow + 32 * (I + 1) + 8 * g);
        }
        if (I >= ib) {
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int u = 0; u < 4; ++u) s[u] = fmaf(acc[I][4 * g + u], v[g][u], s[u]);
          if (I == ib) row = acc[I][re];
        }
      }
      float lo = (s[0] + s[1]) + (s[2] + s[3]), hi = lo;
      half_swap(lo, hi);
      const float p = col > j ? lo + hi : 0.f;
      const bool has_row = (lane >> 5) == ((rr >> 2) & 1);
      pb[col + (has_row ? 128 : 0)] = has_row ? row : p;
    }
    __syncthreads();
    const float p0 = pb[lane];
    float r0 = pb[128 + lane];
    float p1 = 0.f, r1 = 0.f;
    if (NB > 2) {
      p1 = pb[64 + lane];
      r1 = pb[192 + lane];
    }
    // (beta p first: with |x| ~ g, beta is of the size of g^-2 and p^T v of g^3, and
    // beta^2 or p^T v would leave the range of fp32 at g below 1e-9 or above 1e12)
    const float q0 = S.beta * p0, q1 = S.beta * p1;
    const float K = 0.5f * S.beta * tri_wave_sum(NB > 2 ? fmaf(q0, S.v0, q1 * S.v1) : q0 * S.v0);
    const float w0 = fmaf(-K, S.v0, q0), w1 = fmaf(-K, S.v1, q1);
    // the update's operands: lanes < 32 v (w for B), others w (v), of a block
    float b0 = J >= 2 ? w1 : w0, b1 = J >= 2 ? S.v1 : S.v0;
    half_swap(b0, b1);
    const float bop = -((J & 1) ? b1 : b0);
    float a[4] = {S.v0, w0, S.v1, w1};
    half_swap(a[0], a[1]);
    if (NB > 2) half_swap(a[2], a[3]);
    // tile I's update; they are issued one at a time inside the chains below,
    // as an MFMA holds up what follows it until the one before is through
    auto update = [&](auto ic) {
      constexpr int I = decltype(ic)::value;
      if constexpr (I >= 0 && I < NB) {
        if (I >= ib) acc[I] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[I], bop, acc[I], 0, 0, 0);
      }
    };
    update(IntC<NB - 1>{});
    const float vj = tri_at(S.v0, S.v1, j + 1), wj = tri_at(w0, w1, j + 1);
    r0 = fmaf(-vj, w0, fmaf(-wj, S.v0, r0));
    if (NB > 2) r1 = fmaf(-vj, w1, fmaf(-wj, S.v1, r1));
    tri_reflect<NB>(S, j + 1, r0, r1, tri_at(r0, r1, j + 2), vbase + kVLd * ((j + 1) & vmask), s_b, s_beta,
                    J, [&] { update(IntC<NB - 2>{}); }, [&] { update(IntC<NB - 3>{}); });
    update(IntC<NB - 4>{});
  }
  if (J < NB) {
    // the reflectors into the wave's columns, below the diagonal, before the
    // ring's rows are taken again (after the next barrier; the last of them is
    // being written, so the wave reads its own copy of that)
    const int c = lane & 31;
    const float* const v = (c == 31 && J < NB - 1 ? vbase : ring + kVLd * c) + 4 * (lane >> 5);
#pragma unroll
    for (int I = 0; I < NB; ++I)
      if (I >= J) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4v y = ld4(v + 32 * I + 8 * g);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = acc[I][4 * g + e];
            acc[I][4 * g + e] = 32 * I + 8 * g + 4 * (lane >> 5) + e > col ? y[e] : x;
          }
        }
      }
  }
  for (int j = j_own; j < d - 2; ++j) {
    if (J < NB && j < j_own + 2 && lane < 32) scr[256 * (j & 1) + col] = 0.f;
    __syncthreads();
  }
}

// Leaves T's diagonal and subdiagonal in s_a and s_b, the reflectors' scales in
// s_beta (zero past the last) and the reflectors in acc's columns, below the diagonal.
template <int NB>
__device__ __forceinline__ void tri_reduce(f32x16v (&acc)[NB], int J, int d, float* scr, float* s_a, float* s_b,
                                           float* s_beta) {
  const int lane = threadIdx.x & 63;
  TriVec S = {0.f, 0.f, 0.f};
  float* const rb = scr + 256 + 128;           // row 0 takes the buffer that step 0 does not
  __syncthreads();                             // the staged Gram tiles are consumed
  for (int i = threadIdx.x; i < 512; i += kTriThreads) scr[i] = 0.f;
  if (threadIdx.x < 128) s_beta[threadIdx.x] = 0.f;
  __syncthreads();
  if (J < NB && lane < 32) rb[32 * J + lane] = acc[0][0];
  __syncthreads();
  if (J < NB)
    tri_reflect<NB>(S, 0, rb[lane], rb[64 + lane], lane_f(rb[lane], 1),
                    scr + 512 + (J == NB - 1 ? 0 : 32 * kVLd + 128 * J), s_b, s_beta, J, [] {}, [] {});
  tri_steps<NB>(acc, S, J, d, scr, s_b, s_beta);
  __syncthreads();                             // the last step's vectors are read
  if (J < NB) {
    // a_j = A[j][j] of this lane's column
    const int c = lane & 31, h4 = 4 * (lane >> 5), j = 32 * J + c;
    float aj = 0.f;
#pragma unroll
    for (int I = 0; I < NB; ++I)
      if (I == J) {
#pragma unroll
        for (int r = 0; r < 16; ++r) aj += 8 * (r >> 2) + (r & 3) + h4 == c ? acc[I][r] : 0.f;
      }
    float aj2 = aj;
    half_swap(aj, aj2);
    if (lane < 32 && j < d) s_a[j] = aj + aj2;
  }
}

// ---- 2b. compact WY form of the reflectors ----
// The 32 reflectors of block J multiply to I - V T V^T with
// T^-1 = diag(1 / beta) + the strict upper triangle of S = V^T V.  Wave J
// clears the columns past the last reflector, takes S on MFMA (operand A and B
// are both the tile's own registers) and solves for T's columns, one per lane.
// -T goes into the diagonal tile's rows i <= j, where V has no entries.
// sw: 32 x kSLd floats private to the wave.
constexpr int kSLd = 36;

template <int NB>
__device__ __forceinline__ void tri_wy(f32x16v (&acc)[NB], int J, int d, float* sw, const float* s_beta) {
  if (J >= NB) return;
  const int lane = threadIdx.x & 63, c = lane & 31, h4 = 4 * (lane >> 5);
  const int j = 32 * J + c;                    // this lane's reflector
  const bool real = j < d - 2;
  f32x16v S, diag;
#pragma unroll
  for (int r = 0; r < 16; ++r) S[r] = diag[r] = 0.f;
#pragma unroll
  for (int I = 0; I < NB; ++I) {
    if (I < J) continue;
    if (I == J) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int f = 8 * (r >> 2) + (r & 3) + h4;
        const float x = f > c && real ? acc[I][r] : 0.f;
        diag[r] = x;
        S = __builtin_amdgcn_mfma_f32_32x32x2f32(x, x, S, 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc[I][r] = real ? acc[I][r] : 0.f;
        S = __builtin_amdgcn_mfma_f32_32x32x2f32(acc[I][r], acc[I][r], S, 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<f32x4v*>(sw + c * kSLd + 8 * g + h4) = (f32x4v){S[4 * g], S[4 * g + 1], S[4 * g + 2], S[4 * g + 3]};
  __builtin_amdgcn_wave_barrier();             // (a wave's LDS accesses are performed in program order)
  // t[i] = -T[i][c] = beta_i (-(i == c) - sum_{k > i} S[i][k] t[k]); zero for i > c by itself
  float t[32];
#pragma unroll
  for (int i = 31; i >= 0; --i) {
    float s0 = i == c ? 1.f : 0.f, s1 = 0.f;
#pragma unroll
    for (int k4 = (i + 1) & ~3; k4 < 32; k4 += 4) {
      const f32x4v sr = ld4(sw + i * kSLd + k4);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k4 + u > i) {
          if (u & 1) s1 = fmaf(sr[u], t[k4 + u], s1);
          else s0 = fmaf(sr[u], t[k4 + u], s0);
        }
    }
    t[i] = -s_beta[32 * J + i] * (s0 + s1);    // (beta is zero past the last reflector)
    asm volatile("" : "+v"(t[i])::"memory");   // (else every row of S is read first, into scratch)
  }
#pragma unroll
  for (int I = 0; I < NB; ++I)
    if (I == J) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int f0 = 8 * (r >> 2) + (r & 3);
        const float ta = t[f0], tb = t[f0 + 4];
        const float tt = lane < 32 ? ta : tb;
        acc[I][r] = f0 + h4 > c ? diag[r] : tt;
      }
    }
}

// ---- 3a. multisection on Sturm counts ----
// The number of eigenvalues of T below x is the number of sign changes in
// p_0 = 1, p_1, .., p_d with p_{i+1} = (a_i - x) p_i - b_{i-1}^2 p_{i-1} (the
// characteristic polynomials of T's leading blocks).  T is scaled by a power
// of two to |T| <= 1 and b^2 floored at 1e-18 (1e-9 of |T|, below its rounding);
// every four rows the pair is scaled back to about 1, exactly.  The division
// form of the recurrence (pivots p_{i+1} / p_i) spends four issue slots a row
// on the reciprocal: 32 us a unit alone on its CU at rank 64, against 12 us.
// Four rows cost the pair a factor of about 1e-36 at worst (two floored b^2, or
// four pivots of 1e-9); `low` keeps the smallest value scaled back, and a unit
// where it falls below 2^-122 is left to Jacobi.
__device__ __forceinline__ int sturm_count(const float* s_as, const float* s_bs, float x, int d, float& low) {
  float p1 = 1.f, p0 = 0.f;
  int cnt = 0;
  uint32_t bits = 0;
  f32x4v an = ld4(s_as), bn = ld4(s_bs);
  for (int i = 0; i < d; i += 16) {
    // (rows past d, up to the next multiple of 16: a = 4, b^2 = 0 keep the sign)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4v ac = an, bc = bn;
      const int next = (i + 4 * g + 4) & 127;
      an = ld4(s_as + next);
      bn = ld4(s_bs + next);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float p = fmaf(ac[u] - x, p1, -(bc[u] * p0));
        p0 = p1;
        p1 = p;
        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(p), 31);
      }
      const float mx = fmaxf(fabsf(p1), fabsf(p0));
      low = fminf(low, mx);
      // times the power of two that brings mx to [2, 4)
      const float sc = __uint_as_float(0x7f800000u - (__float_as_uint(mx) & 0x7f800000u));
      p1 *= sc;
      p0 *= sc;
    }
    cnt += __popc((bits ^ (bits >> 1)) & 0xffffu);
  }
  return cnt;
}

// First all 256 threads count at 256 points of the whole interval, which
// brackets every eigenvalue to 1/257 of it, then GL lanes an eigenvalue divide
// its bracket by GL + 1 a round: width / (257 * 5^8), 257 * 9^6 or 257 * 3^12,
// all below fp32 rounding of |T|.  s_as, s_bs: T scaled; s_nb: 128 ints.
template <int GL, int ROUNDS>
__device__ __forceinline__ void multisect(const float* s_as, const float* s_bs, float* s_lam, int* s_cnt, int* s_nb,
                                          float glo, float ghi, int exp2, int d, int m, int* s_fail) {
  const int tid = threadIdx.x, lane = tid & 63;
  float low = 1.f;
  constexpr float kFirst = 1.f / 257.f;
  {
    const int c = sturm_count(s_as, s_bs, glo + (ghi - glo) * (float)(tid + 1) * kFirst, d, low);
    s_cnt[tid] = c;
    __syncthreads();
    // the points with at most q eigenvalues below: q + 1 of them lie below the next
    const int c0 = tid > 0 ? s_cnt[tid - 1] : 0;
    for (int q = c0; q < c; ++q) s_nb[q] = tid;
    if (tid == 255)
      for (int q = c; q < d; ++q) s_nb[q] = 256;
    __syncthreads();
  }
  if (tid < GL * m) {
    const int k = tid / GL, t = tid % GL;
    const int q = d - 1 - k;                   // ascending index of the k-th largest
    constexpr float kStep = 1.f / (GL + 1);
    const int n0 = s_nb[q];
    float lo = n0 > 0 ? glo + (ghi - glo) * (float)n0 * kFirst : glo;
    float hi = n0 < 256 ? glo + (ghi - glo) * (float)(n0 + 1) * kFirst : ghi;
    for (int it = 0; it < ROUNDS; ++it) {
      const float w = hi - lo;
      const int cnt = sturm_count(s_as, s_bs, lo + w * (float)(t + 1) * kStep, d, low);
      // the points at or below the eigenvalue: a prefix of the group's lanes
      const uint64_t bal = __ballot(cnt <= q);
      const int nb = __popc((uint32_t)(bal >> (lane & ~(GL - 1))) & ((1u << GL) - 1u));
      const float nlo = nb > 0 ? lo + w * (float)nb * kStep : lo;
      const float nhi = nb < GL ? lo + w * (float)(nb + 1) * kStep : hi;
      lo = nlo;
      hi = fmaxf(nhi, nlo);
    }
    if (t == 0) s_lam[k] = __builtin_amdgcn_ldexpf(0.5f * (lo + hi), exp2);
  }
  if (!(low >= 0x1p-122f)) *s_fail = 1;
}

// ---- 4. V_m = Q Z ----
// A wave takes 16 columns of Z with all their rows in registers, as 16x16 MFMA
// accumulators: lane (kg, t) = (l / 16, l % 16), element r of zt[q] is row
// 16 q + 4 kg + r of column t.  Per block of 32 reflectors (last block first),
// Z -= V T (V^T Z): C = V^T Z, Y = -T C, Z += V Y, three chains of
// v_mfma_f32_16x16x4_f32 whose B operands are accumulators of the step before
// (element r as B holds exactly rows 4 kg + r); A comes from LDS, where the
// block's wave has staged V [reflector][row] and -T [row][column].
template <int NB, int B>
__device__ __forceinline__ void tri_apply(const float* V, const float* T, f32x4v (&zt)[2 * NB]) {
  const int lane = threadIdx.x & 63, t = lane & 15, k4 = 4 * (lane >> 4);
  f32x4v C[2], Y[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) C[u] = Y[u] = (f32x4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 2 * B; q < 2 * NB; ++q) {
    const f32x4v a0 = ld4(V + t * kVLd + 16 * q + k4), a1 = ld4(V + (16 + t) * kVLd + 16 * q + k4);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      C[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[r], zt[q][r], C[0], 0, 0, 0);
      C[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[r], zt[q][r], C[1], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)                  // T is upper triangular: its (1, 0) tile is zero
#pragma unroll
    for (int u = i; u < 2; ++u) {
      const f32x4v a = ld4(T + (16 * i + t) * kSLd + 16 * u + k4);
#pragma unroll
      for (int r = 0; r < 4; ++r) Y[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], C[u][r], Y[i], 0, 0, 0);
    }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 2 * B; q < 2 * NB; ++q)
        zt[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(V[(16 * u + k4 + r) * kVLd + 16 * q + t], Y[u][r], zt[q], 0, 0, 0);
}

extern __shared__ __align__(16) float tri_lds[];

// Brings the other groups' tiles to group 0, through X: (S - 1) NB / S tiles of
// 4 x 256 lanes of 16 bytes.
template <int NB, int S>
__device__ __forceinline__ void tri_gram_join(const f32x16v (&part)[NB / S], f32x16v (&acc)[NB], int g, float* X) {
  constexpr int NT = NB / S;
  const int t = threadIdx.x & (kTriThreads - 1);
  auto slot = [&](int I, int q) { return X + (((I - NT) * 4 + q) * kTriThreads + t) * 4; };
  __syncthreads();                             // the staged tiles are read
  if (g > 0) {
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4v*>(slot(NT * g + u, q)) =
            (f32x4v){part[u][4 * q], part[u][4 * q + 1], part[u][4 * q + 2], part[u][4 * q + 3]};
  }
  __syncthreads();
  if (g == 0) {
#pragma unroll
    for (int u = 0; u < NT; ++u) acc[u] = part[u];
#pragma unroll
    for (int I = NT; I < NB; ++I)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4v y = ld4(slot(I, q));
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[I][4 * q + e] = y[e];
      }
  }
}

// S groups of four waves form G, each a share of the tiles; the first goes on
// alone.  A unit alone on its CU leaves the Gram stages to four waves' chains of
// waits otherwise (more units on it fill each other's), and at S = 2 a wave may
// hold 256 registers: 168, where 128 spill 146 values.
// P.z_groups: groups of 32 columns in the Z area; twice those of m let two lanes
// take an eigenvector
template <int NB, int S>
__global__ __launch_bounds__(kTriThreads * S, S > 1 ? 2 : 4) void form_tri_kernel(const FormParams /*by value, read in place*/) {
  const FormParams& P = *static_cast<const FormParams*>((const void*)__builtin_amdgcn_kernarg_segment_ptr());
  const int unit = blockIdx.x;
  const int h = unit % P.n_heads;
  const int l = (unit / P.n_heads) % P.n_layers;
  const int c = unit / (P.n_heads * P.n_layers);
  const int d = P.dim, m = P.m;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // The role of a wave rotates with the unit: the last column blocks work
  // longest in the reduction, and the units that share a CU should not put
  // them on the same SIMD.
  const int J = (wave + (unit >> 3) + (unit >> 8)) & 3;
  const int group = wave >> 2;                 // (0 where S is 1)
  float* const Z = tri_lds;
  float* const sv = Z + P.z_groups * kZGroup;
  float* const s_a = sv;                       // T's diagonal
  float* const s_b = sv + 128;                 // T's subdiagonal
  float* const s_beta = sv + 2 * 128;          // reflector scales
  float* const s_b2 = sv + 3 * 128;            // b_i^2
  float* const s_b2s = sv + 4 * 128;           // b_{i-1}^2 (0 at i = 0)
  float* const s_lam = sv + 5 * 128;           // eigenvalues, descending
  int* const s_cs = reinterpret_cast<int*>(sv + 6 * 128);   // run start of each eigenvalue's cluster
  float* const s_r2 = sv + 7 * 128;            // [4][128] partial sums
  float* const s_misc = sv + 11 * 128;         // Gershgorin lo, hi
  int* const s_fail = reinterpret_cast<int*>(s_misc + 2);

  f32x16v acc[NB];
  {
    const float* const delta =
        P.delta + (int64_t)c * P.delta_s[0] + (int64_t)l * P.delta_s[1] + (int64_t)h * P.delta_s[2];
    uint16_t* const Tb = reinterpret_cast<uint16_t*>(Z);
    const int g = S > 1 ? group : 0;
    const int sc = tid & 127;
    f32x16v part[NB / S];
    if (P.n_orbit == 1 && P.unit_bytes > 0) {
      const TriRows src = {__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(delta), (short)0, P.unit_bytes, 0x00020000),
                           sc < d ? 4u * (uint32_t)sc : 0x7ffffff0u, 4 * (int32_t)P.delta_s[3], P.unit_bytes};
      tri_gram<NB, S, true>(src, P.n_tokens, d, J, g, Tb, part);
    } else {
      const TriOrbit src = {P, delta, (uint32_t)min(sc, d - 1)};
      tri_gram<NB, S, false>(src, P.n_tokens, d, J, g, Tb, part);
    }
    if constexpr (S > 1) {
      tri_gram_join<NB, S>(part, acc, g, Z);
      if (g > 0) return;                       // (a barrier waits for the waves that are left)
    } else {
#pragma unroll
      for (int I = 0; I < NB; ++I) acc[I] = part[I];
    }
  }
  tri_reduce<NB>(acc, J, d, Z, s_a, s_b, s_beta);
  __syncthreads();
  tri_wy<NB>(acc, J, d, Z + 32 * kSLd * J, s_beta);

  // ---- 3. the m largest eigenpairs of T ----
  if (wave == 0) {                             // Gershgorin interval and b^2
    float lo = 3.4e38f, hi = -3.4e38f;
    bool finite = true;
    for (int i = lane; i < d; i += 64) {
      const float bl = i > 0 ? s_b[i - 1] : 0.f, br = i < d - 1 ? s_b[i] : 0.f;
      const float r = fabsf(bl) + fabsf(br);
      lo = fminf(lo, s_a[i] - r);
      hi = fmaxf(hi, s_a[i] + r);
      finite = finite && fabsf(s_a[i]) + r <= 3.4e38f;
      s_b2[i] = i < d - 1 ? fmaxf(br * br, 1.17549435e-38f) : 0.f;
      s_b2s[i] = i > 0 ? fmaxf(bl * bl, 1.17549435e-38f) : 0.f;
    }
    for (int o = 32; o > 0; o >>= 1) {
      lo = fminf(lo, __shfl_xor(lo, o, 64));
      hi = fmaxf(hi, __shfl_xor(hi, o, 64));
    }
    const bool ok = __all(finite);
    if (lane == 0) {
      s_misc[0] = lo;
      s_misc[1] = hi;
      *s_fail = ok && (lo != 0.f || hi != 0.f) ? 0 : 1;
    }
  }
  // Leaves the unit to Jacobi (the same on every thread), as soon as it is known:
  // the vectors of a multiple eigenvalue search the twist once a member, and
  // eigenvalues that are not numbers, or of T = 0, count as one such (a unit of 64
  // columns, rank 32, whose T is not finite: 237 us, 80 for an ordinary one).
  auto failed = [&]() -> bool {
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(*s_fail) == 0) return false;
    if (tid == 0) P.W[(int64_t)c * P.w_s[0] + (int64_t)l * P.w_s[1] + (int64_t)h * P.w_s[2]] = kFormFailMark;
    return true;
  };
  if (failed()) return;
  const float glo = s_misc[0], ghi = s_misc[1];
  const float tnorm = fmaxf(fabsf(glo), fabsf(ghi));   // |T| bound
  {
    // T scaled to |T| <= 1, in the space of the partial sums
    float* const s_as = s_r2, * const s_bs = s_r2 + 128;
    int* const s_cnt = reinterpret_cast<int*>(s_r2 + 256);
    const int e = __builtin_amdgcn_frexp_expf(tnorm);
    if (tid < 128) {
      s_as[tid] = tid < d ? __builtin_amdgcn_ldexpf(s_a[tid], -e) : 4.f;
      const float b = tid > 0 && tid < d ? __builtin_amdgcn_ldexpf(s_b[tid - 1], -e) : 0.f;
      s_bs[tid] = tid > 0 && tid < d ? fmaxf(b * b, 1e-18f) : 0.f;
    }
    __syncthreads();
    const float lo = __builtin_amdgcn_ldexpf(glo, -e), hi = __builtin_amdgcn_ldexpf(ghi, -e);
    if (m <= 32) multisect<8, 6>(s_as, s_bs, s_lam, s_cnt, s_cs, lo, hi, e, d, m, s_fail);
    else if (m <= 64) multisect<4, 8>(s_as, s_bs, s_lam, s_cnt, s_cs, lo, hi, e, d, m, s_fail);
    else multisect<2, 12>(s_as, s_bs, s_lam, s_cnt, s_cs, lo, hi, e, d, m, s_fail);
  }
  if (failed()) return;
  // clusters: runs of eigenvalues within 1e-3 |T| of their predecessor
  // (equal ones always, also when T = 0): s_cs[j] is the last run start at or
  // before j, a running maximum over the starts (wave 0, 64 entries a pass)
  if (wave == 0) {
    int carry = 0;
    for (int base = 0; base < m; base += 64) {
      const int j = base + lane;
      int v = (j < m && (j == 0 || !(s_lam[j - 1] - s_lam[j] <= 1e-3f * tnorm))) ? j : 0;
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(v, o, 64);
        if (lane >= o) v = v > u ? v : u;
      }
      v = v > carry ? v : carry;
      if (j < m) s_cs[j] = v;
      carry = __shfl(v, 63, 64);
    }
  }
  __syncthreads();
  // The twist rank of an eigenvalue is its place in its run of numerically
  // equal ones (within 2^-20 |T|), so that the members of an exactly
  // multiple eigenvalue take different twists; every other one takes its
  // best twist, which gives the accurate vector.
  auto twist_rank = [&](int k) {
    int rank = 0;
    while (rank < k && rank < d - 1 && s_lam[k - rank - 1] - s_lam[k - rank] <= 0x1p-20f * tnorm) ++rank;
    return rank;
  };
  if (m <= 64 && P.z_groups >= 2 * ((m + 31) >> 5)) {
    // two lanes per eigenvalue k = lane: wave 0 holds the vector's column k,
    // wave 1 a spare column (free until the back-transformation)
    const int spare = ((m + 31) >> 5) * kZGroup;
    float* const s_n2 = s_r2;                  // [2][64] partial sums of squares
    int* const s_tw = reinterpret_cast<int*>(s_r2 + 128);   // [64] twists
    const bool pair = wave < 2 && lane < m;
    float* const zk = zcol(Z, lane & 63);
    if (pair) tw_pivots(s_a, s_b2, s_b2s, zk + wave * spare, kZLd, d, s_lam[lane], wave == 0);
    __syncthreads();
    if (wave == 0 && lane < m) {
      const int r = tw_twist(s_a, zk, zk + spare, kZLd, d, s_lam[lane], twist_rank(lane));
      s_tw[lane] = r;
      zk[r * kZLd] = 1.f;                      // (row r of the spare column is not read again)
    }
    __syncthreads();
    if (pair) {
      const int r = s_tw[lane];
      s_n2[wave * 64 + lane] = wave == 0 ? tw_up(s_b, zk + spare, zk, kZLd, r) : tw_down(s_b, zk, kZLd, d, r);
    }
    __syncthreads();
    if (pair) {                                // rows split between the two waves
      const float inv = 1.f / sqrtf(1.f + s_n2[lane] + s_n2[64 + lane]);
      const int hg = ((d >> 2) + 1) >> 1;      // groups of the first wave
      const int g0 = wave == 0 ? 0 : hg, g1 = wave == 0 ? hg : (d >> 2);
      for (int g = g0; g < g1; ++g) {
#pragma unroll
        for (int u = 0; u < 4; ++u) zk[(4 * g + u) * kZLd] *= inv;
      }
    }
  } else if (tid < m) {
    twisted_vector(s_a, s_b, s_b2, s_b2s, zcol(Z, tid), kZLd, d, s_lam[tid], twist_rank(tid));
  }
  __syncthreads();
  // cluster members orthogonalised against the members before them (wave 0):
  // z_k stays in registers (rows lane and lane + 64) through its member's pass
  if (wave == 0) {
    const bool r0 = lane < d, r1 = lane + 64 < d;
    for (int k = 1; k < m; ++k) {
      const int c0 = s_cs[k];
      if (c0 == k) continue;
      float* const ck = zcol(Z, k) + lane * kZLd;
      float zk0 = r0 ? ck[0] : 0.f, zk1 = r1 ? ck[64 * kZLd] : 0.f;
      for (int i = c0; i < k; ++i) {
        const float* const ci = zcol(Z, i) + lane * kZLd;
        const float zi0 = r0 ? ci[0] : 0.f, zi1 = r1 ? ci[64 * kZLd] : 0.f;
        const float dt = tri_wave_sum(fmaf(zi0, zk0, zi1 * zk1));
        zk0 -= dt * zi0;
        zk1 -= dt * zi1;
      }
      const float n2 = tri_wave_sum(fmaf(zk0, zk0, zk1 * zk1));
      // a member that was mostly inside the span of the ones before it is
      // not trusted (twisted vectors of an exactly multiple eigenvalue)
      if (lane == 0 && !(n2 >= 0.25f)) *s_fail = 1;
      const float inv = n2 > 0.f ? 1.f / sqrtf(n2) : 0.f;
      if (r0) ck[0] = zk0 * inv;
      if (r1) ck[64 * kZLd] = zk1 * inv;
    }
  }
  __syncthreads();
  // every vector must satisfy |T z - lambda z| <= 2^-16 |T| (good ones reach
  // ~d u |T|); a larger or non-finite residual sends the unit to Jacobi.
  // The rows of a vector are split over four waves (two at rank > 64), the
  // partial sums meeting in LDS
  {
    const int mc = (m + 63) >> 6, parts = 4 / mc;
    const int k = lane + 64 * (wave % mc), part = wave / mc;
    const int i0 = part * (d / parts), i1 = i0 + d / parts;
    if (k < m) {
      const float* const zk = zcol(Z, k);
      const float lam = s_lam[k], inv_tn = tnorm > 0.f ? 1.f / tnorm : 0.f;
      float r2 = 0.f;
#pragma unroll 8
      for (int i = i0; i < i1; ++i) {
        float t = (s_a[i] - lam) * zk[i * kZLd];
        if (i > 0) t += s_b[i - 1] * zk[(i - 1) * kZLd];
        if (i < d - 1) t += s_b[i] * zk[(i + 1) * kZLd];
        t *= inv_tn;
        r2 += t * t;
      }
      s_r2[part * 128 + k] = r2;
    }
    __syncthreads();
    if (tid < m) {
      float r2 = 0.f;
      for (int q = 0; q < parts; ++q) r2 += s_r2[q * 128 + tid];
      if (!(r2 <= 0x1p-32f)) *s_fail = 1;
    }
  }
  if (failed()) return;
  uint16_t* const Wout = P.W + (int64_t)c * P.w_s[0] + (int64_t)l * P.w_s[1] + (int64_t)h * P.w_s[2];

  // ---- 4. V_m = Q Z, 64 columns at a time; the blocks' V and T are staged
  // over the columns that are in registers by then (m <= 64), else past them ----
  float* const Vs = m <= 64 ? Z : Z + ((m + 31) >> 5) * kZGroup;
  float* const Ts = Vs + 32 * kVLd;
  for (int k0 = 0; k0 < m; k0 += 64) {
    const int t = lane & 15, k4 = 4 * (lane >> 4), k = k0 + 16 * wave + t;
    f32x4v zt[2 * NB];
#pragma unroll
    for (int q = 0; q < 2 * NB; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * q + k4 + r;
        zt[q][r] = (k < m && i < d) ? zcol(Z, k)[i * kZLd] : 0.f;
      }
#pragma unroll
    for (int B = NB - 1; B >= 0; --B) {
      __syncthreads();                         // Z's columns are read, the last block is consumed
      if (J == B) {
        int c = lane & 31;
        asm volatile("" : "+v"(c));            // (else the masked tiles are formed once, before the loop over k0, and spill)
        const int h4 = 4 * (lane >> 5);
#pragma unroll
        for (int I = B; I < NB; ++I)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            f32x4v v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float x = acc[I][4 * g + e];
              const bool low = 8 * g + h4 + e > c;
              v[e] = I > B || low ? x : 0.f;
              if (I == B) Ts[(8 * g + h4 + e) * kSLd + c] = low ? 0.f : x;
            }
            *reinterpret_cast<f32x4v*>(Vs + c * kVLd + 32 * I + 8 * g + h4) = v;
          }
      }
      __syncthreads();
      if (k0 + 16 * wave < m) {
        if (B == 3) tri_apply<NB, NB == 4 ? 3 : 0>(Vs, Ts, zt);
        if (B == 2) tri_apply<NB, NB >= 3 ? 2 : 0>(Vs, Ts, zt);
        if (B == 1) tri_apply<NB, NB >= 2 ? 1 : 0>(Vs, Ts, zt);
        if (B == 0) tri_apply<NB, 0>(Vs, Ts, zt);
      }
    }
    if (k < m) {
      uint16_t* const wr = Wout + (int64_t)k * P.w_s[3] + k4;
#pragma unroll
      for (int q = 0; q < 2 * NB; ++q)
        if (16 * q + k4 < d) {                 // d is a multiple of 4: the four rows are in or out together
          const u32x2v o = {form_pack2(zt[q][0], zt[q][1]), form_pack2(zt[q][2], zt[q][3])};
          if (P.w_vec) {
            *reinterpret_cast<u32x2v*>(wr + 16 * q) = o;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) wr[16 * q + e] = (uint16_t)(o[e >> 1] >> (16 * (e & 1)));
          }
        }
    }
  }
  if (P.sigma != nullptr && tid < m) {
    const float lam = s_lam[tid];
    P.sigma[(int64_t)c * P.sigma_s[0] + (int64_t)l * P.sigma_s[1] + (int64_t)h * P.sigma_s[2] + tid] =
        sqrtf(lam > 0.f ? lam : 0.f);
  }
  if (P.sweeps_done != nullptr && tid == 0) P.sweeps_done[unit] = 0;
}

template <int NB, int S>
hipError_t launch_tri(const FormParams& p, hipStream_t s) {
  static std::atomic<bool> lds_set[kMaxDevices];
  const hipError_t e = ensure_lds_limit((const void*)form_tri_kernel<NB, S>, 4 * tri_lds_floats(6), lds_set);
  if (e != hipSuccess) return e;
  static_assert(S == 1 || (S * kTriGramBytes <= 4 * kZGroup * 4 && (NB - NB / S) * 4096 * 4 <= 4 * kZGroup * 4),
                "the Gram buffers, and the tiles handed over, fit Z");
  FormParams q = p;
  // Z: the groups m needs, at least two (the Gram stage).  Launches of at most
  // two units per CU can afford twice that at m > 32: two lanes per vector (calls
  // of 264 units of 128 x 128, rank 64: 227 us with two groups, 218 with four; 512:
  // 239 and 229; but 520, whose third unit on a CU then waits: 279 and 372).
  const int ng = (p.m + 31) / 32;
  // m > 64 needs two more for the staged reflectors.
  q.z_groups = ng > 2 ? ng + 2 : S > 1 ? 4 : ng < 2 ? 2 : (p.n_units <= 512 ? 4 : 2);
  hipLaunchKernelGGL((form_tri_kernel<NB, S>), dim3((uint32_t)p.n_units), dim3(kTriThreads * S),
                     4 * tri_lds_floats(q.z_groups), s, q);
  return hipGetLastError();
}

}  // namespace

// The Gram stages are split where each unit has a CU to itself (256 of them), at
// any number of rows (calls with S = 1 and 2, rank 64: 8 units of 1024 x 128 218 and
// 200 us, of 64 x 128 175 and 170; 256 units of 1024 x 128 249 and 231, of 64 x 128
// 180 and 173; rank 8, 256 units of 16 x 128 170 and 168).
constexpr int kTriSplitUnits = 256;

hipError_t launch_form_tridiag(const FormParams& p, hipStream_t s) {
  switch ((p.dim + 31) / 32) {
    case 1: return launch_tri<1, 1>(p, s);
    case 2: return launch_tri<2, 1>(p, s);
    case 3: return launch_tri<3, 1>(p, s);
    default:
      return p.n_units <= kTriSplitUnits ? launch_tri<4, 2>(p, s) : launch_tri<4, 1>(p, s);
  }
}

}  // namespace kamera

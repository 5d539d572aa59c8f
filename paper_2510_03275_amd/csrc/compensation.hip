// Block compensation of Algorithm 1 (the block loop), fp64 on the device.
//
//   hessian  H += 2 X^T X for calibration activations X (m x K).
//   factor   U = Cholesky((H + lambda I)^-1)^T, upper, U^T U = (H + lambda I)^-1.
//            Computed without forming the inverse: with J the index reversal,
//            J (H + lambda I) J = L L^T (blocked Cholesky, 64-column panels)
//            and U = J L^-1 J (blocked triangular inverse), because
//            (J L^-1 J)^T (J L^-1 J) = J (L L^T)^-1 J = (H + lambda I)^-1.
//   encode   the weight's row scales come from the uncompensated W (the plain
//            encoder); W is then carried in fp64 and walked in blocks of B
//            columns: block b is rounded to fp32 and encoded with those
//            scales (the same rotate / upsample / scan kernels), its
//            reconstruction Q_b = (s * C_b) E^T (E = Had D^T, the table of the
//            activation expansion, in fp64, against the packed codes) gives the error E_b = W_b - Q_b, and
//            the later columns are corrected with GPTQ's block step without its
//            column-wise part, W_F -= E_b diag(U_QQ)^-1 U_QF (each column's
//            error divided by its pivot), or optionally with the
//            optimal-brain-surgeon correction of the jointly quantized block,
//            W_F -= E_b U_QQ^-1 U_QF.
//
// All of it is dense fp64 linear algebra: one GEMM on the fp64 matrix cores
// with general strides (64 x 64 tile per workgroup, 16-deep k slices through
// LDS) serves the Hessian, the panel solves, the trailing updates, the
// triangular inverses and the block corrections.  The 64 x 64 diagonal
// blocks of the Cholesky factor are factored and inverted in registers by one
// workgroup, fused into the trailing update that produces them; another small
// kernel inverts given triangular 64-blocks in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sdq_internal.h"

namespace sdq {
namespace {

constexpr int kT = 64;     // factorisation panel / GEMM tile
constexpr int kTK = 16;    // GEMM k step
constexpr int kER = 32;    // rows of a block error tile
constexpr int kStage = kT * kTK / 256;   // operand elements staged per thread and k step
// Triangular operands of a GEMM: their zeros are left out of the K range.
constexpr int kTriB = 1;   // B[p][j] = 0 for p < j
constexpr int kTriA = 2;   // A[i][p] = 0 for p > i

// Cholesky factor and inverse of one 64 x 64 block in place: the lower part
// of A (row stride lda, unit column stride) is read, A = L L^T is written back
// with the upper part zeroed and X = L^-1 (lower) is written.  Symmetric
// elimination without square roots: step j takes column j of the reduced
// matrix (pivot d_j), forms the multipliers m_i = c_i / d_j of the rows below
// it and subtracts m_i times row j from row i, in the reduced matrix and in a
// copy of the identity, which becomes L'^-1 for the unit lower factor of
// A = L' D L'^T.  Then column j of L is c / sqrt(d_j) and L^-1 = D^-1/2 L'^-1
// (row i divided by sqrt(d_i)).  Thread t keeps a 4 x 4 sample of the reduced
// matrix and of the inverse in registers: rows t / 16 + 16 r, columns t % 16 + 16 c.
// So after each sixteen columns every thread is done with one of its rows and
// columns, and together with the triangles (c <= r; the inverse up to column j)
// 14, 12, 9 and 5 of its 32 elements are updated per step in the four phases (a
// contiguous 4 x 4 tile: 32 throughout).  With it the trailing updates that end
// in this, where it bounds them, went from 45-49 to 34 us (k = 4096, the last 40
// of 63); what is left is the latency of each column's chain, about 0.4 us.  Per step, the owners of the next column and of the next row of the
// inverse update those first and publish them in a two-slot LDS ring, with the
// next-but-one diagonal entry; from that entry every thread forms the next pivot
// and its reciprocal while the rest is updated, so only a multiply and an FMA lie
// between two barriers on the column-to-column path (one barrier per column).
// Upper entries of the diagonal samples are updated too and never read.  A pivot
// that is not positive sets *info and is taken as 1.  Needs 256 threads and 322
// doubles of LDS at lds.
__device__ __forceinline__ void chol64_tile(double* A, int64_t lda, double* X, int64_t ldx, int* info,
                                            double* lds) {
  double(*ct)[kT] = reinterpret_cast<double(*)[kT]>(lds);            // column j in slot j % 2
  double(*xr)[kT] = reinterpret_cast<double(*)[kT]>(lds + 2 * kT);   // row j of L'^-1, slot j % 2
  double* ev = lds + 4 * kT;                                          // diagonal entry j in slot j % 2
  double* dv = lds + 4 * kT + 2;                                      // pivots
  const int tid = threadIdx.x;
  const int ti = tid / 16, tk = tid % 16;
  double a[4][4], x[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = ti + 16 * r, k = tk + 16 * c;
      a[r][c] = k <= i ? A[i * lda + k] : 0.0;
      x[r][c] = i == k ? 1.0 : 0.0;
    }
  }
  if (tk == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) ct[0][ti + 16 * r] = a[r][0];
  }
  if (ti == 0) xr[0][tk] = x[0][0];
  if (ti == 1 && tk == 1) ev[1] = a[0][0];
  __syncthreads();
  double d = ct[0][0];
  if (!(d > 0.0)) {
    if (tid == 0) info[0] = 1;
    d = 1.0;
  }
  if (tid == 0) dv[0] = d;
  double rd = 1.0 / d;
  // Step j = 16 q + jj; the next column and row are in sample cn, the next but one
  // diagonal entry in sample e2 (4: past the end).
  auto step = [&](auto qc, auto cnc, auto e2c, int jj) {
    constexpr int q = decltype(qc)::value, cn = decltype(cnc)::value, e2 = decltype(e2c)::value;
    const int sl = jj & 1, sn = sl ^ 1;
    // All of the step's LDS reads first, unconditionally.
    double crv[4], ccv[4], xk[4];
#pragma unroll
    for (int r = q; r < 4; ++r) crv[r] = ct[sl][ti + 16 * r];
#pragma unroll
    for (int c = q; c < 4; ++c) ccv[c] = ct[sl][tk + 16 * c];
#pragma unroll
    for (int c = 0; c <= q; ++c) xk[c] = xr[sl][tk + 16 * c];
    const double cj = ct[sl][cn < 4 ? 16 * q + jj + 1 : 0];
    const double en = ev[sn];
    double m[4], ck[4];
    m[q] = crv[q] * (ti > jj ? rd : 0.0);                  // (entries above j are finite)
    ck[q] = tk > jj ? ccv[q] : 0.0;
#pragma unroll
    for (int r = q + 1; r < 4; ++r) {
      m[r] = crv[r] * rd;
      ck[r] = ccv[r];
    }
    if constexpr (cn < 4) {
      const int tn = (jj + 1) % 16;
      if (tk == tn) {
#pragma unroll
        for (int r = cn; r < 4; ++r) ct[sn][ti + 16 * r] = a[r][cn] - m[r] * ck[cn];
      }
      if (ti == tn) {
#pragma unroll
        for (int c = 0; c <= cn; ++c) xr[sn][tk + 16 * c] = c <= q ? x[cn][c] - m[cn] * xk[c <= q ? c : q] : x[cn][c];
      }
      if constexpr (e2 < 4) {
        const int t2 = (jj + 2) % 16;
        if (ti == t2 && tk == t2) ev[sl] = a[e2][e2] - m[e2] * ck[e2];
      }
      // next pivot: entry (j + 1, j + 1) after this step's update
      double dn = en - (cj * rd) * cj;
      if (!(dn > 0.0)) {
        if (tid == 0) info[0] = 1;
        dn = 1.0;
      }
      if (tid == 0) dv[16 * q + jj + 1] = dn;
      rd = 1.0 / dn;
    }
#pragma unroll
    for (int r = q; r < 4; ++r) {
#pragma unroll
      for (int c = q; c <= r; ++c) a[r][c] -= m[r] * ck[c];
#pragma unroll
      for (int c = 0; c <= q; ++c) x[r][c] -= m[r] * xk[c];
    }
    __syncthreads();
  };
  auto phase = [&](auto qc) {
    constexpr int q = decltype(qc)::value;
    using Next = std::integral_constant<int, q + 1>;
#pragma unroll 1
    for (int jj = 0; jj < 14; ++jj) step(qc, qc, qc, jj);
    step(qc, qc, Next{}, 14);
    step(qc, Next{}, Next{}, 15);
  };
  phase(std::integral_constant<int, 0>{});
  phase(std::integral_constant<int, 1>{});
  phase(std::integral_constant<int, 2>{});
  phase(std::integral_constant<int, 3>{});
  double* sq = ct[0];   // square roots of the pivots (the ring is free now)
  if (tid < kT) sq[tid] = sqrt(dv[tid]);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = ti + 16 * r, k = tk + 16 * c;
      A[i * lda + k] = k < i ? a[r][c] / sq[k] : (k == i ? sq[i] : 0.0);
      X[i * ldx + k] = k <= i ? x[r][c] / sq[i] : 0.0;
    }
  }
}

__global__ __launch_bounds__(256) void chol64_kernel(double* A, int64_t lda, double* X, int64_t ldx,
                                                     int* info) {
  __shared__ double lds[4 * kT + 2 + kT];
  chol64_tile(A, lda, X, ldx, info, lds);
}

// C = beta C + alpha A B; element (i, p) of A at A[i * rsa + p * csa], likewise
// B and C; blockIdx.z selects a batch (strides bsa, bsb, bsc).  lower_only = 1 (M = N)
// covers only the tiles on or below the diagonal of C; lower_only = 2 (a symmetric
// product) does too but also updates the transposed position of
// every tile below the diagonal, so both triangles are written.  beta == 0
// never reads C.  A and B
// may overlap C only where every output tile depends on the same rows of A
// alone (an in-place panel solve with N <= 64): a workgroup reads all of its
// operands before it writes.
//
// fp64 matrix cores: a 64 x 64 tile per workgroup, four waves in a 2 x 2 grid
// of 32 x 32 (four v_mfma_f64_16x16x4f64 accumulators each).  Operands go
// through LDS in 16-deep k slices (converted to fp64 on the way), the next
// slice loaded into registers while the current one is multiplied.  Lane
// layout of the instruction: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] and receives D[l / 16 + 4 v][l % 16] in item v.
typedef double double4_t __attribute__((ext_vector_type(4)));

template <typename TA, typename TB, bool kChol = false>
__global__ __launch_bounds__(256) void gemm64_kernel(
    int64_t M, int64_t N, int64_t K, double alpha, const TA* A, int64_t rsa, int64_t csa,
    int64_t bsa, const TB* B, int64_t rsb, int64_t csb, int64_t bsb, double beta, double* C,
    int64_t rsc, int64_t csc, int64_t bsc, int lower_only, int tri, double* cx, int64_t ldx, int* info) {
  __shared__ double As[kTK][kT + 2];
  __shared__ double Bs[kTK][kT + 2];
  const int tid = threadIdx.x;
  const int lane = tid % 64, wave = tid / 64;
  const int wr = wave / 2, wc = wave % 2;
  int64_t ty = blockIdx.y, tx = blockIdx.x;
  if (lower_only) {
    // A one-dimensional grid over the tiles on or below the diagonal, row by row,
    // each XCD a contiguous range (workgroups go to the eight XCDs in turn, each
    // with its own L2).  A square grid whose upper half returned at once gave
    // the XCDs and CUs unequal shares.
    const int64_t g = gridDim.x, xcd = tx % 8;
    const int64_t t = xcd * (g / 8) + min<int64_t>(xcd, g % 8) + tx / 8;
    ty = static_cast<int64_t>((sqrt(8.0 * static_cast<double>(t) + 1.0) - 1.0) * 0.5);
    while ((ty + 1) * (ty + 2) / 2 <= t) ++ty;
    while (ty * (ty + 1) / 2 > t) --ty;
    tx = t - ty * (ty + 1) / 2;
  } else if (tri == kTriB && (ty / 8) % 2) {
    // Triangular B: the K range shrinks along a row of tiles, and a CU gets every
    // eighth row of one column (256 CUs, eight XCDs); every other eight rows run
    // backwards, which evens the CUs out (2048-blocks: 349 us without the K
    // ranges, 221 with them; without this order they gained nothing).
    tx = gridDim.x - 1 - tx;
  }
  const int64_t i0 = ty * kT, j0 = tx * kT;
  A += static_cast<int64_t>(blockIdx.z) * bsa;
  B += static_cast<int64_t>(blockIdx.z) * bsb;
  C += static_cast<int64_t>(blockIdx.z) * bsc;
  const int64_t kb = tri == kTriB ? j0 : 0;                          // K range (j0, i0: multiples of the slice)
  const int64_t ke = tri == kTriA ? min<int64_t>(K, i0 + kT) : K;
  // Staging: element e = tid + 256 q of the slice, consecutive threads along
  // the operand's contiguous index.
  const bool a_pfast = csa == 1;
  const bool b_jfast = csb == 1;
  // Element q of a thread: row ai + q aii at p = ap + q api (and likewise B).  Loads
  // are unconditional, from clamped places: rows and columns past the matrix
  // feed outputs that are not stored, and what lies past K is stored as zero.
  const int ap = a_pfast ? tid % kTK : tid / kT, ai = a_pfast ? tid / kTK : tid % kT;
  const int bp = b_jfast ? tid / kT : tid % kTK, bj = b_jfast ? tid % kT : tid / kTK;
  const int api = a_pfast ? 0 : 4, aii = a_pfast ? 16 : 0;
  const int bpi = b_jfast ? 4 : 0, bji = b_jfast ? 0 : 16;
  const TA* ag[kStage];
  const TB* bg[kStage];
#pragma unroll
  for (int q = 0; q < kStage; ++q) {
    ag[q] = A + min<int64_t>(i0 + ai + q * aii, M - 1) * rsa + (kb + min<int64_t>(ap + q * api, K - 1 - kb)) * csa;
    bg[q] = B + min<int64_t>(j0 + bj + q * bji, N - 1) * csb + (kb + min<int64_t>(bp + q * bpi, K - 1 - kb)) * rsb;
  }
  TA ra[kStage];
  TB rb[kStage];
  auto load = [&](int64_t p0) {
    if (p0 + kTK <= K) {
#pragma unroll
      for (int q = 0; q < kStage; ++q) {
        ra[q] = ag[q][(p0 - kb) * csa];
        rb[q] = bg[q][(p0 - kb) * rsb];
      }
    } else {
#pragma unroll
      for (int q = 0; q < kStage; ++q) {   // a last, partial slice
        const bool av = p0 + ap + q * api < K, bv = p0 + bp + q * bpi < K;
        ra[q] = ag[q][av ? (p0 - kb) * csa : 0];
        rb[q] = bg[q][bv ? (p0 - kb) * rsb : 0];
        ra[q] = av ? ra[q] : TA(0);
        rb[q] = bv ? rb[q] : TB(0);
      }
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int q = 0; q < kStage; ++q) {
      As[ap + q * api][ai + q * aii] = static_cast<double>(ra[q]);
      Bs[bp + q * bpi][bj + q * bji] = static_cast<double>(rb[q]);
    }
  };
  double4_t acc[2][2];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[r][c] = double4_t{0.0, 0.0, 0.0, 0.0};
  const int lr = lane % 16, lk = lane / 16;
  load(kb);
  store();
  __syncthreads();
  for (int64_t p0 = kb; p0 < ke; p0 += kTK) {
    const bool more = p0 + kTK < ke;
    if (more) load(p0 + kTK);
#pragma unroll
    for (int kk = 0; kk < kTK / 4; ++kk) {
      double a[2], b[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) a[r] = As[4 * kk + lk][32 * wr + 16 * r + lr];
#pragma unroll
      for (int c = 0; c < 2; ++c) b[c] = Bs[4 * kk + lk][32 * wc + 16 * c + lr];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], b[c], acc[r][c], 0, 0, 0);
    }
    __syncthreads();
    if (more) {
      store();
      __syncthreads();
    }
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t gi = i0 + 32 * wr + 16 * r + lk + 4 * v, gj = j0 + 32 * wc + 16 * c + lr;
        if (gi < M && gj < N) {
          double* cp = C + gi * rsc + gj * csc;
          double val = alpha * acc[r][c][v];
          if (beta != 0.0) val += beta * *cp;
          *cp = val;
          if (lower_only == 2 && i0 > j0) {
            double* mp = C + gj * rsc + gi * csc;
            double mv = alpha * acc[r][c][v];
            if (beta != 0.0) mv += beta * *mp;
            *mp = mv;
          }
        }
      }
  if constexpr (kChol) {
    // The first tile goes on to its Cholesky factor and inverse (the tile's
    // stores above are visible to the whole workgroup after the barrier).
    if (i0 == 0 && j0 == 0) {
      __syncthreads();
      chol64_tile(C, rsc, cx, ldx, info, &As[0][0]);
    }
  }
}

// The block error of the compensated encoder straight from the codes and the
// weights: E = W_b - (s C_b) Eb^T with C_b the packed codes of samples j0 .. j0 + M - 1
// (M a multiple of 32, j0 too: a 16-deep slice is one ternary word or half a
// binary one) and Eb the B x M table; out[r][t] = E[r][t] / u[t][t], or
// E[r][t] where u is null.  The codes are decoded into the LDS slice, so the scaled
// codes, the copy of the block and the division take no pass of their own.  32 x 64
// tile (each wave 16 x 32), so that 4096 rows and 256 columns give two workgroups
// per CU and one multiplies while the other waits for its loads, issued two slices
// ahead.  A block of 4096 rows and 512 samples: 61 us of passes and product before,
// 33 with 64 x 64 tiles, 30 so; 14 us at the matrix cores' 77 TFLOP/s.
template <int BITS>
__global__ __launch_bounds__(256) void block_error_kernel(
    const uint32_t* __restrict__ codes, const float* __restrict__ scales, int64_t n, int64_t n_chunks, int64_t j0s,
    int64_t M, const double* __restrict__ e64, const double* __restrict__ w, int64_t ldw, int B,
    const double* __restrict__ u, int64_t ldu, double* __restrict__ out) {
  __shared__ double As[2][kTK][kER + 2];
  __shared__ double Bs[2][kTK][kT + 2];
  const int tid = threadIdx.x;
  const int lane = tid % 64, wave = tid / 64;
  const int wr = wave / 2, wc = wave % 2;
  const int64_t i0 = static_cast<int64_t>(blockIdx.y) * kER;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kT;
  // Codes: thread t decodes samples 2 (t % 8) and the next of row t / 8; the table:
  // sample t % 16 of rows t / 16 + 16 q.  Rows past n have codes of 0 (padding) or
  // are not stored.
  const int64_t row = min<int64_t>(i0 + tid / 8, n - 1);
  const double s = static_cast<double>(scales[row]);
  const uint32_t* crow = codes + ((row / kPanel) * n_chunks * kPanel + row % kPanel) * 4;
  const double* eb = e64 + (t0 + tid / 16) * M + tid % 16;
  uint32_t word[2];
  double rb[2][4];
  auto load = [&](int set, int64_t p) {
    const int64_t p0 = min<int64_t>(p, M - kTK);               // (a slice past the end is not multiplied)
    const int64_t bit = (j0s + p0) * BITS;                     // of the row's code string
    const int64_t wi = bit / 32;
    word[set] = crow[(wi / 4) * kPanel * 4 + wi % 4] >> (bit % 32);
#pragma unroll
    for (int q = 0; q < 4; ++q) rb[set][q] = eb[p0 + 16 * q * M];
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const uint32_t f = (word[buf] >> (BITS * (2 * (tid % 8) + q))) & ((1u << BITS) - 1u);
      const double code = BITS == 1 ? (f ? 1.0 : -1.0) : (f == 1u ? 1.0 : (f == 3u ? -1.0 : 0.0));
      As[buf][2 * (tid % 8) + q][tid / 8] = s * code;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) Bs[buf][tid % 16][tid / 16 + 16 * q] = rb[buf][q];
  };
  double4_t acc[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) acc[c] = double4_t{0.0, 0.0, 0.0, 0.0};
  const int lr = lane % 16, lk = lane / 16;
  auto slice = [&](int cur, int64_t p0) {
    load(cur, p0 + 2 * kTK);
#pragma unroll
    for (int kk = 0; kk < kTK / 4; ++kk) {
      double b[2];
      const double a = As[cur][4 * kk + lk][16 * wr + lr];
#pragma unroll
      for (int c = 0; c < 2; ++c) b[c] = Bs[cur][4 * kk + lk][32 * wc + 16 * c + lr];
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[c], acc[c], 0, 0, 0);
    }
    store(cur ^ 1);
    __syncthreads();
  };
  load(0, 0);
  load(1, kTK);
  store(0);
  __syncthreads();
  for (int64_t p0 = 0; p0 < M; p0 += 2 * kTK) {    // M is a multiple of 32
    slice(0, p0);
    slice(1, p0 + kTK);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int64_t t = t0 + 32 * wc + 16 * c + lr;
    const double piv = u ? u[t * ldu + t] : 1.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t gi = i0 + 16 * wr + lk + 4 * v;
      if (gi < n) {
        const double e = w[gi * ldw + t] - acc[c][v];
        out[gi * B + t] = u ? e / piv : e;
      }
    }
  }
}

// Inverse X = L^-1 of lower-triangular 64 x 64 diagonal blocks, one per
// workgroup (grid x: blocks along a diagonal, stride sa1 / sx1; grid y:
// batches, stride sa2 / sx2), in three levels: the four 16 x 16 diagonal
// blocks by forward substitution (one column per thread), then pairs of
// diagonal blocks are joined as X21 = -X22 (L21 X11), 16 -> 32 and 32 -> 64,
// every output of a product on its own thread.
__global__ __launch_bounds__(256) void trinv64_kernel(const double* A, int64_t lda, int64_t sa1, int64_t sa2,
                                                      double* X, int64_t ldx, int64_t sx1, int64_t sx2) {
  __shared__ double a[kT][kT + 1];
  __shared__ double x[kT][kT + 1];
  A += blockIdx.x * sa1 + blockIdx.y * sa2;
  X += blockIdx.x * sx1 + blockIdx.y * sx2;
  const int tid = threadIdx.x;
  for (int e = tid; e < kT * kT; e += 256) {
    const int i = e / kT, k = e % kT;
    a[i][k] = k <= i ? A[i * lda + k] : 0.0;
  }
  __syncthreads();
  __shared__ double rd[kT];          // 1 / L[i][i]
  __shared__ double tt[32 * 32];     // L21 X11 of the current level
  if (tid < kT) rd[tid] = 1.0 / a[tid][tid];
  for (int e = tid; e < kT * kT; e += 256) x[e / kT][e % kT] = 0.0;
  __syncthreads();
  if (tid < kT) {
    const int o = 16 * (tid / 16), c = tid % 16;
    for (int i = c; i < 16; ++i) {
      double s = i == c ? 1.0 : 0.0;
      for (int k = c; k < i; ++k) s -= a[o + i][o + k] * x[o + k][o + c];
      x[o + i][o + c] = s * rd[o + i];
    }
  }
  __syncthreads();
  for (int b = 16; b < kT; b *= 2) {
    const int pairs = kT / (2 * b);
    for (int e = tid; e < pairs * b * b; e += 256) {
      const int pr = e / (b * b), i = (e / b) % b, j = e % b, r = 2 * b * pr;
      double s = 0.0;
      for (int k = j; k < b; ++k) s += a[r + b + i][r + k] * x[r + k][r + j];
      tt[(pr * b + i) * b + j] = s;
    }
    __syncthreads();
    for (int e = tid; e < pairs * b * b; e += 256) {
      const int pr = e / (b * b), i = (e / b) % b, j = e % b, r = 2 * b * pr;
      double s = 0.0;
      for (int k = 0; k <= i; ++k) s += x[r + b + i][r + b + k] * tt[(pr * b + k) * b + j];
      x[r + b + i][r + j] = -s;
    }
    __syncthreads();
  }
  __syncthreads();
  for (int e = tid; e < kT * kT; e += 256) {
    const int i = e / kT, k = e % kT;
    X[i * ldx + k] = x[i][k];
  }
}

// dst[i][j] = src[n-1-i][n-1-j] (+ lam on the diagonal) where kept (i >= j
// for keep_lower, else j >= i), 0 elsewhere; grid y selects a batch.
__global__ void reverse_tri_kernel(const double* __restrict__ src, int64_t lds, int64_t ss,
                                   int64_t n, double* __restrict__ dst, int64_t ldd, int64_t sd,
                                   int keep_lower, double lam) {
  src += blockIdx.y * ss;
  dst += blockIdx.y * sd;
  for (int64_t e = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; e < n * n;
       e += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t i = e / n, j = e % n;
    const bool keep = keep_lower ? i >= j : j >= i;
    dst[i * ldd + j] = keep ? src[(n - 1 - i) * lds + (n - 1 - j)] + (i == j ? lam : 0.0) : 0.0;
  }
}

__global__ void fill_f64_kernel(double* __restrict__ p, int64_t count, double v) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < count;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = v;
}

__global__ void clear_info_kernel(int* info) { if (threadIdx.x == 0) info[0] = 0; }

__global__ void widen_kernel(const float* __restrict__ w, int64_t count, double* __restrict__ w64) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < count;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    w64[i] = static_cast<double>(w[i]);
}

unsigned grid1(int64_t count) {
  return static_cast<unsigned>(std::min<int64_t>((count + 255) / 256, 8192));
}

// lower_only as for the kernel; tri: kTriA, kTriB or 0.
template <typename TA, typename TB>
void gemm64(int64_t M, int64_t N, int64_t K, double alpha, const TA* A, int64_t rsa, int64_t csa,
            const TB* B, int64_t rsb, int64_t csb, double beta, double* C, int64_t rsc, int64_t csc,
            hipStream_t stream, int lower_only = 0, int batch = 1, int64_t bsa = 0, int64_t bsb = 0,
            int64_t bsc = 0, int tri = 0) {
  if (M <= 0 || N <= 0) return;
  const int64_t by = (M + kT - 1) / kT, bx = (N + kT - 1) / kT;
  const dim3 grid(static_cast<unsigned>(lower_only ? by * (by + 1) / 2 : bx), static_cast<unsigned>(lower_only ? 1 : by),
                  static_cast<unsigned>(batch));
  gemm64_kernel<TA, TB><<<grid, dim3(256), 0, stream>>>(M, N, K, alpha, A, rsa, csa, bsa, B, rsb, csb,
                                                        bsb, beta, C, rsc, csc, bsc, lower_only, tri, nullptr, 0,
                                                        nullptr);
}

// Trailing update of a right-looking Cholesky step, C -= P P^T on the tiles
// on or below the diagonal (P: n x 64, row stride ld; C: n x n, row stride
// ld), whose first tile then factors and inverts the next diagonal block
// (L into C's first tile, its inverse into X).
void trailing_update_chol(int64_t n, const double* P, double* C, int64_t ld, double* X, int64_t ldx, int* info,
                          hipStream_t stream) {
  const int64_t tiles = (n + kT - 1) / kT;
  gemm64_kernel<double, double, true><<<dim3(static_cast<unsigned>(tiles * (tiles + 1) / 2)), dim3(256), 0, stream>>>(
      n, n, int64_t{kT}, -1.0, P, ld, int64_t{1}, 0, P, int64_t{1}, ld, 0, 1.0, C, ld, int64_t{1}, 0, 1, 0,
      X, ldx, info);
}

// Lower-triangular inverse X = L^-1 of a batch of n x n matrices (n a multiple
// of 64; batch stride s): the diagonal 64-blocks of X must already hold the
// inverses of L's, X's strictly upper part zero; tmp holds n^2 / 4 per batch.
// For a lower-triangular [L11 0; L21 L22] with X11 = L11^-1 and X22 = L22^-1,
// the missing block is X21 = -X22 (L21 X11).  A power-of-two size (64 2^j)
// joins its diagonal blocks pairwise up a binary tree, two b x b x b products
// per pair, batched over the pairs of a level (one matrix) or over the
// matrices (one launch per pair); any other size splits off its largest
// power-of-two leading block, inverts the rest recursively and joins the two.
void trtri_pow2(const double* L, double* X, int64_t n, int64_t ld, int64_t s, int batch, double* tmp,
                hipStream_t stream) {
  for (int64_t b = kT; b < n; b *= 2) {
    const int64_t pairs = n / (2 * b);
    const int64_t ps = 2 * b * (ld + 1);                  // diagonal step between pairs
    auto join = [&](int64_t off, int nbat, int64_t mstride) {
      gemm64(b, b, b, 1.0, L + off + b * ld, ld, int64_t{1}, X + off, ld, int64_t{1}, 0.0, tmp, b,
             int64_t{1}, stream, 0, nbat, mstride, mstride, b * b, kTriB);
      gemm64(b, b, b, -1.0, X + off + b * ld + b, ld, int64_t{1}, tmp, b, int64_t{1}, 0.0, X + off + b * ld,
             ld, int64_t{1}, stream, 0, nbat, mstride, b * b, mstride, kTriA);
    };
    if (batch == 1) {
      join(0, static_cast<int>(pairs), ps);
    } else {
      for (int64_t pr = 0; pr < pairs; ++pr) join(pr * ps, batch, s);
    }
  }
}

void trtri_lower(const double* L, double* X, int64_t n, int64_t ld, int64_t s, int batch, double* tmp,
                 hipStream_t stream) {
  int64_t n1 = kT;
  while (2 * n1 < n) n1 *= 2;
  if (2 * n1 == n || n1 == n) {
    trtri_pow2(L, X, n, ld, s, batch, tmp, stream);
    return;
  }
  const int64_t n2 = n - n1;                              // 0 < n2 < n1
  trtri_pow2(L, X, n1, ld, s, batch, tmp, stream);
  trtri_lower(L + n1 * (ld + 1), X + n1 * (ld + 1), n2, ld, s, batch, tmp, stream);
  gemm64(n2, n1, n1, 1.0, L + n1 * ld, ld, int64_t{1}, X, ld, int64_t{1}, 0.0, tmp, n1, int64_t{1}, stream, 0,
         batch, s, s, n2 * n1, kTriB);
  gemm64(n2, n1, n2, -1.0, X + n1 * ld + n1, ld, int64_t{1}, tmp, n1, int64_t{1}, 0.0, X + n1 * ld, ld,
         int64_t{1}, stream, 0, batch, s, n2 * n1, s, kTriA);
}

}  // namespace

// ---------------------------------------------------------------------------

sdq_status launch_hessian_accumulate(const float* x, int64_t m, int64_t k, double* h, hipStream_t stream) {
  // H[i][j] += 2 sum_p X[p][i] X[p][j]
  gemm64(k, k, m, 2.0, x, int64_t{1}, k, x, k, int64_t{1}, 1.0, h, k, int64_t{1}, stream, 2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, "hessian launch");
  return SDQ_OK;
}

size_t hessian_factor_ws_bytes(int64_t k) {
  return 256 + align_up(static_cast<size_t>(k) * k * 8, 256) * 2 + align_up(static_cast<size_t>(k) * k * 2, 256);
}

sdq_status launch_hessian_factor(const double* h, int64_t k, double lam, double* u, void* ws,
                                 hipStream_t stream) {
  char* p = static_cast<char*>(ws);
  int* info = reinterpret_cast<int*>(p);
  double* A = reinterpret_cast<double*>(p + 256);
  double* X = reinterpret_cast<double*>(p + 256 + align_up(static_cast<size_t>(k) * k * 8, 256));
  double* tmp = reinterpret_cast<double*>(p + 256 + 2 * align_up(static_cast<size_t>(k) * k * 8, 256));
  const int64_t kk = k * k;
  clear_info_kernel<<<1, 64, 0, stream>>>(info);
  fill_f64_kernel<<<grid1(kk), 256, 0, stream>>>(X, kk, 0.0);
  reverse_tri_kernel<<<dim3(grid1(kk), 1), 256, 0, stream>>>(h, k, 0, k, A, k, 0, 1, lam);
  // Right-looking blocked Cholesky in 64-column steps: the panel below the
  // diagonal block is solved with the block's inverse, then the trailing lower
  // part is updated, and the same launch factors the next diagonal block.
  const int64_t t = k / kT;
  chol64_kernel<<<1, 256, 0, stream>>>(A, k, X, k, info);
  for (int64_t j = 0; j + 1 < t; ++j) {
    const int64_t d = j * kT, r0 = d + kT, rows = k - r0;
    // L[r0:, d] = A[r0:, d] L_dd^-T, in place
    gemm64(rows, int64_t{kT}, int64_t{kT}, 1.0, A + r0 * k + d, k, int64_t{1}, X + d * k + d, int64_t{1}, k,
           0.0, A + r0 * k + d, k, int64_t{1}, stream);
    // A[r0:, r0:] -= L[r0:, d] L[r0:, d]^T (lower), then block r0 factored
    trailing_update_chol(rows, A + r0 * k + d, A + r0 * k + r0, k, X + r0 * k + r0, k, info, stream);
  }
  trtri_lower(A, X, k, k, 0, 1, tmp, stream);
  reverse_tri_kernel<<<dim3(grid1(kk), 1), 256, 0, stream>>>(X, k, 0, k, u, k, 0, 0, 0.0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, "hessian factor launch");
  return SDQ_OK;
}

// Workspace of the compensated encoder: the plain encoder's, then (256-byte
// aligned) scratch row maxima, W64 (n x k), E and G (n x B each), and per block
// the reversed diagonal block of U, its inverse, the inverse reversed back
// (nb x B x B each) and the triangular-inverse scratch (nb x 64 x B).
struct CompWs {
  QuantWs q;
  uint32_t* rmax_scratch;
  double* w64;
  double* ebuf;
  double* gbuf;
  double* lb;
  double* xb;
  double* vb;
  double* tmp;
};

size_t comp_ws_layout(const sdq_layout* L, CompWs* out, void* base) {
  char* p = static_cast<char*>(base);
  size_t off = align_up(quant_ws_layout(L, nullptr, nullptr), 256);
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = align_up(off + bytes, 256);
    return p ? p + at : nullptr;
  };
  CompWs w;
  if (p) quant_ws_layout(L, &w.q, base);
  const size_t n = static_cast<size_t>(L->n), B = static_cast<size_t>(L->block), nb = static_cast<size_t>(L->nb);
  w.rmax_scratch = reinterpret_cast<uint32_t*>(take(static_cast<size_t>(L->n_pad) * 4));
  w.w64 = reinterpret_cast<double*>(take(n * L->k * 8));
  w.ebuf = reinterpret_cast<double*>(take(n * B * 8));
  w.gbuf = reinterpret_cast<double*>(take(n * B * 8));
  w.lb = reinterpret_cast<double*>(take(nb * B * B * 8));
  w.xb = reinterpret_cast<double*>(take(nb * B * B * 8));
  w.vb = reinterpret_cast<double*>(take(nb * B * B * 8));
  w.tmp = reinterpret_cast<double*>(take(nb * kT * B * 8));
  if (out) *out = w;
  return off;
}

sdq_status launch_quantize_compensated(const float* w, const sdq_layout* L, const Tables* T,
                                       const double* u, int update, void* codes, float* scales, void* ws,
                                       hipStream_t stream) {
  CompWs cw;
  comp_ws_layout(L, &cw, ws);
  const int64_t n = L->n, k = L->k, B = L->block, nb = L->nb, M = L->m_up;
  // Base-3 layouts: every pass works on 2-bit fields in the workspace, which
  // are repacked at the end.
  const bool base3 = L->packing == SDQ_PACK_BASE3;
  const sdq_layout Fv = fields_view(L);
  const sdq_layout* F = &Fv;
  void* fcodes = base3 ? static_cast<void*>(cw.q.codes2) : codes;
  // 1. The plain encoding: row scales of the raw W, and block 0's final codes.
  clear_rmax(cw.q, L, stream);
  sdq_status st = launch_encode_blocks(w, k, 0, nb, F, T, fcodes, scales, cw.q, cw.q.rmax, cw.q.rmax, stream);
  if (st != SDQ_OK) return st;
  // 2. Joint update only: V_b = U_bb^-1 for every block: U_bb reversed is
  //    lower triangular; invert it (64-blocks, then the off-diagonal blocks)
  //    and reverse back.
  const int64_t bb = B * B;
  const bool joint = update == SDQ_COMP_JOINT;
  if (joint) {
    fill_f64_kernel<<<grid1(nb * bb), 256, 0, stream>>>(cw.xb, nb * bb, 0.0);
    reverse_tri_kernel<<<dim3(grid1(bb), static_cast<unsigned>(nb)), 256, 0, stream>>>(
        u, k, B * k + B, B, cw.lb, B, bb, 1, 0.0);
    trinv64_kernel<<<dim3(static_cast<unsigned>(B / kT), static_cast<unsigned>(nb)), 256, 0, stream>>>(
        cw.lb, B, kT * B + kT, bb, cw.xb, B, kT * B + kT, bb);
    trtri_lower(cw.lb, cw.xb, B, B, bb, static_cast<int>(nb), cw.tmp, stream);
    reverse_tri_kernel<<<dim3(grid1(bb), static_cast<unsigned>(nb)), 256, 0, stream>>>(
        cw.xb, B, bb, B, cw.vb, B, bb, 0, 0.0);
  }
  // 3. The walk over the blocks, W in fp64.
  widen_kernel<<<grid1(n * k), 256, 0, stream>>>(w, n * k, cw.w64);
  for (int64_t b = 0; b < nb; ++b) {
    if (b > 0) {   // the block of W64, rounded to fp32
      st = launch_encode_blocks(cw.w64 + b * B, k, b, 1, F, T, fcodes, scales, cw.q, cw.rmax_scratch,
                                cw.q.rmax, stream);
      if (st != SDQ_OK) return st;
    }
    if (b == nb - 1) break;
    // E_b = W_b - (s C_b) E^T, and G = E_b diag(U_bb)^-1 or (joint) G = E_b V_b
    double* err = joint ? cw.ebuf : cw.gbuf;
    const double* piv = joint ? nullptr : u + b * B * k + b * B;
    const dim3 egrid(static_cast<unsigned>(B / kT), static_cast<unsigned>((n + kER - 1) / kER));
    if (F->bits == 1)
      block_error_kernel<1><<<egrid, 256, 0, stream>>>(static_cast<const uint32_t*>(fcodes), scales, n, F->n_chunks,
                                                       b * M, M, T->e64, cw.w64 + b * B, k, static_cast<int>(B),
                                                       piv, k, err);
    else
      block_error_kernel<2><<<egrid, 256, 0, stream>>>(static_cast<const uint32_t*>(fcodes), scales, n, F->n_chunks,
                                                       b * M, M, T->e64, cw.w64 + b * B, k, static_cast<int>(B),
                                                       piv, k, err);
    if (joint)
      gemm64(n, B, B, 1.0, cw.ebuf, B, int64_t{1}, cw.vb + b * bb, B, int64_t{1}, 0.0, cw.gbuf, B, int64_t{1},
             stream);
    // W_F -= G U[Q, F]
    const int64_t f0 = (b + 1) * B;
    gemm64(n, k - f0, B, -1.0, cw.gbuf, B, int64_t{1}, u + b * B * k + f0, k, int64_t{1}, 1.0, cw.w64 + f0, k,
           int64_t{1}, stream);
  }
  if (base3) {
    st = launch_repack_base3(cw.q.codes2, L, codes, stream);
    if (st != SDQ_OK) return st;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, "compensated encoder launch");
  return SDQ_OK;
}

size_t comp_ws_bytes(const sdq_layout* L) { return comp_ws_layout(L, nullptr, nullptr); }

}  // namespace sdq

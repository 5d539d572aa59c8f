// Prefill path of sdq_linear (m > 16 activation rows), the contraction on FP6 x
// FP4 matrix cores:
//
//   gemm     y[i, r] = s_r * sum_j x_tilde[i, j] C[r, j] with x_tilde as three FP6
//            digit planes (expand_prefill.hip: 15 bits of fixed point and one
//            power-of-two scale per 32 samples) and the codes as FP4, which
//            holds +-1, +-2 and 0 exactly: v_mfma_scale_f32_32x32x64_f8f6f4,
//            one product per plane into the same fp32 sums, the planes'
//            weights 1, 2^-5, 2^-10 and the block scales as MX scale operands.
//   reduce   adds the partial sums where K is split over workgroups.
//
// Why digits: an FP6 x FP4 product runs at four times the fp16 rate, so three
// planes take 0.75 of the fp16 matrix time (register-only probes on MI355X,
// random operands: 6.07 against 1.67 PFLOP/s, 2.0 per three planes), the
// planes' rounding is below fp16's, and a ternary or binary code becomes its
// FP4 value in one or two instructions per eight codes (fp16: sixteen).
//
// Operand layout of the instruction (checked on the device): lane l supplies
// row (A) or column (B) l % 32 and the 32 consecutive k of half l / 32, packed
// low bits first; the scale operand is one byte per lane for its 32 values;
// accumulator v holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32.  A K
// step is 64 samples.  The digit planes are stored as operand images: per step
// and 32-row group three planes of 64 lanes x 16 bytes, then 64 lanes x 8
// bytes, then the 64 block scales, so a tile is copied to LDS as one run and a wave
// reads it as runs of 1024, 512 and 64 bytes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "sdq_internal.h"

namespace sdq {
namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));
// LDS is read through these and not through HIP's uint2 / uint4: reads of class type
// lose the compiler's knowledge of which buffer they read (see ring_buffer).
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void* dig_lds_ptr;
typedef __attribute__((address_space(1))) const void* dig_gbl_ptr;

constexpr int kXcdCount = 8;

// vmcnt(n) alone (expcnt and lgkmcnt not waited on).
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0xF70; }

// Workgroup `id` of `total` to a contiguous range per XCD (workgroups are dealt
// to the eight XCDs round-robin, and each XCD has its own L2).
__device__ inline int64_t xcd_place(int64_t id, int64_t total) {
  const int64_t xcd = id % kXcdCount, j = id / kXcdCount;
  const int64_t per = total / kXcdCount, rem = total % kXcdCount;
  return xcd * per + (xcd < rem ? xcd : rem) + j;
}

// The FP4 operand of one column's 32 codes.  Ternary: the 2-bit field f at the
// top of a nibble is the value 2 code (01 -> 0100 = 2, 11 -> 1100 = -2, 00 -> 0);
// the odd codes of a word sit there already.  Binary: bit b in the sign of 0010
// is -code (1 - 2 b); the row scale takes the sign back.
template <int LEVELS>
__device__ inline i32x8 fp4_codes(uint32_t w0, uint32_t w1) {
  i32x8 r = {0, 0, 0, 0, 0, 0, 0, 0};
  if constexpr (LEVELS == 3) {
    r[0] = static_cast<int>((w0 << 2) & 0xCCCCCCCCu);
    r[1] = static_cast<int>(w0 & 0xCCCCCCCCu);
    r[2] = static_cast<int>((w1 << 2) & 0xCCCCCCCCu);
    r[3] = static_cast<int>(w1 & 0xCCCCCCCCu);
  } else {
#pragma unroll
    for (int d = 0; d < 4; ++d) r[d] = static_cast<int>(((w0 << (3 - d)) & 0x88888888u) | 0x22222222u);
  }
  return r;
}

// Buffer J of a workgroup's ring of tiles.  An array each: in front of an LDS read
// the compiler waits for every outstanding copy into the same array.
template <int TB, int J>
__device__ inline uint8_t* ring_buffer() {
  __shared__ __attribute__((aligned(1024))) uint8_t buf[TB];
  return buf;
}

struct DigitParts {           // partial sums of a split contraction (splits > 1)
  float* base = nullptr;
  int64_t off[kMaxGroup] = {};     // of each linear's [splits][stride]
  int64_t stride[kMaxGroup] = {};
};

// WM x WN waves, each RT x CT accumulator tiles of 32 x 32: a workgroup tile of
// RG = WM RT row groups (32 activation rows each) x 256 weight rows, over the
// K steps of its split.  The step's x_tilde tile and its codes (BN / 64 panels, 64
// rows x 16 bytes each) come straight from global memory to a ring of kRing LDS
// buffers, kRing - 1 steps ahead; one plain barrier per step with a counted wait, so
// that the copies of the following steps stay in flight.  Codes loaded to
// registers between the copies to LDS held up a workgroup's start (a 64 x 256
// tile stopped after its first eight steps: 38 us, against 8 without the code
// loads, 9 without the copies and 17 with both through LDS) and took the
// registers of four steps; whole calls differ by a few per cent.
// The sums are kept 2^-kSumShift times their value, since codes times x_tilde may add
// up past fp32 where the row scale brings the result back into it (rows of x from about
// 2^120 on); fp32 sums lose nothing by it down to rows of 2^-126.
// APART: a contraction called apart, which returns if fp16 x_tilde is there (a template
// parameter, since the test in front of everything else cost a whole call 0.4 us).
constexpr int kRing = 4;
constexpr int kSumShift = 8;
template <int LEVELS, int WM, int WN, int RT, int CT, int MINW, bool APART>
__global__ __launch_bounds__(64 * WM * WN, MINW) void gemm_digits_kernel(
    const uint8_t* __restrict__ planes, LinearSet S, int64_t m, int64_t n_chunks, int64_t n_rg, int n_steps,
    int64_t m_tiles, int64_t n_tiles, int steps_per, int accumulate, DigitParts part, const float* form) {
  if (APART && !(*form < 0.0f)) return;
  constexpr int RG = WM * RT;
  constexpr int W = WM * WN;
  constexpr int BN = 32 * CT * WN;                 // weight rows of the tile
  static_assert(BN % kPanel == 0, "whole panels");
  constexpr int TU = RG * kDigitTile / 16;         // 16-byte units of an x_tilde tile
  constexpr int NX = (TU + 63) / 64;               // copies of 64 units
  constexpr int NC = NX + BN / kPanel;       // and one per panel of codes
  constexpr int FC = (NC + W - 1) / W;             // copies per wave
  constexpr int TB = (NC + (NC % W ? 1 : 0)) * 1024;   // LDS bytes per buffer (the last KB takes the surplus copies)
  constexpr int CODES = NX * 1024;                 // the codes' place in it
  static_assert((kRing - 2) * FC <= 63, "vmcnt range");
  auto ring = [](auto jc) { return ring_buffer<TB, decltype(jc)::value % kRing>(); };
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int half = lane / 32;
  const int wm = wave / WN, wn = wave % WN;
  // Order of the work: splits slowest, then pairs of row tiles across the column
  // tiles, so that the workgroups of one XCD share x_tilde and code slices.
  const int64_t tiles = m_tiles * n_tiles;
  const int64_t u = xcd_place(blockIdx.x, gridDim.x);
  const int64_t split = u / tiles, t = u % tiles;
  const int64_t p = t / (2 * n_tiles), r2 = t % (2 * n_tiles);
  const int64_t in_pair = min<int64_t>(2, m_tiles - 2 * p);
  const int64_t nt = r2 / in_pair, mt = 2 * p + r2 % in_pair;
  int lin = 0;
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i)
    if (i < S.count && nt >= S.first[i]) lin = i;
  const int64_t n = S.n[lin];
  const int64_t rg0 = mt * RG;
  const int64_t n0 = (nt - S.first[lin]) * BN + wn * 32 * CT;
  const int it0 = static_cast<int>(split) * steps_per;
  const int n_it = min(n_steps - it0, steps_per);

  // Copy j of a step is 64 lanes x 16 bytes; wave w issues copies w, w + W, ..., FC
  // of them (one wait count serves all waves, without a branch; a surplus copy
  // reads one unit).  Row groups past the last read the last, panels past the
  // last read the last: what they feed is not stored.
  const int64_t panels = (n + kPanel - 1) / kPanel, panel0 = (nt - S.first[lin]) * (BN / kPanel);
  const uint8_t* __restrict__ cbase = static_cast<const uint8_t*>(S.codes[lin]) + panel0 * n_chunks * (kPanel * 16);
  uint32_t a_off[FC];
#pragma unroll
  for (int j = 0; j < FC; ++j) {
    const int cj = wave + W * j;
    const int unit = min(64 * cj + lane, TU - 1);
    const int rs = static_cast<int>(min<int64_t>(unit / (kDigitTile / 16), n_rg - 1 - rg0));
    const int q = static_cast<int>(min<int64_t>(cj - NX, panels - 1 - panel0));
    a_off[j] = cj >= NC ? 0u
               : cj < NX ? static_cast<uint32_t>(rs * kDigitTile + 16 * (unit % (kDigitTile / 16)))
                         : static_cast<uint32_t>(q) * static_cast<uint32_t>(n_chunks) * (kPanel * 16) + 16 * lane;
  }
  auto fill = [&](uint8_t* buf, int it) {
    const int s = min(it, n_steps - 1);
    const int64_t ch = min<int64_t>(LEVELS == 3 ? s : s / 2, n_chunks - 1);
    const uint8_t* ps = planes + (static_cast<int64_t>(s) * n_rg + rg0) * kDigitTile;
    const uint8_t* cs = cbase + ch * (kPanel * 16);
#pragma unroll
    for (int j = 0; j < FC; ++j) {
      const int cj = wave + W * j;
      __builtin_amdgcn_global_load_lds((dig_gbl_ptr)((cj < NX ? ps : cs) + a_off[j]),
                                       (dig_lds_ptr)(buf + 1024 * min(cj, NC)), 16, 0, 0);
    }
  };
  // Wait until at most kRing - 2 steps' copies of this wave are outstanding, then for
  // every wave: the next step's are there.  Nothing is scheduled across it.
  auto landed = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm((kRing - 2) * FC));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  floatx16 acc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[r][c][v] = 0.0f;

  // One step: reads buffer J, refills the one the previous step read.
  auto step = [&](auto jc, int it) {
    constexpr int J = decltype(jc)::value;
    const uint8_t* buf = ring(jc) + wm * RT * kDigitTile;
    const uint8_t* cbuf = ring(jc) + CODES + wn * CT * 512 + 16 * (lane % 32) + 8 * half;
    int sa[RT];
    i32x8 a[3][RT];
    auto read = [&](int pl) {
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const uint8_t* ap = buf + r * kDigitTile + pl * kDigitPlane;
        const u32x4 lo = *reinterpret_cast<const u32x4*>(ap + 16 * lane);
        const u32x2 hi = *reinterpret_cast<const u32x2*>(ap + 1024 + 8 * lane);
        a[pl][r] = i32x8{static_cast<int>(lo.x), static_cast<int>(lo.y), static_cast<int>(lo.z),
                         static_cast<int>(lo.w), static_cast<int>(hi.x), static_cast<int>(hi.y), 0, 0};
      }
    };
    i32x8 b[CT];
    auto products = [&](int pl) {
      const int sb = (LEVELS == 3 ? 126 : 127) - 5 * pl - kSumShift;   // plane weight 2^-5pl, codes as 2 code
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int c = 0; c < CT; ++c)
          acc[r][c] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[pl][r], b[c], acc[r][c], 2, 4, 0, sa[r], 0, sb);
    };
    // Every LDS read of the step comes before its refill (the compiler takes a
    // copy issued in the same step for one into this buffer).
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      if constexpr (LEVELS == 3) {
        const u32x2 w = *reinterpret_cast<const u32x2*>(cbuf + 512 * c);
        b[c] = fp4_codes<3>(w.x, w.y);
      } else {   // words 2 half (even steps) and 2 half + 1 (odd steps) of the chunk
        b[c] = fp4_codes<2>(*reinterpret_cast<const uint32_t*>(cbuf + 512 * c + 4 * (it & 1)), 0u);
      }
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) sa[r] = buf[r * kDigitTile + 3 * kDigitPlane + lane];
    read(0);
    read(1);
    products(0);
    read(2);
    __builtin_amdgcn_sched_barrier(0);
    fill(ring(std::integral_constant<int, J + kRing - 1>{}), it + kRing - 1);
    products(1);
    products(2);
    landed();
  };
  using J0 = std::integral_constant<int, 0>;
  using J1 = std::integral_constant<int, 1>;
  using J2 = std::integral_constant<int, 2>;
  using J3 = std::integral_constant<int, 3>;
  fill(ring(J0{}), it0);
  __builtin_amdgcn_sched_barrier(0);
  fill(ring(J1{}), it0 + 1);
  __builtin_amdgcn_sched_barrier(0);
  fill(ring(J2{}), it0 + 2);
  landed();
  static_assert(kRing == 4, "steps of a round");
  int it = it0;
  for (const int whole = it0 + n_it / kRing * kRing; it < whole; it += kRing) {
    step(J0{}, it);
    step(J1{}, it + 1);
    step(J2{}, it + 2);
    step(J3{}, it + 3);
  }
  if (n_it % kRing) {                              // n_it is even
    step(J0{}, it);
    step(J1{}, it + 1);
  }
  // the last copies (never read) land before the workgroup's LDS is released
  __builtin_amdgcn_s_waitcnt(0);

  const float* __restrict__ scales = S.scales[lin];
  float* __restrict__ y = part.base ? part.base + part.off[lin] + split * part.stride[lin] : S.y[lin];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int64_t col = n0 + 32 * c + lane % 32;
    if (col >= n) continue;
    const float s0 = LEVELS == 2 ? -scales[col] : scales[col];
    constexpr float up = static_cast<float>(1 << kSumShift);
    const bool small = fabsf(s0) < 0x1p100f;                 // (both products are exact)
    const float s = small ? s0 * up : s0, back = small ? 1.0f : up;
    auto store = [&](auto whole, auto add) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int64_t row = (rg0 + wm * RT + r) * 32 + 8 * (v / 4) + 4 * half + v % 4;
          if (decltype(whole)::value || row < m) {
            float* out = y + row * n + col;
            const float val = acc[r][c][v] * back * s;
            *out = decltype(add)::value ? *out + val : val;
          }
        }
    };
    if (accumulate) store(std::false_type{}, std::true_type{});
    else if ((rg0 + RG) * 32 <= m) store(std::true_type{}, std::false_type{});
    else store(std::false_type{}, std::false_type{});
  }
}

// y (+)= the sum of a linear's partial sums, in the order of the splits.  V
// floats per thread and load (4 where y is 16-byte aligned).  APART as above.
template <int V, bool APART>
__global__ __launch_bounds__(256) void reduce_digits_kernel(LinearSet S, DigitParts part, int64_t m, int splits,
                                                            int accumulate, const float* form) {
  if (APART && !(*form < 0.0f)) return;
  const int lin = blockIdx.y;
  const int64_t cnt = m * S.n[lin];
  const float* __restrict__ src = part.base + part.off[lin];
  const int64_t stride = part.stride[lin];
  float* __restrict__ y = S.y[lin];
  for (int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * V; i < cnt;
       i += static_cast<int64_t>(gridDim.x) * 256 * V) {
    if (V == 4 && i + 4 <= cnt) {
      float4 a = *reinterpret_cast<const float4*>(src + i);
      for (int s = 1; s < splits; ++s) {
        const float4 b = *reinterpret_cast<const float4*>(src + s * stride + i);
        a.x += b.x;
        a.y += b.y;
        a.z += b.z;
        a.w += b.w;
      }
      float4* out = reinterpret_cast<float4*>(y + i);
      if (accumulate) {
        const float4 b = *out;
        a.x += b.x;
        a.y += b.y;
        a.z += b.z;
        a.w += b.w;
      }
      *out = a;
    } else {
      for (int64_t e = i; e < min<int64_t>(cnt, i + V); ++e) {
        float a = src[e];
        for (int s = 1; s < splits; ++s) a += src[s * stride + e];
        y[e] = accumulate ? y[e] + a : a;
      }
    }
  }
}

// The tile shapes: row groups x weight rows, the workgroups that fit a CU, and
// the time (us) of a K step on a CU that runs one of them, and of each where
// several run.  Fitted, as are the costs of the partial sums below, to 3700
// timings of contractions on MI355X (12 groups of linears with k_up 960 to 24576
// and 700 to 28672 rows, m 17 to 2048, 1 to 16 splits): within 6 % for half of
// them (17-20 % low on the largest, where it does not matter to the choice).  Of
// nine shapes timed: 32 x 256 (many short tiles) up to a few hundred rows, 64 x
// 512 for large products (28672 x 16384 at m = 2048: 1204 us, 128 x 512 with a
// ring of five 1196, 128 x 256 1266, 256 x 256 1308, 32 x 256 1438), where wide
// tiles matter because x_tilde takes nine times the bytes of the codes.  128 x 512
// fills a CU's LDS with one workgroup, and the fit chose it next to never.
struct DigitShape {
  int rg, bn, per_cu;
  double step_us, step_each_us;
};
constexpr DigitShape kShapes[] = {
    {1, 256, 4, 0.273, 0.170},  // 4 waves, each 32 x 64
    {2, 512, 2, 0.680, 0.534},  // 4 waves, each 64 x 128
};
constexpr int kShapeCount = static_cast<int>(sizeof(kShapes) / sizeof(kShapes[0]));

// Estimated time of a plan (up to a constant).
double digit_plan_us(const DigitShape& s, int sp, int64_t tiles, int64_t steps, double outs, int64_t cus) {
  const int64_t on_cu = (tiles * sp + cus - 1) / cus;
  const int64_t full = on_cu / s.per_cu, rest = on_cu % s.per_cu;
  const double step = full * s.per_cu * s.step_each_us + (rest ? std::max(s.step_us, rest * s.step_each_us) : 0.0);
  return step * steps + (sp > 1 ? 2.1 + (sp + 1) * outs * 1.18e-6 : 0.0);
}

int64_t column_tiles(const int64_t* n, int count, int bn) {
  int64_t t = 0;
  for (int j = 0; j < count; ++j) t += (n[j] + bn - 1) / bn;
  return t;
}

int64_t part_floats(const int64_t* n, int count, int64_t m) {
  int64_t t = 0;
  for (int j = 0; j < count; ++j) t += (m * n[j] + 3) / 4 * 4;
  return t;
}

}  // namespace

DigitPlanes digit_planes(const sdq_layout* L, int64_t m, void* ws, size_t at) {
  DigitPlanes d;
  d.n_rg = (m + 31) / 32;
  d.n_steps = 2 * ((L->k_up + 127) / 128);
  d.row_fac = static_cast<float*>(ws);
  d.planes = static_cast<uint8_t*>(ws) + at;
  d.bytes = at + align_up(static_cast<size_t>(d.n_steps) * d.n_rg * kDigitTile, 256);
  return d;
}

// The split of the contraction.  SDQ_DIGIT_PLAN="shape,splits" asks for a plan (a
// tuning and test aid, read on every call), where K and the workspace allow it.
DigitPlan digit_plan(const int64_t* n, int count, int64_t k_up, int64_t m, size_t part_bytes) {
  const int64_t n_rg = (m + 31) / 32, pairs = (k_up + 127) / 128;
  const int64_t cus = device_compute_units();
  double outs = 0;
  for (int j = 0; j < count; ++j) outs += static_cast<double>(m) * n[j];
  const size_t one_part = static_cast<size_t>(part_floats(n, count, m)) * sizeof(float);
  DigitPlan best;
  double best_us = 1e30;
  int shape = -1, splits = -1;
  const char* env = std::getenv("SDQ_DIGIT_PLAN");
  if (env && std::sscanf(env, "%d,%d", &shape, &splits) == 2 && (shape < 0 || shape >= kShapeCount)) shape = -1;
  for (int i = 0; i < kShapeCount; ++i) {
    if (shape >= 0 && i != shape) continue;
    const int64_t tiles = (n_rg + kShapes[i].rg - 1) / kShapes[i].rg * column_tiles(n, count, kShapes[i].bn);
    for (int sp = 1; sp <= 16; ++sp) {
      const int64_t per = (pairs + sp - 1) / sp;
      if (sp > 1 && ((sp - 1) * per >= pairs || (tiles * (sp - 1) >= 4 * cus && shape < 0))) continue;
      if (sp > 1 && one_part * sp > part_bytes) break;
      const double us = digit_plan_us(kShapes[i], sp, tiles, 2 * per, outs, cus);
      if (us < best_us || (shape >= 0 && sp == splits)) {
        best_us = shape >= 0 && sp == splits ? 0.0 : us;
        best.shape = i;
        best.splits = sp;
        best.steps_per = static_cast<int>(2 * per);
        best.part_bytes = sp > 1 ? one_part * sp : 0;
      }
    }
  }
  return best;
}

sdq_status launch_digit_contract(int64_t m, LinearSet S, const sdq_layout* L, bool accumulate, void* ws, size_t at,
                                 void* part_ws, size_t part_bytes, bool by_form, hipStream_t stream) {
  const DigitPlanes d = digit_planes(L, m, ws, at);
  const float* form = by_form ? prefill_form(ws, m) : nullptr;
  const DigitPlan plan = digit_plan(S.n, S.count, L->k_up, m, part_bytes);
  const DigitShape& shape = kShapes[plan.shape];
  S.first[0] = 0;
  for (int j = 0; j < S.count; ++j) S.first[j + 1] = S.first[j] + (S.n[j] + shape.bn - 1) / shape.bn;
  for (int j = S.count + 1; j <= kMaxGroup; ++j) S.first[j] = S.first[S.count];
  const int64_t n_tiles = S.first[S.count];
  const int64_t m_tiles = (d.n_rg + shape.rg - 1) / shape.rg;
  DigitParts part;
  if (plan.splits > 1) {
    part.base = static_cast<float*>(part_ws);
    int64_t off = 0;
    for (int j = 0; j < S.count; ++j) {
      part.off[j] = off;
      part.stride[j] = (m * S.n[j] + 3) / 4 * 4;
      off += part.stride[j] * plan.splits;
    }
  }
  const int acc = accumulate && plan.splits == 1 ? 1 : 0;
  const dim3 grid(static_cast<unsigned>(m_tiles * n_tiles * plan.splits));
#define SDQ_DIG(LV, I, WM, WN, RT, CT, MINW)                                                             \
  case I:                                                                                                \
    static_assert(kShapes[I].rg == WM * RT && kShapes[I].bn == 32 * WN * CT, "shape");                   \
    gemm_digits_kernel<LV, WM, WN, RT, CT, MINW, APART><<<grid, dim3(64 * WM * WN), 0, stream>>>(        \
        d.planes, S, m, L->n_chunks, d.n_rg, static_cast<int>(d.n_steps), m_tiles, n_tiles,              \
        plan.steps_per, acc, part, form);                                                                \
    break
#define SDQ_DIG_SHAPES(LV)                                                                               \
  switch (plan.shape) {                                                                                  \
    SDQ_DIG(LV, 0, 1, 4, 1, 2, 4);                                                                       \
    SDQ_DIG(LV, 1, 1, 4, 2, 4, 2);                                                                       \
  }
  auto gemm = [&](auto apart) {
    constexpr bool APART = decltype(apart)::value;
    if (L->levels == 2) {
      SDQ_DIG_SHAPES(2)
    } else {
      SDQ_DIG_SHAPES(3)
    }
  };
  if (by_form) gemm(std::true_type{});
  else gemm(std::false_type{});
#undef SDQ_DIG_SHAPES
#undef SDQ_DIG
  if (plan.splits > 1) {
    int64_t most = 0;
    bool al = true;
    for (int j = 0; j < S.count; ++j) {
      most = std::max(most, m * S.n[j]);
      al = al && reinterpret_cast<uintptr_t>(S.y[j]) % 16 == 0;
    }
    const int v = al ? 4 : 1;
    const dim3 rgrid(static_cast<unsigned>(std::min<int64_t>((most + 256 * v - 1) / (256 * v), 4096)),
                     static_cast<unsigned>(S.count));
    auto reduce = al ? (by_form ? reduce_digits_kernel<4, true> : reduce_digits_kernel<4, false>)
                     : (by_form ? reduce_digits_kernel<1, true> : reduce_digits_kernel<1, false>);
    reduce<<<rgrid, dim3(256), 0, stream>>>(S, part, m, plan.splits, accumulate ? 1 : 0, form);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, "digit-plane GEMM launch");
  return SDQ_OK;
}

}  // namespace sdq

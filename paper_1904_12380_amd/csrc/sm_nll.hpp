// The negative log-likelihood kernels: one loss per row, nothing kept.
//
//   loss = ln S - max(x[label] - M, lo),   S = sum_j exp(max(x_j - M, lo))
//
// A loss needs the row's (max, sum) and one logit, so a row is streamed
// through registers and no value outlives its exponential: there is no limit
// on the row length, and the loads run a step ahead of the arithmetic.
//
//   k_nll_group   rows of at most 512 aligned strips (kNllGroupMaxStrips, about
//                 2048 columns): G lanes per row.
//   k_nll_rows    one wavefront (NT = 64) or one workgroup per row.
//   k_nll_split   a few long rows: each cut into equal chunks, one workgroup
//                 per chunk, the last of a row's workgroups to finish merges.
//
// All of them are bound by HBM reads (4 bytes per element).  Rows may start
// at any 4-byte address: 128-bit loads cover the aligned strips, and the up
// to three columns before and after them are masked (k_nll_group) or read as
// single elements.  Measured per call (graph replay over rotated inputs,
// before -> after this split of the work): 16384 x 50001 971 -> 482 us
// (6.8 TB/s), 335 x 50001 25.5 -> 16.3, 8188 x 2049 43.9 -> 13.1,
// 4 x 4194304 32.6 -> 15.0, 167772 x 100 38.6 -> 13.4, 129055 x 130
// 31.5 -> 13.4.  The old path held rows in registers, read rows that are not
// whole 16-byte strips 32 bits at a time, and took rows over 2^21 columns in
// two passes.
//
// The clip and the sum: an element with x - M < lo adds e^lo instead of
// e^(x - M).  With lo <= -48 and S >= 1 the two differ by under 1.5e-21 S,
// so the sums here leave the clip out (the label's own logit keeps it).
// -inf adds 0, a NaN or +inf element makes S NaN.
#pragma once

#include "sm_kernels.hpp"

namespace smx {

// exp(d) for d <= 0 (or NaN), within the fast exponential's bound
// (kExpFast): the sum terms.
__device__ __forceinline__ float nll_term(float x, float m) {
  return __builtin_amdgcn_exp2f((x - m) * 0x1.715476p+0f);
}

// exp(m - m_new) for m <= m_new within 1.5 ulp (0 below about -87), for
// rescaling partial sums: the difference and the argument in binary64 as in
// exp_shift_clip (a difference rounded to fp32 is off by up to |d| 2^-24, which
// the exponential turns into that relative error of the sum).
__device__ __forceinline__ float nll_rescale(float m, float m_new) {
  const double d = fmax(static_cast<double>(m) - static_cast<double>(m_new), -126.0);
  const float th = static_cast<float>(d * kLog2e);
  const double r = __builtin_fma(static_cast<double>(th), -kLn2, d);
  const float e0 = __builtin_amdgcn_exp2f(th);
  return __builtin_fmaf(e0, static_cast<float>(r), e0);
}

// c in scalar registers, formed where it is used: the compiler otherwise keeps
// the constants below in vector registers across the loops around them (10
// more, one wavefront per SIMD less).
__device__ __forceinline__ double scalar_here(double c) {
  asm volatile("" : "+s"(c));
  return c;
}

// exp(d) for -126 <= d <= 0 in binary64, within 1e-11 relative:
// d = n ln 2 + 16 q with |q| <= ln 2 / 32, e^q by its Taylor series to q^5
// (truncated at q^6 / 720 < 2e-13), squared four times, times 2^n.
__device__ __forceinline__ double exp_rescale(double d) {
  const double n = __builtin_rint(d * scalar_here(kLog2e));
  const double q = __builtin_fma(n, scalar_here(-kLn2), d) * 0x1p-4;
  double e = __builtin_fma(q, scalar_here(1.0 / 120), scalar_here(1.0 / 24));
  e = __builtin_fma(q, e, scalar_here(1.0 / 6));
  e = __builtin_fma(q, e, 0.5);
  e = __builtin_fma(q, e, 1.0);
  e = __builtin_fma(q, e, 1.0);
  e *= e;
  e *= e;
  e *= e;
  e *= e;
  return __builtin_ldexp(e, static_cast<int>(n));
}

// A lane's running max m and sum s of exp(x - m); a lane that has seen only
// -inf has m = -inf, s = 0.  A lane takes one step after another, thousands on
// a long row that is not split, so the sum and its rescaling are binary64: in
// fp32, steps that look alike round alike, and 384 x 4194304 (1024 steps) was
// off by 1.5e-5 on logits that repeat with the step and 1.3e-5 on logits that
// rise steadily, above the stated bound.  The exponential of a rescaling runs
// only where a lane's max has grown.
struct RunningSum {
  float m = kNegInf;
  double s = 0.0;

  // Brings m to m_new, the max with the next step's logits (called before
  // their exponentials: fewer registers).
  __device__ __forceinline__ void grow(float m_new) {
    if (m < m_new)
      s *= exp_rescale(fmax(static_cast<double>(m) - static_cast<double>(m_new), -126.0));
    m = m_new;
  }
  // The sum against the row's max m_row.
  __device__ __forceinline__ float share(float m_row) const {
    return static_cast<float>(s) * nll_rescale(m, m_row == kNegInf ? 0.0f : m_row);
  }
};

struct NllSum : RunningSum {
  template <int N>
  __device__ __forceinline__ void add(const float (&v)[N]) {
    grow(fmaxf(m, array_max(v)));
    const float ref = m == kNegInf ? 0.0f : m;
    float t[8];
#pragma unroll
    for (int i = 0; i < N; ++i)
      t[i % 8] = i < 8 ? nll_term(v[i], ref) : t[i % 8] + nll_term(v[i], ref);
    s += static_cast<double>(tree_sum(t));
  }
};

// The loss from the row's max and sum and the label's logit.
__device__ __forceinline__ float nll_loss(float xl, bool bad, float m, float s, Clip clip) {
  return bad ? __builtin_nanf("") : -log_out(xl, row_shift(m, clip), log_of_sum(s));
}

// The lane's share of the segment p[0, n): thread t of NT.  Whole aligned
// 16-byte strips, U per lane and step, the next step's loads issued
// before this step is folded in (Sum::add); the up to six columns outside them
// go one each to the first threads.  `after_first` runs once the first step's
// loads are issued (the label's logit is loaded there: before them, the loads
// would wait for the label).  NTL: streaming loads.
template <int NT, int U, bool NTL, typename Sum, typename F>
__device__ __forceinline__ Sum stream_sum(const float* p, int64_t n, int t, F after_first) {
  const int64_t to_aligned = (4 - ((reinterpret_cast<uintptr_t>(p) >> 2) & 3)) & 3;
  const int64_t head = to_aligned < n ? to_aligned : n;
  const float* ps = p + head;
  const int64_t strips = (n - head) >> 2;
  const int tail = static_cast<int>((n - head) & 3);
  // One edge column per thread: the head's, then the tail's.
  float edge = kNegInf;
  if (t < head) edge = p[t];
  if (t >= head && t - head < tail) edge = ps[4 * strips + t - head];
  Sum acc;
  acc.m = fmaxf(acc.m, edge);
  acc.s = edge == kNegInf ? 0.0 : 1.0 + (edge - edge);  // NaN for a NaN or +inf edge
  f32x4 q[U];
  auto ld = [](const float* a) {
    return NTL ? ld_stream(a) : *reinterpret_cast<const f32x4*>(a);
  };
  auto load = [&](int64_t i0) {
    const float* pi = ps + 4 * i0;  // uniform base, 32-bit lane offsets
    if (i0 + NT * U <= strips) {
#pragma unroll
      for (int u = 0; u < U; ++u) q[u] = ld(pi + 4 * (t + NT * u));
    } else {
      const int left = static_cast<int>(strips - i0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        q[u] = f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
        if (t + NT * u < left) q[u] = ld(pi + 4 * (t + NT * u));
      }
    }
  };
  if (strips > 0) load(0);
  __builtin_amdgcn_sched_barrier(0);
  after_first();
  for (int64_t i0 = 0; i0 < strips; i0 += NT * U) {
    float v[4 * U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[4 * u + 0] = q[u].x;
      v[4 * u + 1] = q[u].y;
      v[4 * u + 2] = q[u].z;
      v[4 * u + 3] = q[u].w;
    }
    if (i0 + NT * U < strips) load(i0 + NT * U);
    acc.add(v);
  }
  return acc;
}

template <int NT, int U, typename F>
__device__ __forceinline__ NllSum nll_stream(const float* p, int64_t n, int t, F after_first) {
  return stream_sum<NT, U, true, NllSum>(p, n, t, after_first);
}

// (m, s) over the NT threads' shares; the same bits on every thread.
template <int NT>
__device__ __forceinline__ float2 nll_combine(NllSum a, float* red_max, float* red_sum) {
  const float m = block_max<NT / 64>(a.m, red_max);
  return make_float2(m, block_sum<NT / 64>(a.share(m), red_sum));
}

// One wavefront (NT = 64, four rows per workgroup) or one workgroup of NT
// threads per row.
template <int NT, int U>
__global__ __launch_bounds__(NT < 256 ? 256 : NT)
    __attribute__((amdgpu_waves_per_eu(NT == 64 ? 7 : 8))) void k_nll_rows(
        const float* x, const int64_t* labels, float* y, int64_t rows, int64_t cols, Clip clip) {
  constexpr int kRows = NT == 64 ? 4 : 1;  // rows per workgroup
  __shared__ float red_max[NT / 64];
  __shared__ float red_sum[NT / 64];
  const int t = NT == 64 ? __lane_id() : threadIdx.x;
  const int w = NT == 64 ? __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6) : 0;
  for (int64_t row = static_cast<int64_t>(blockIdx.x) * kRows + w; row < rows;
       row += static_cast<int64_t>(gridDim.x) * kRows) {
    const float* xr = x + row * cols;
    const int64_t label = labels[row];
    const bool bad = label < 0 || label >= cols;
    float xl;
    const NllSum own = nll_stream<NT, U>(xr, cols, t, [&] { xl = xr[bad ? 0 : label]; });
    const float2 ms = nll_combine<NT>(own, red_max, red_sum);
    if (t == 0) y[row] = nll_loss(xl, bad, ms.x, ms.y, clip);
  }
}

// G lanes per row, the whole row in U strips per lane: the aligned strips
// around the row, columns outside it replaced by -inf (they lie in the same
// 16-byte blocks as the row's ends).  G * U strips cover the row with its
// phase (cols + 3 columns, or cols where every row starts on a 16-byte
// boundary) and G * (U - 1) do not, and phases move a row's end by at most
// one strip: only the first and the last two strips of a lane can hold
// columns outside the row.
//
// With G <= 16 a load instruction covers pieces of 4 or more rows, and the
// piece beside each of them is taken by the next one: those loads keep their
// lines in the cache (a 64 MiB call on 100 columns took 13.4 us against 16.6
// with streaming loads, 130 columns 13.4 against 16.8, 255 columns 13.0
// against 13.8).  With G >= 32 streaming loads were level or faster.
template <int G, int U>
__global__ __launch_bounds__(256) void k_nll_group(const float* x, const int64_t* labels,
                                                   float* y, int64_t rows, int64_t cols,
                                                   Clip clip) {
  constexpr int R = 64 / G;
  const int lane = __lane_id();
  const int j = lane % G;
  const int lim = static_cast<int>(cols);
  // Every row starts on a 16-byte boundary: no strip straddles a row's end.
  const bool whole = (reinterpret_cast<uintptr_t>(x) & 15) == 0 && lim % 4 == 0;
  const int64_t step = static_cast<int64_t>(gridDim.x) * 4 * R;
  for (int64_t r0 = (static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6)) * R; r0 < rows;
       r0 += step) {
    const int64_t row = r0 + lane / G;
    const bool ok = row < rows;
    const float* xr = x + (ok ? row : r0) * cols;
    const int a = static_cast<int>((reinterpret_cast<uintptr_t>(xr) >> 2) & 3);
    const int64_t label = labels[ok ? row : r0];
    float v[4 * U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c0 = 4 * (j + G * u) - a;
      f32x4 q = f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
      if (c0 < lim) q = G <= 16 ? *reinterpret_cast<const f32x4*>(xr + c0) : ld_stream(xr + c0);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * u + i] = q[i];
    }
    if (!whole) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u > 0 && u < U - 2) continue;
        const int c0 = 4 * (j + G * u) - a;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool in = static_cast<unsigned>(c0 + i) < static_cast<unsigned>(lim);
          v[4 * u + i] = in ? v[4 * u + i] : kNegInf;
        }
      }
    }
    const bool bad = label < 0 || label >= cols;
    const float xl = xr[bad ? 0 : label];
    const float m = seg_max<G>(array_max(v));
    // Eight interleaved partial sums, as the log outputs take them
    // (exp_strip): where both modes hold a row alike, the loss is minus the
    // log output bit for bit.
    float t[8];
#pragma unroll
    for (int i = 0; i < 4 * U; ++i) t[i % 8] = i < 8 ? nll_term(v[i], m) : t[i % 8] + nll_term(v[i], m);
    const float s = seg_sum<G>(tree_sum(t));
    if (ok && j == 0) y[row] = nll_loss(xl, bad, m, s, clip);
  }
}

// A few rows: workgroup (row, g) takes the chunk [g * chunk, (g + 1) * chunk)
// of its row (chunk a multiple of 4, at most 64 chunks).  It publishes its
// pair in the row's exchange entry and counts itself out; the one that brings
// the count to the row's chunks merges the pairs and writes the loss.  No
// workgroup waits for another one (see sm_exchange.hpp for the entry).
template <int NT, int U>
__global__ __launch_bounds__(NT) void k_nll_split(const float* x, const int64_t* labels,
                                                  float* y, XchArgs xa, int64_t cols,
                                                  int chunks, int64_t chunk, Clip clip) {
  const uint64_t t0 = wall_clock();
  __shared__ float red_max[NT / 64];
  __shared__ float red_sum[NT / 64];
  const int tid = threadIdx.x;
  const int lrow = blockIdx.x / chunks;
  const int g = blockIdx.x - lrow * chunks;
  const float* xr = x + lrow * cols;
  const int64_t c0 = g * chunk;
  const int64_t n = cols - c0 < chunk ? cols - c0 : chunk;
  const int64_t label = labels[lrow];
  const bool bad = label < 0 || label >= cols;
  float xl;
  const NllSum own = nll_stream<NT, U>(xr + c0, n, tid, [&] { xl = xr[bad ? 0 : label]; });
  const float2 part = nll_combine<NT>(own, red_max, red_sum);
  if (tid >= 64) return;
  const uint64_t deadline = t0 + xa.limit_ticks;
  uint64_t* const entry = wave_entry(xa, lrow, deadline);
  if (entry == nullptr) {
    if (tid == 0) y[lrow] = __builtin_nanf("");
    return;
  }
  uint64_t* const slots = entry_slots(entry);
  uint32_t last = 0;
  if (tid == 0) {
    xch::st_agent(&slots[g], encode_pair(part.x, part.y));
    // The pair is stored before it is counted, so the workgroup that brings
    // the count to the row's chunks finds every pair.
    __builtin_amdgcn_s_waitcnt(0);
    last = depart_entry(entry, chunks, 1u) ? 1u : 0u;
  }
  last = __builtin_amdgcn_readfirstlane(last);
  if (!last) return;
  // A slot that still reads empty is read again (bounded), so the merge does
  // not rest on when a completed store becomes visible.
  bool ok = true;
  const uint64_t q = poll_slots(slots, chunks, deadline, &ok);
  const float pm = tid < chunks ? decode_m(q) : kNegInf;
  const float ps = tid < chunks ? decode_s(q) : 0.0f;
  const float m = seg_max<64>(pm);
  const float s = seg_sum<64>(ps * nll_rescale(pm, m == kNegInf ? 0.0f : m));
  const float loss = nll_loss(xl, bad || !ok, m, s, clip);
  if (tid == 0) {
    y[lrow] = loss;
    if (!ok) count_give_up(xa, xch::kDiagWaitGiveUps);
  }
  // The slot reads have returned (the loss depends on them).
  asm volatile("" : : "v"(loss));
  if (tid < chunks) xch::st_agent(&slots[tid], 0ull);
  if (tid == 0) release_entry(entry);
}

}  // namespace smx

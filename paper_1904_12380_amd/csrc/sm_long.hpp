// Rows too long for a one-pass launch (a row of them does not fit in the
// registers of the workgroups that can meet at one exchange entry): two
// kernels per group of rows, both streaming.
//
//   k_long_stats  wpr workgroups per row, each leaving the (max, sum) of an
//                 equal chunk of the row in a slot of one of the row's
//                 exchange entries (kEntrySlots workgroups to an entry; a row
//                 holds up to kLongMaxEntries consecutive ones).
//   k_long_apply  the same workgroups per row: each merges the row's slots,
//                 streams its chunk again and writes the outputs; the last of
//                 the row's workgroups releases the entries.
//
// Bound by memory: x crosses twice, y once.  The host groups rows so that a
// group's x stays in the memory-side cache between the two kernels: the first
// reads x with plain loads, which leave it there, the second reads it from
// there while HBM takes the writes.  Measured against the two passes before it
// (64 workgroups per row, chunks held in registers one after another):
// 8 x 4194304 81 -> 71 us (26.7 + 43.6, 6.1 TB/s in the second kernel),
// 1 x 4194304 37 -> 18.7, 1 x 33554432 277 -> 75, 8 x 2000001 56 -> 40.6,
// 20 x 2500000 130 -> 108.  No workgroup waits for another one of its
// own kernel.  Rows may start at any 4-byte address: 128-bit loads and, where
// x and y have the same phase, stores on the aligned strips, single columns
// around them.
#pragma once

#include "sm_nll.hpp"

namespace smx {

// A lane's running max and sum of exp(x - m) with the accurate exponential
// (log outputs: the fast one, as their other row sums).  Unclipped, as
// NllSum: a clipped term is under 1.5e-21 of a row sum.
template <int MODE>
struct LongSum : RunningSum {
  __device__ __forceinline__ static float term(float x, RowShift rs) {
    if constexpr (MODE == kLogOut || MODE == kExpFast)
      return nll_term(x, rs.m);
    else
      return exp_shift_clip<kExpAccurate>(x, rs);
  }
  // The shift of a max (0 while it is -inf), clipped terms dropped.
  __device__ __forceinline__ static RowShift shift(float m) {
    return row_shift(m == kNegInf ? 0.0f : m, Clip{kClipFloor, 0.0f, kClipFloor});
  }
  template <int N>
  __device__ __forceinline__ void add(const float (&v)[N]) {
    grow(fmaxf(m, array_max(v)));
    const RowShift rs = shift(m);
    float t[8];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i % 8] = i < 8 ? term(v[i], rs) : t[i % 8] + term(v[i], rs);
    s += static_cast<double>(tree_sum(t));
  }
};

constexpr int kLongThreads = 512;
constexpr int kLongStrips = 4;  // strips per lane and step
constexpr int kLongMaxEntries = 16;  // exchange entries of a row

template <int NT, int MODE>
__global__ __launch_bounds__(NT) void k_long_stats(const float* x, XchArgs xa, int64_t cols,
                                                   int wpr, int entries, int64_t chunk) {
  const uint64_t t0 = wall_clock();
  __shared__ float red_max[NT / 64];
  __shared__ float red_sum[NT / 64];
  const int tid = threadIdx.x;
  const int lrow = blockIdx.x / wpr;
  const int w = blockIdx.x - lrow * wpr;
  const int64_t c0 = w * chunk;
  const int64_t n = cols - c0 < chunk ? cols - c0 : chunk;
  const LongSum<MODE> own =
      stream_sum<NT, kLongStrips, false, LongSum<MODE>>(x + lrow * cols + c0, n, tid, [] {});
  const float m = block_max<NT / 64>(own.m, red_max);
  const float s = block_sum<NT / 64>(own.share(m), red_sum);
  if (tid < 64) {
    uint64_t* entry =
        wave_entry(xa, lrow * entries + w / xch::kEntrySlots, t0 + xa.limit_ticks);
    if (tid == 0 && entry != nullptr)
      xch::st_agent(&entry_slots(entry)[w % xch::kEntrySlots], encode_pair(m, s));
  }
}

// Puts entry `e` of the launch back to rest, its first `slots` slots (at most
// kEntrySlots) zeroed; by one wavefront, once nothing reads the entry.
__device__ __forceinline__ void release_long_entry(const XchArgs& xa, int e, int slots) {
  uint64_t* const entry = find_entry(xa, e);
  if (__lane_id() < slots) xch::st_agent(&entry_slots(entry)[__lane_id()], 0ull);
  if (__lane_id() == 0) release_entry(entry);
}

template <int NT, int MODE>
__global__ __launch_bounds__(NT) void k_long_apply(const float* x, float* y, XchArgs xa,
                                                   int64_t cols, int wpr, int entries,
                                                   int64_t chunk, Clip clip) {
  constexpr int U = kLongStrips;
  __shared__ float bcast[2];
  const int tid = threadIdx.x;
  const int lane = __lane_id();
  const int lrow = blockIdx.x / wpr;
  const int w = blockIdx.x - lrow * wpr;
  // Wavefront 0: the row's entries checked, one lane each (k_long_stats has
  // ended, so each holds the row or never will), and its slots merged.
  bool found = false;
  if (tid < 64) {
    const bool mine =
        lane >= entries || xch::ld_agent(find_entry(xa, lrow * entries + lane)) ==
                               row_tag(xa, lrow * entries + lane);
    found = __builtin_amdgcn_ballot_w64(!mine) == 0;
    if (!found && tid == 0) count_give_up(xa, xch::kDiagJoinGiveUps);
    uint64_t q[kLongMaxEntries];
#pragma unroll
    for (int k = 0; k < kLongMaxEntries; ++k) {
      q[k] = encode_pair(kNegInf, 0.0f);
      if (found && k * xch::kEntrySlots + lane < wpr)
        q[k] = xch::ld_agent(&entry_slots(find_entry(xa, lrow * entries + k))[lane]);
    }
    float m = decode_m(q[0]);
#pragma unroll
    for (int k = 1; k < kLongMaxEntries; ++k) m = fmaxf(m, decode_m(q[k]));
    m = seg_max<64>(m);
    // In binary64: one rounding here is the same in all of the row's outputs.
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kLongMaxEntries; ++k)
      s += static_cast<double>(decode_s(q[k])) *
           static_cast<double>(nll_rescale(decode_m(q[k]), m == kNegInf ? 0.0f : m));
    s = wave_sum64(s);
    if (tid == 0) {
      const float last = MODE == kLogOut ? log_of_sum(static_cast<float>(s))
                                         : static_cast<float>(1.0 / s);
      bcast[0] = found ? m : __builtin_nanf("");
      bcast[1] = found ? last : __builtin_nanf("");
    }
  }
  __syncthreads();
  const RowShift rs = row_shift(bcast[0], clip);
  const float scale = bcast[1];  // ln S or 1 / S
  auto out = [&](float xv) {
    if constexpr (MODE == kLogOut)
      return log_out(xv, rs, scale);
    else
      return exp_shift_clip<MODE>(xv, rs) * scale;
  };

  const int64_t c0 = w * chunk;
  const int64_t n = cols - c0 < chunk ? cols - c0 : chunk;
  const float* p = x + lrow * cols + c0;
  float* o = y + lrow * cols + c0;
  const int64_t to_aligned = (4 - ((reinterpret_cast<uintptr_t>(p) >> 2) & 3)) & 3;
  const int64_t head = to_aligned < n ? to_aligned : n;
  const int64_t strips = (n - head) >> 2;
  const int tail = static_cast<int>((n - head) & 3);
  const bool same = ((reinterpret_cast<uintptr_t>(p) ^ reinterpret_cast<uintptr_t>(o)) & 15) == 0;
  if (tid < head) o[tid] = out(p[tid]);
  if (tid >= head && tid - head < tail) {
    const int64_t c = head + 4 * strips + tid - head;
    o[c] = out(p[c]);
  }
  const float* ps = p + head;
  float* os = o + head;
  f32x4 q[U];
  auto load = [&](int64_t i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + tid + NT * u;
      if (i < strips) q[u] = *reinterpret_cast<const f32x4*>(ps + 4 * i);
    }
  };
  load(0);
  for (int64_t i0 = 0; i0 < strips; i0 += NT * U) {
    f32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = q[u];
    load(i0 + NT * U);  // nothing past the chunk
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + tid + NT * u;
      const f32x4 e = {out(v[u].x), out(v[u].y), out(v[u].z), out(v[u].w)};
      if (i < strips) {
        if (same) {
          st_stream(os + 4 * i, e);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) __builtin_nontemporal_store(e[k], os + 4 * i + k);
        }
      }
    }
  }
  if (found) {
    // The slot reads have returned (the outputs above depend on them).  The
    // row's workgroups count themselves out in two steps, by entry and then
    // entry by entry out of the first one (counts on one address take about
    // 70 ns each, one after another).
    const int mine = w % entries;
    const int group = wpr / entries + (mine < wpr % entries ? 1 : 0);
    uint32_t last = 0;
    if (tid == 0) {
      uint64_t* const e = find_entry(xa, lrow * entries + mine);
      if (depart_entry(e, group, 1u)) {
        uint32_t* const total = reinterpret_cast<uint32_t*>(find_entry(xa, lrow * entries) + 2);
        last = xch::add_agent32(total, 1u) == static_cast<uint32_t>(entries) - 1u ? 1u : 0u;
        if (last) __hip_atomic_store(total, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    last = __builtin_amdgcn_readfirstlane(last);
    if (last) {
      for (int k = 0; k < entries; ++k)
        release_long_entry(xa, lrow * entries + k, wpr - k * xch::kEntrySlots);
    }
  } else if (tid < 64 && w == 0) {
    // The row lacks an entry, which k_long_stats could not join in time: all of
    // the row's workgroups see that (the entry cannot gain the row's tag any
    // more), so none of them reads a slot or counts itself out, and the row's
    // first one gives back the entries that the row did claim.
    for (int k = 0; k < entries; ++k) {
      const int e = lrow * entries + k;
      if (xch::ld_agent(find_entry(xa, e)) == row_tag(xa, e))
        release_long_entry(xa, e, wpr - k * xch::kEntrySlots);
    }
  }
}

}  // namespace smx

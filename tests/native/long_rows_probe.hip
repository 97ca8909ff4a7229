// The two kernels of rows in two passes over an exchange table that the caller
// owns, so that a test can hold an entry and look at the table afterwards.
// Launched as run_plan() does for one group of rows (softmax_api.hip).
#include "../../paper_1904_12380_amd/csrc/sm_long.hpp"

#define PROBE_API extern "C" __attribute__((visibility("default")))

PROBE_API int64_t probe_scratch_words() { return smx::xch::kScratchWords; }
PROBE_API int64_t probe_entry_words() { return smx::xch::kEntryWords; }
PROBE_API int64_t probe_entries() { return smx::xch::kEntries; }

// Softmax of `rows` rows in `wpr` workgroups each of `chunk` columns; 0 or the
// HIP error.
PROBE_API int probe_long_rows(const float* x, float* y, uint64_t* scratch, uint64_t key,
                              uint32_t base, int64_t rows, int64_t cols, int wpr, int64_t chunk,
                              uint32_t limit_ticks, hipStream_t stream) {
  using namespace smx;
  if (rows < 1 || wpr < 1 || chunk < 4 || chunk % 4 != 0 || (wpr - 1) * chunk >= cols ||
      wpr * chunk < cols || wpr > kLongMaxEntries * xch::kEntrySlots)
    return -1;
  const int entries = (wpr + xch::kEntrySlots - 1) / xch::kEntrySlots;
  if (rows * entries > xch::kMaxRowsPerLaunch) return -1;
  const Clip clip{kClipLo, kExpClipLo, kClipLo};
  const uint32_t grid = static_cast<uint32_t>(rows * wpr);
  const XchArgs xa{scratch, key, limit_ticks, base};
  k_long_stats<kLongThreads, kExpAccurate>
      <<<grid, kLongThreads, 0, stream>>>(x, xa, cols, wpr, entries, chunk);
  k_long_apply<kLongThreads, kExpAccurate>
      <<<grid, kLongThreads, 0, stream>>>(x, y, xa, cols, wpr, entries, chunk, clip);
  return static_cast<int>(hipGetLastError());
}

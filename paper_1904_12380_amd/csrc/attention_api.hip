// C ABI of the fused softmax attention: argument checks and the launch.
// Declaration and contract: include/softmax_mi355x.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>

#include "../../include/softmax_mi355x.h"
#include "sm_attention.hpp"
#include "sm_attention_wave.hpp"
#include "sm_host.hpp"

namespace {

using namespace smx;
using namespace smx_host;

// sizes: all >= 0, lk in [1, 64] when there is work, d and dv at most
// SOFTMAX_ATTN_MAX_DIM, and every tensor's byte count fits in int64.
int check_attention_sizes(int64_t batch, int64_t lq, int64_t lk, int64_t d, int64_t dv) {
  if (batch < 0 || lq < 0 || lk < 0 || d < 0 || dv < 0) return SOFTMAX_ERR_INVALID_ARG;
  if (lq > INT32_MAX / 2 || d > SOFTMAX_ATTN_MAX_DIM || dv > SOFTMAX_ATTN_MAX_DIM)
    return SOFTMAX_ERR_INVALID_ARG;
  if (lk > SOFTMAX_ATTN_MAX_KEYS) return SOFTMAX_ERR_INVALID_ARG;
  if (batch == 0 || lq == 0 || dv == 0) return SOFTMAX_OK;
  if (lk == 0) return SOFTMAX_ERR_INVALID_ARG;
  const int64_t per_q = lq * std::max<int64_t>(d, dv);
  const int64_t per_k = lk * std::max<int64_t>(d, dv);
  if (batch > INT64_MAX / 4 / std::max(per_q, per_k)) return SOFTMAX_ERR_INVALID_ARG;
  return SOFTMAX_OK;
}

// The DAM tile (d = dv = 200, 49 or 50 keys) with d known at compile time,
// on the ping-pong schedule: one workgroup of 8 wavefronts per CU, 160 KiB
// of LDS (two buffers of K_b, V_b and a zero row).  The kernel scores the
// last key tile on the VALU and needs at most 2 keys there.
constexpr int kAttnDamDim = 200;

bool dam_tile(int lk, int d, int dv) {
  return d == kAttnDamDim && dv == kAttnDamDim && lk > 48 && lk <= 50 &&
         (lk * (d + dv) + dv + 16) * 4 <= kAttnLdsBytes;
}

template <bool WIDE>
hipError_t run_attention_dam(const float* q, const float* k, const float* v, float* o,
                             int64_t batch, int lq, int lk, int d, int dv, float scale, Clip c,
                             int64_t cus, hipStream_t s) {
  const int64_t items = batch * ((lq + 63) / 64);
  const int64_t grid = std::min(items, cus);
  void* args[] = {&q, &k, &v, &o, &batch, &lq, &lk, &d, &dv, &scale, &c};
  return launch(reinterpret_cast<const void*>(&k_attention_pp<4, WIDE, kAttnDamDim>), grid, 512,
                args, s);
}

// ---------------------------------------------------------------------------
// One wavefront per block of queries (sm_attention_wave.hpp): everything but
// the DAM tile.

// Instances: NQ x NK x access (rows of whole 128-byte lines read once: nt
// loads; other rows of whole 16-byte strips; other rows; and the last two with
// plain stores, for up to kAttnPlainMaxKeyTiles key tiles).
enum WaveAccess { kWaveStream, kWaveWhole, kWaveRagged, kWaveWholePlain, kWaveRaggedPlain };
constexpr int kWaveAccesses = 5;

// Outputs of at least this many bytes, in rows that are not whole 32-byte
// sectors, are stored without the nontemporal policy where few enough keys
// leave the stores the larger part of the work (up to kAttnPlainMaxKeyTiles
// key tiles, from kAttnPlainMinDv columns): a row's neighbouring blocks then
// meet in the L2 instead of leaving it as partial sectors.  64 x 512 x 16 x 8 x
// 604 40.2 -> 26.6 us, 147 x 1401 x 13 x 8 x 94 45.3 -> 29.1, 421 x 76 x 40 x 408
// x 769 100.8 -> 92.4; but with 64 keys 64 x 512 x 64 x 8 x 604 45.0 -> 49.1, on
// 38 MiB 64 x 256 x 48 x 8 x 604 21.8 -> 23.7, on 58 columns 42.9 -> 48.1.
constexpr int64_t kAttnPlainMinBytes = int64_t(64) << 20;
constexpr int kAttnPlainMaxKeyTiles = 3;
constexpr int kAttnPlainMinDv = 64;

template <int NQ, int NK>
const void* wave_fn_access(WaveAccess access) {
  auto cast = [](auto f) { return reinterpret_cast<const void*>(f); };
  if constexpr (NK <= kAttnPlainMaxKeyTiles) {
    if (access == kWaveWholePlain) return cast(&k_attention_wave<NQ, NK, false, false, true>);
    if (access == kWaveRaggedPlain) return cast(&k_attention_wave<NQ, NK, true, false, true>);
  }
  switch (access) {
    case kWaveStream: return cast(&k_attention_wave<NQ, NK, false, true, false>);
    case kWaveWhole: return cast(&k_attention_wave<NQ, NK, false, false, false>);
    default: return cast(&k_attention_wave<NQ, NK, true, false, false>);
  }
}

template <int NQ>
const void* wave_fn_nk(int nk, WaveAccess access) {
  switch (nk) {
    case 1: return wave_fn_access<NQ, 1>(access);
    case 2: return wave_fn_access<NQ, 2>(access);
    case 3: return wave_fn_access<NQ, 3>(access);
    default: return wave_fn_access<NQ, 4>(access);
  }
}

const void* wave_fn(int nq, int nk, WaveAccess access) {
  switch (nq) {
    case 1: return wave_fn_nk<1>(nk, access);
    case 2: return wave_fn_nk<2>(nk, access);
    default: return wave_fn_nk<3>(nk, access);
  }
}

// Query tiles per wavefront: two (each K and V operand serves two matrix
// ops), or three for 33 to 48 queries, where two would leave one of four tiles
// empty (4096 x 33 x 37 x 50 x 50 33 us against 43).  Four tiles measured
// level on 64 queries at 8192 items and 2-30% slower below (1024 x 64 x 64 x
// 64 x 64 20.2 us against 16.9).  Fewer while that would leave fewer than
// kAttnMinWavesPerCU wavefronts per CU: 256 x 64 x 64 x 64 x 64 ran 7.6 us
// with one tile (1024 wavefronts) and 10.2 with two (512).
constexpr int64_t kAttnMinWavesPerCU = 4;

// Resident workgroups per CU of an instance, from the runtime's occupancy
// calculator (the same on every gfx950 device), once per instance.
std::atomic<int> g_wave_per_cu[3][4][kWaveAccesses][2];

int wave_per_cu(const void* fn, int nq, int nk, WaveAccess access, int waves, int* out) {
  std::atomic<int>& slot = g_wave_per_cu[nq - 1][nk - 1][access][waves > 1];
  int n = slot.load(std::memory_order_relaxed);
  if (n == 0) {
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, 64 * waves, 0);
    if (e != hipSuccess) return fail_hip(e);
    if (n <= 0) return SOFTMAX_ERR_HIP;
    slot.store(n, std::memory_order_relaxed);
  }
  *out = n;
  return SOFTMAX_OK;
}

int run_attention_wave(const float* q, const float* k, const float* v, float* o, int64_t batch,
                       int lq, int lk, int d, int dv, float scale, Clip c, int64_t cus,
                       hipStream_t s) {
  auto blocks = [&](int n) { return batch * ((lq + 16 * n - 1) / (16 * n)); };
  const int tiles = (lq + 15) / 16;
  int nq = tiles == 3 ? 3 : std::min(tiles, 2);
  while (nq > 1 && blocks(nq) < kAttnMinWavesPerCU * cus) --nq;
  const int nk = (lk + 15) / 16;
  const int64_t items = blocks(nq);
  const bool plain = dv % 8 != 0 && dv >= kAttnPlainMinDv && nk <= kAttnPlainMaxKeyTiles &&
                     batch * lq * dv * 4 >= kAttnPlainMinBytes;
  const WaveAccess access = d % 4 != 0 ? (plain ? kWaveRaggedPlain : kWaveRagged)
                            : plain    ? kWaveWholePlain
                            : items == batch && d % 32 == 0 && dv % 32 == 0 ? kWaveStream
                                                                            : kWaveWhole;
  const void* fn = wave_fn(nq, nk, access);
  // Four wavefronts per workgroup share a batch element's K and V through
  // their CU's cache; at most one item per CU takes a CU each (100 x 16 x 50 x
  // 200 x 200 ran 13.4 us so, 17.8 on 25 CUs).
  const int waves = items <= cus ? 1 : 4;
  int per_cu = 0;
  const int rc = wave_per_cu(fn, nq, nk, access, waves, &per_cu);
  if (rc != SOFTMAX_OK) return rc;
  // Resident workgroups only, each looping over items: the next item's first
  // operands load during this one's softmax and value product.
  const int64_t grid = std::min(ceil_div(items, waves), int64_t(per_cu) * cus);
  void* args[] = {&q, &k, &v, &o, &batch, &lq, &lk, &d, &dv, &scale, &c};
  const hipError_t e = launch(fn, grid, 64 * waves, args, s);
  return e == hipSuccess ? SOFTMAX_OK : fail_hip(e);
}

}  // namespace

extern "C" {

SOFTMAX_API int softmax_attention_fwd(const float* q, const float* k, const float* v,
                                      float* o, int64_t batch, int64_t lq, int64_t lk,
                                      int64_t d, int64_t dv, float scale, float clip_lo,
                                      hipStream_t stream) {
  Clip c;
  bool wide = false;
  int rc = make_clip(clip_lo, &c, &wide);
  if (rc != SOFTMAX_OK) return rc;
  if (!std::isfinite(scale)) return SOFTMAX_ERR_INVALID_ARG;
  rc = check_attention_sizes(batch, lq, lk, d, dv);
  if (rc != SOFTMAX_OK) return rc;
  if (batch == 0 || lq == 0 || dv == 0) return SOFTMAX_OK;

  const int64_t qbytes = batch * lq * d * 4;
  const int64_t kbytes = batch * lk * d * 4;
  const int64_t vbytes = batch * lk * dv * 4;
  const int64_t obytes = batch * lq * dv * 4;
  if (o == nullptr || v == nullptr) return SOFTMAX_ERR_INVALID_ARG;
  if (d > 0 && (q == nullptr || k == nullptr)) return SOFTMAX_ERR_INVALID_ARG;
  // The output may not overlap any input.
  const uintptr_t po = reinterpret_cast<uintptr_t>(o);
  auto overlaps = [&](const float* p, int64_t n) {
    const uintptr_t pp = reinterpret_cast<uintptr_t>(p);
    return n > 0 && pp < po + static_cast<uintptr_t>(obytes) &&
           po < pp + static_cast<uintptr_t>(n);
  };
  if (overlaps(q, qbytes) || overlaps(k, kbytes) || overlaps(v, vbytes))
    return SOFTMAX_ERR_INVALID_ARG;

  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e);
  if (qbytes > 0 && (rc = check_device_range(q, qbytes, dev)) != SOFTMAX_OK) return rc;
  if (kbytes > 0 && (rc = check_device_range(k, kbytes, dev)) != SOFTMAX_OK) return rc;
  if ((rc = check_device_range(v, vbytes, dev)) != SOFTMAX_OK) return rc;
  if ((rc = check_device_range(o, obytes, dev)) != SOFTMAX_OK) return rc;

  int cus = 0;
  if ((rc = device_cus(dev, &cus)) != SOFTMAX_OK) return rc;
  // 16-byte aligned rows throughout (the DAM tile's LDS copies).
  const bool vec4 = d % 4 == 0 && dv % 4 == 0 && aligned16(q) && aligned16(k) &&
                    aligned16(v) && aligned16(o);
  const int ilq = static_cast<int>(lq), ilk = static_cast<int>(lk);
  const int id = static_cast<int>(d), idv = static_cast<int>(dv);
  // The DAM tile runs 64-query items on the ping-pong kernel, one per CU and
  // turn; many items of one query tile fill a quarter of it and run faster a
  // wavefront each (2000 x 16 x 50 x 200 x 200 45 us against 61, 2000 x 1
  // 35 against 59; 2000 x 32 level; 100 x 16 13.4 against 10.0).
  if (vec4 && dam_tile(ilk, id, idv) && (lq > 16 || batch < kAttnMinWavesPerCU * cus)) {
    e = wide ? run_attention_dam<true>(q, k, v, o, batch, ilq, ilk, id, idv, scale, c, cus, stream)
             : run_attention_dam<false>(q, k, v, o, batch, ilq, ilk, id, idv, scale, c, cus,
                                        stream);
    return e == hipSuccess ? SOFTMAX_OK : fail_hip(e);
  }
  return run_attention_wave(q, k, v, o, batch, ilq, ilk, id, idv, scale, c, cus, stream);
}

}  // extern "C"

// Fused softmax attention with one wavefront per block of queries.
//
// The mapping of sm_attention.hpp (scores transposed, S^T = K Q^T, the
// softmax in the accumulators, the weights used as they lie for the value
// product), with every operand read straight from memory into the registers
// of the one wavefront that uses it:
//
//   * A wavefront takes 16 NQ queries of a batch element (NQ = 1..3 query
//     tiles against NK = 1..4 key tiles); each K and V operand it loads serves
//     NQ matrix ops.
//   * No LDS, no barrier: the wavefronts of a workgroup run items of their
//     own, and two or more wavefronts per SIMD overlap one's loads and softmax
//     with another's matrix ops.
//   * Operands are loaded ahead: the next 32 columns of Q and K during this
//     pair of blocks' matrix ops, the next item's first 32 during this one's
//     softmax and value product, the first V rows before the softmax, the
//     next key tiles of V during this one's matrix ops.
//   * Loads need 4-byte alignment only, so any d and dv take 128-bit loads.
//     The last 16-column block of Q and K is masked; a lane whose four columns
//     would pass the row's end reads the row's last four and drops the ones
//     that another lane has.  The last dv % 64 columns of V take as many
//     16-column tiles as they need; a lane that would pass the row's end takes
//     the row's last columns and writes the same values as its neighbour.
//
// Measured per call (graph replay over rotated inputs), against the kernels
// this one replaced (K and V through LDS, two workgroups per CU, one item at
// a time; 32-bit loads from memory for rows that are not whole strips):
//   8192 x 64 x 64 x 64 x 64   141 -> 109 us (4.9 TB/s)
//   16384 x 4 x 37 x 50 x 50   101 -> 59      4096 x 33 x 37 x 50 x 50  75 -> 34
//   2048 x 40 x 60 x 256 x 256 119 -> 81      65536 x 1 x 50 x 64 x 64 672 -> 303
//   16384 x 16 x 16 x 16 x 16   68 -> 16      64 x 64 x 64 x 64 x 64   8.3 -> 5.9
// Bound by HBM where a block has few queries or a small d (64 x 64 heads with
// d = 64 have 16 flops per byte), by the fp32 matrix rate on larger ones.
#pragma once

#include "sm_attention.hpp"

namespace smx {

// Cache policy of the operand loads and of the output stores (the aux
// argument of the buffer instructions): nontemporal.  Stores take it (3-7% on
// most shapes, up to 40% on large outputs of whole 32-byte rows) but on large
// outputs whose rows are not whole 32-byte sectors (PLAIN; the rule is beside
// kAttnPlainMinBytes).  The policy is an instruction field: chosen by a branch
// at run time, the stores cost 2% on average and up to 12%.  Loads take it (STREAM) where one wavefront reads
// all of a batch element's K and V and rows are whole 128-byte lines: 64 x 64
// heads of d = 64 115 -> 108 us per 8192, 40 x 60 of d = 256 80 -> 75 per
// 2048; elsewhere the next loads or wavefronts want the same lines, and it
// cost up to 40%.
constexpr int kAttnNt = 2;

typedef __attribute__((ext_vector_type(4))) unsigned u32x4m;
typedef __attribute__((ext_vector_type(3))) unsigned u32x3m;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2m;

__device__ __forceinline__ float as_f32(unsigned u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ unsigned as_u32(float f) { return __builtin_bit_cast(unsigned, f); }

// x itself, as a value the compiler cannot see through: offsets built from it
// are formed at their loads and stores instead of being kept in registers
// for all of them across the kernel (which spilled 30 to 130 registers).
__device__ __forceinline__ unsigned attn_opaque(unsigned x) {
  asm volatile("" : "+v"(x));
  return x;
}

// N consecutive floats at byte offset off (4-byte aligned) into v[0 .. N),
// zero past the resource.
template <int N, bool STREAM>
__device__ __forceinline__ void buf_load_n(float (&v)[4], __amdgpu_buffer_rsrc_t r, unsigned off) {
  const int o = static_cast<int>(off);
  if constexpr (N == 4) {
    const u32x4m q = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, STREAM ? kAttnNt : 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = as_f32(q[i]);
  } else if constexpr (N == 3) {
    const u32x3m q = __builtin_amdgcn_raw_buffer_load_b96(r, o, 0, STREAM ? kAttnNt : 0);
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] = as_f32(q[i]);
  } else if constexpr (N == 2) {
    const u32x2m q = __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, STREAM ? kAttnNt : 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = as_f32(q[i]);
  } else {
    v[0] = as_f32(__builtin_amdgcn_raw_buffer_load_b32(r, o, 0, STREAM ? kAttnNt : 0));
  }
}

template <int N, bool PLAIN>
__device__ __forceinline__ void buf_store_n(__amdgpu_buffer_rsrc_t r, unsigned off,
                                            const float (&v)[4]) {
  constexpr int kAux = PLAIN ? 0 : kAttnNt;
  const int o = static_cast<int>(off);
  if constexpr (N == 4)
    __builtin_amdgcn_raw_buffer_store_b128(
        u32x4m{as_u32(v[0]), as_u32(v[1]), as_u32(v[2]), as_u32(v[3])}, r, o, 0, kAux);
  else if constexpr (N == 3)
    __builtin_amdgcn_raw_buffer_store_b96(u32x3m{as_u32(v[0]), as_u32(v[1]), as_u32(v[2])}, r, o,
                                          0, kAux);
  else if constexpr (N == 2)
    __builtin_amdgcn_raw_buffer_store_b64(u32x2m{as_u32(v[0]), as_u32(v[1])}, r, o, 0, kAux);
  else
    __builtin_amdgcn_raw_buffer_store_b32(as_u32(v[0]), r, o, 0, kAux);
}

template <bool STREAM>
__device__ __forceinline__ f32x4m buf_load_f4(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(
      f32x4m, __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(off), 0, STREAM ? kAttnNt : 0));
}

// Byte offset of columns t0 .. t0 + 3 of the row at byte offset `row`, past
// every resource from column d on.  RAGGED (d > 4, not a multiple of 4): a
// lane whose four would pass the row's end reads the row's last four instead;
// attn_drop then zeroes the first ones, which the lane before it has.
template <bool RAGGED>
__device__ __forceinline__ unsigned attn_cols(unsigned row, int t0, int d) {
  const int t = RAGGED && t0 + 4 > d ? d - 4 : t0;
  return t0 < d ? row + 4u * static_cast<unsigned>(t) : static_cast<unsigned>(kBufOff);
}
__device__ __forceinline__ f32x4m attn_drop(f32x4m x, int t0, int d) {
  const int skip = t0 + 4 - d;
  return f32x4m{skip > 0 ? 0.0f : x[0], skip > 1 ? 0.0f : x[1], skip > 2 ? 0.0f : x[2], x[3]};
}

// Byte offset in a row of the lane's columns of a block of U 16-column tiles
// at c0: U consecutive columns per lane, the row's last U for a lane that
// would pass its end (it then computes and writes the same values as its
// neighbour), past every resource for a lane past it.
template <int U>
__device__ __forceinline__ unsigned attn_col_off(int c0, int dv, int j) {
  const int c = c0 + U * j;
  return c < dv ? 4u * static_cast<unsigned>(c + U <= dv ? c : dv - U)
                : static_cast<unsigned>(kBufOff);
}

// The value operands of key tile kt: key rows 16 kt + 4 g + r at the lane's
// columns.
struct AttnV {
  float r[4][4];
};
template <int U, bool STREAM>
__device__ __forceinline__ void attn_v_load(AttnV& a, __amdgpu_buffer_rsrc_t rv, unsigned col,
                                            int dv, int kt, int g) {
  const unsigned off = attn_opaque(col + 16u * static_cast<unsigned>(g * dv));
#pragma unroll
  for (int r = 0; r < 4; ++r)
    buf_load_n<U, STREAM>(a.r[r], rv, off + 4u * static_cast<unsigned>((16 * kt + r) * dv));
}

// One block of U 16-column tiles of O = P V: the value operands of key tiles
// 0 .. VD - 1 are in vr (or on their way), tile kt at slot kt % VD; a slot is
// loaded again as soon as it has been used, with this block's tile kt + VD or
// (U = 4) the next block's first ones, at next_col.
template <int NQ, int NK, int VD, int U, bool STREAM, bool PLAIN>
__device__ __forceinline__ void attn_pv_block(const float (&p)[NQ][4 * NK], AttnV (&vr)[VD],
                                              __amdgpu_buffer_rsrc_t rv,
                                              __amdgpu_buffer_rsrc_t ro, unsigned col,
                                              unsigned next_col, int dv, int lk, int g) {
  static_assert(NK % VD == 0, "tile kt sits at slot kt % VD in every block");
  f32x4m acc[NQ][U];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int u = 0; u < U; ++u) acc[q][u] = f32x4m{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int kt = 0; kt < NK; ++kt) {
    AttnV& cur = vr[kt % VD];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // A step whose smallest key (lane group 0) is past lk has weight 0 in
      // every lane.
      if (kt < NK - 1 || 16 * kt + r < lk) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int u = 0; u < U; ++u)
            acc[q][u] = mfma16x16x4(p[q][4 * kt + r], cur.r[r][u], acc[q][u]);
      }
    }
    if (kt + VD < NK)
      attn_v_load<U, STREAM>(cur, rv, col, dv, kt + VD, g);
    else if (U == 4)
      attn_v_load<4, STREAM>(cur, rv, next_col, dv, kt + VD - NK, g);
    __builtin_amdgcn_sched_barrier(0);
  }
  const unsigned off = attn_opaque(col + 16u * static_cast<unsigned>(g * dv));
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float v[4];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = acc[q][u][r];
      buf_store_n<U, PLAIN>(ro, off + 4u * static_cast<unsigned>((16 * q + r) * dv), v);
    }
  }
}

// The last block of a row of value columns, of U < 4 tiles.
template <int NQ, int NK, int VD, int U, bool STREAM, bool PLAIN>
__device__ __forceinline__ void attn_pv_last(const float (&p)[NQ][4 * NK], AttnV (&vr)[VD],
                                             bool loaded, __amdgpu_buffer_rsrc_t rv,
                                             __amdgpu_buffer_rsrc_t ro, int c0, int dv, int lk,
                                             int j, int g) {
  const unsigned col = attn_col_off<U>(c0, dv, j);
  if (!loaded) {
#pragma unroll
    for (int kt = 0; kt < VD; ++kt) attn_v_load<U, STREAM>(vr[kt], rv, col, dv, kt, g);
  }
  attn_pv_block<NQ, NK, VD, U, STREAM, PLAIN>(p, vr, rv, ro, col, 0u, dv, lk, g);
}

// Key tiles of V on their way at once (a divisor of NK: a block's tile 0 is
// always in slot 0): one where more would spill.
template <int NQ, int NK>
constexpr int kAttnVDepth = NQ * NK >= 9 ? 1 : NK == 4 ? 2 : NK;

template <int NQ, int NK, bool RAGGED, bool STREAM, bool PLAIN = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_attention_wave(
    const float* q, const float* k, const float* v, float* o, int64_t batch, int lq, int lk,
    int d, int dv, float scale, Clip clip) {
  constexpr int VD = kAttnVDepth<NQ, NK>;
  const int lane = __lane_id();
  const int j = lane & 15;
  const int g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int qblocks = (lq + 16 * NQ - 1) / (16 * NQ);
  const int64_t items = batch * qblocks;
  const int64_t waves = blockDim.x >> 6;
  const int64_t step = static_cast<int64_t>(gridDim.x) * waves;
  const int nblk = (d + 15) >> 4;
  const int npair = (nblk + 1) >> 1;
  const unsigned row = 4u * static_cast<unsigned>(j * d);
  const unsigned tile = 64u * static_cast<unsigned>(d);  // 16 rows

  // Q and K operands: two slots of a pair of 16-column blocks.  A pair's two
  // loads take the two halves of the same 128-byte lines one after the other,
  // before other loads can evict them (a block at a time, HBM reads were 25%
  // over the operands' bytes).  Blocks past the row's end load nothing
  // (offsets past the resource), without a branch, so every wait counts only
  // the loads before it.
  f32x4m qf[2][2][NQ], kf[2][2][NK];
  __amdgpu_buffer_rsrc_t rq, rk;
  int64_t b = 0;
  int q0 = 0, nq = 0;
  auto load = [&](int pair, int slot) {
    const unsigned o0 = attn_opaque(attn_cols<RAGGED>(row, 32 * pair + 4 * g, d));
    const unsigned o1 = attn_opaque(attn_cols<RAGGED>(row, 32 * pair + 16 + 4 * g, d));
#pragma unroll
    for (int kt = 0; kt < NK; ++kt) {
      kf[slot][0][kt] = buf_load_f4<STREAM>(rk, o0 + kt * tile);
      kf[slot][1][kt] = buf_load_f4<STREAM>(rk, o1 + kt * tile);
    }
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      qf[slot][0][qt] = buf_load_f4<STREAM>(rq, o0 + qt * tile);
      qf[slot][1][qt] = buf_load_f4<STREAM>(rq, o1 + qt * tile);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // The item's place and the first pair of its blocks on their way.
  auto start = [&](int64_t item) {
    b = qblocks == 1 ? item : item / qblocks;
    q0 = static_cast<int>(item - b * qblocks) * 16 * NQ;
    nq = lq - q0 < 16 * NQ ? lq - q0 : 16 * NQ;
    rq = make_rsrc(q + (b * lq + q0) * static_cast<int64_t>(d), nq * d * 4);
    rk = make_rsrc(k + b * lk * static_cast<int64_t>(d), lk * d * 4);
    if (!(RAGGED && d < 4)) load(0, 0);
  };

  int64_t item = static_cast<int64_t>(blockIdx.x) * waves + w;
  if (item < items) start(item);
  for (; item < items; item += step) {
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(v + b * lk * static_cast<int64_t>(dv), lk * dv * 4);
    const __amdgpu_buffer_rsrc_t ro =
        make_rsrc(o + (b * lq + q0) * static_cast<int64_t>(dv), nq * dv * 4);

    // ---- scores S^T = K Q^T ------------------------------------------------
    f32x4m acc[NQ][NK];
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
      for (int kt = 0; kt < NK; ++kt) acc[qt][kt] = f32x4m{0.0f, 0.0f, 0.0f, 0.0f};
    auto mul = [&](const f32x4m (&qm)[NQ], const f32x4m (&km)[NK]) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int kt = 0; kt < NK; ++kt)
#pragma unroll
          for (int qt = 0; qt < NQ; ++qt)
            acc[qt][kt] = mfma16x16x4(km[kt][s], qm[qt][s], acc[qt][kt]);
    };
    if (RAGGED && d < 4) {
      // One block, 32-bit loads.
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt)
        qf[0][0][qt] = buf_load4<false>(rq, static_cast<int>(row + qt * tile) + 16 * g, 4 * g < d,
                                        d - 4 * g);
#pragma unroll
      for (int kt = 0; kt < NK; ++kt)
        kf[0][0][kt] = buf_load4<false>(rk, static_cast<int>(row + kt * tile) + 16 * g, 4 * g < d,
                                        d - 4 * g);
      mul(qf[0][0], kf[0][0]);
      if (item + step < items) start(item + step);
    } else {
      auto mul_pair = [&](int pair, int slot) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int blk = 2 * pair + h;
          if (blk < nblk) {
            if (RAGGED && 16 * blk + 16 > d) {
              const int t0 = 16 * blk + 4 * g;
#pragma unroll
              for (int qt = 0; qt < NQ; ++qt) qf[slot][h][qt] = attn_drop(qf[slot][h][qt], t0, d);
#pragma unroll
              for (int kt = 0; kt < NK; ++kt) kf[slot][h][kt] = attn_drop(kf[slot][h][kt], t0, d);
            }
            mul(qf[slot][h], kf[slot][h]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      for (int pair = 0; pair < npair; pair += 2) {
        load(pair + 1, 1);
        mul_pair(pair, 0);
        if (pair + 2 < npair) load(pair + 2, 0);
        mul_pair(pair + 1, 1);
      }
      // The next item's first pair is on its way while this one's softmax and
      // value product run.
      if (item + step < items) start(item + step);
    }

    // The first value rows are on their way while the softmax runs.
    const int nfull = dv >> 6;
    const int rest = dv - 64 * nfull;
    const int ulast = (rest + 15) >> 4;  // tiles of the last block, 0: none
    AttnV vr[VD];
    if (nfull > 0 || ulast == 4) {
      const unsigned col = attn_col_off<4>(0, dv, j);
#pragma unroll
      for (int kt = 0; kt < VD; ++kt) attn_v_load<4, STREAM>(vr[kt], rv, col, dv, kt, g);
    } else if (ulast == 3) {
      const unsigned col = attn_col_off<3>(0, dv, j);
#pragma unroll
      for (int kt = 0; kt < VD; ++kt) attn_v_load<3, STREAM>(vr[kt], rv, col, dv, kt, g);
    } else if (ulast == 2) {
      const unsigned col = attn_col_off<2>(0, dv, j);
#pragma unroll
      for (int kt = 0; kt < VD; ++kt) attn_v_load<2, STREAM>(vr[kt], rv, col, dv, kt, g);
    } else {
      const unsigned col = attn_col_off<1>(0, dv, j);
#pragma unroll
      for (int kt = 0; kt < VD; ++kt) attn_v_load<1, STREAM>(vr[kt], rv, col, dv, kt, g);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- clipped softmax over the keys of query 16 qt + j -------------------
    // Only the last key tile can hold keys past lk (NK = ceil(lk / 16)).
    float p[NQ][4 * NK];
    auto key_ok = [&](int i) {
      return (i >> 2) < NK - 1 || 16 * (i >> 2) + 4 * g + (i & 3) < lk;
    };
    const bool wide = clip.lo < kClipWide;
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      float m = -__builtin_inff();
#pragma unroll
      for (int i = 0; i < 4 * NK; ++i) {
        p[qt][i] = acc[qt][i >> 2][i & 3] * scale;
        m = key_ok(i) ? fmaxf(m, p[qt][i]) : m;
      }
      m = fmaxf(m, row16_partner(m));
      m = fmaxf(m, half32_partner(m));
      const RowShift rs = row_shift(m, clip);
      if (wide) {
#pragma unroll
        for (int i = 0; i < 4 * NK; ++i) p[qt][i] = exp_shift_clip<kExpWide>(p[qt][i], rs);
      } else {
#pragma unroll
        for (int i = 0; i < 4 * NK; ++i) p[qt][i] = exp_shift_clip<kExpAccurate>(p[qt][i], rs);
      }
#pragma unroll
      for (int i = 0; i < 4 * NK; ++i) p[qt][i] = key_ok(i) ? p[qt][i] : 0.0f;
      float sum = tree_sum(p[qt]);
      sum = sum + row16_partner(sum);
      sum = sum + half32_partner(sum);
      const float rcp = 1.0f / sum;
#pragma unroll
      for (int i = 0; i < 4 * NK; ++i) p[qt][i] = p[qt][i] * rcp;
      __builtin_amdgcn_sched_barrier(0);
    }

    // ---- O = P V ------------------------------------------------------------
    // Full 64-column blocks (and a last one of four tiles), then the rest.
    const int n4 = nfull + (ulast == 4 ? 1 : 0);
    for (int cb = 0; cb < n4; ++cb) {
      const unsigned next = cb + 1 < n4 ? attn_col_off<4>(64 * (cb + 1), dv, j)
                                        : static_cast<unsigned>(kBufOff);
      attn_pv_block<NQ, NK, VD, 4, STREAM, PLAIN>(p, vr, rv, ro, attn_col_off<4>(64 * cb, dv, j),
                                                  next, dv, lk, g);
    }
    if (ulast == 3)
      attn_pv_last<NQ, NK, VD, 3, STREAM, PLAIN>(p, vr, nfull == 0, rv, ro, 64 * nfull, dv, lk, j,
                                                 g);
    else if (ulast == 2)
      attn_pv_last<NQ, NK, VD, 2, STREAM, PLAIN>(p, vr, nfull == 0, rv, ro, 64 * nfull, dv, lk, j,
                                                 g);
    else if (ulast == 1)
      attn_pv_last<NQ, NK, VD, 1, STREAM, PLAIN>(p, vr, nfull == 0, rv, ro, 64 * nfull, dv, lk, j,
                                                 g);
  }
}

}  // namespace smx

// hb_tile.hip -- traversal (Algorithms 2 and 3 of Sec. 4.1) for feature tiles
// too wide, or trees too deep, for the row-parallel kernel to fill a CU.
//
// The row-parallel kernel (hb_fast.h) gives every lane a row and every wave
// all the trees, so the rows whose features fit in LDS fix the waves on a CU:
// 100 columns leave one wave per SIMD, 200 columns none that pays. Here a
// workgroup is always 16 waves (four per SIMD): R rows across lanes times
// G = 1024 / R groups of waves, each group walking its own share of the trees
// that are staged in LDS. The walk is bound by the latency of its dependent
// LDS reads, so what counts is the number of walks in flight, R / 64 times the
// staged trees, and that vector work of one wave runs under the LDS waits of
// the three others on its SIMD.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <type_traits>

#include "hb_tile.h"
#include "hb_tile_shape.h"

namespace hb {
namespace {

constexpr int kThreads = kTileThreads, kStage = kTileStage;
constexpr int kWaves = kThreads / 64;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int ids4 __attribute__((ext_vector_type(4), aligned(kTileIdStoreAlign)));
typedef __attribute__((address_space(3))) const uint32_t lds_u32;
typedef __attribute__((address_space(3))) const uint64_t lds_u64;
typedef __attribute__((address_space(3))) const float lds_f32;
typedef __attribute__((address_space(3))) const uint16_t lds_u16;
typedef __attribute__((address_space(3))) uint16_t lds_u16w;
typedef __attribute__((address_space(3))) float lds_f32w;

__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

struct TileArgs {
  const float *X;
  int64_t n_rows;
  int32_t F, Fs;             // tile columns, row stride of X
  const int32_t *cols;       // as EnsembleDev::cols
  int32_t *leaf_ids;
  OutArgs out;
  const int32_t *tree_class;
  const uint4 *recs;         // TileDev::recs
  int32_t tree_bytes;
  int32_t depth;             // PTT: D
  const int32_t *tree_depth; // TT: [T]
  const float *leafv;        // TileDev::leafv, [padded T][leaf_slots][LD]
  const int32_t *leaf_id;    // [T][leaf_slots]
  int32_t id_base;           // >= 0: every caller id is id_base + leaf slot
  int32_t leaf_slots, LD;
  const float *thr;          // RANK: TileDev::thr, thr_off
  const int32_t *thr_off;
  int32_t lg_rows;           // log2 R
  int32_t nt, per;           // trees per chunk; of them, per wave group
  int32_t n_chunks;
  int32_t split;             // chunks per workgroup of a tree split (blockIdx.y), 0: all
  double *partial;           // [parts][n_rows][K]: a split's raw sums
  int32_t bufs;              // chunk buffers: 2, or 1 (twice the trees, a second barrier per chunk)
  int32_t buf_off, stage_off;  // LDS byte offsets of the chunk buffers and the leaf-slot staging
  int32_t scratch;           // RANK: floats of LDS from buf_off on, for the thresholds
  int32_t st_chunks;         // chunks per leaf-id flush
  int32_t ids_vec;           // leaf-id rows start 16-byte aligned: stored 16 bytes at a time
};

// LDS byte offset of row r within a column of the tile. 16-bit tiles put the
// rows of two waves in the halves of one word, so that the 64 lanes of a wave
// read 64 words.
template <bool RANK>
__device__ __forceinline__ uint32_t row_off(uint32_t r) {
  return RANK ? ((r >> 7) << 8) + ((r & 63u) << 2) + ((r >> 5) & 2u) : r << 2;
}

// LDS byte address of a record's feature in this lane's column position: one
// multiply-add of a 16-bit half of the record's word (PTT and TT fp32 records
// hold the feature in the low half, rank records in the high one) with the
// column stride, which 16 bits hold too (4 bytes of at most 1,024 rows).
template <bool HIGH>
__device__ __forceinline__ uint32_t xaddr16(uint32_t w, uint32_t stride, uint32_t xlane) {
  uint32_t r;
  if constexpr (HIGH)
    asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(w), "s"(stride), "v"(xlane));
  else
    asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(stride), "v"(xlane));
  return r;
}

// Tile columns f .. f + 3 (below end) of an input row, as xval gives them. The
// category look-ups are taken for all four columns side by side, without
// branches that depend on the column: their four dependent loads (column,
// descriptor, value, set word) then overlap (101 leaf-wise trees, 354 tile
// columns of which 282 are category sets: one look-up after the other took
// half of the call).
__device__ __forceinline__ f32x4 tile_values(const TileArgs &a, const float *row, int f, int end) {
  f32x4 v = {0, 0, 0, 0};
  if (!a.cols) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (f + j < end) v[j] = row[f + j];
    return v;
  }
  const uint32_t *cu = reinterpret_cast<const uint32_t *>(a.cols);
  uint32_t c[4], any = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    c[j] = cu[min(f + j, end - 1)];
    any |= c[j];
  }
  if (!__any((any & (uint32_t)kColCat) != 0)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = row[c[j] & (uint32_t)kColMask];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if ((c[j] & (uint32_t)kColNanLeft) && __builtin_isnan(v[j])) v[j] = -__builtin_inff();
    return v;
  }
  uint32_t at[4], col[4], words[4], bits[4];
  bool cat[4], in[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    cat[j] = (c[j] & (uint32_t)kColCat) != 0;
    at[j] = cat[j] ? c[j] & (uint32_t)kColMask : 0u;  // (entry 0 exists: read and not used)
    col[j] = cu[at[j]];
    words[j] = cu[at[j] + (cat[j] ? 1u : 0u)];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = row[cat[j] ? col[j] : c[j] & (uint32_t)kColMask];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    in[j] = cat[j] && v[j] >= 0.0f && v[j] < 32.0f * (float)words[j];  // (a NaN is in no set)
    const uint32_t k = in[j] ? (uint32_t)v[j] : 0u;
    bits[j] = cu[in[j] ? at[j] + 2u + (k >> 5) : 0u] >> (k & 31u);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const bool nan = __builtin_isnan(v[j]), nan_left = (c[j] & (uint32_t)kColNanLeft) != 0;
    const bool left = nan ? nan_left : in[j] && (bits[j] & 1u);
    v[j] = cat[j] ? (left ? 0.0f : 1.0f) : (nan && nan_left) ? -__builtin_inff() : v[j];
  }
  return v;
}

// The workgroup's rows into an fp32 tile. A wave takes blocks of 8 rows by 8
// lanes of four consecutive columns (one 128-byte line of a row per eight
// lanes), four blocks in flight.
__device__ __forceinline__ void load_tile(const TileArgs &a, uint32_t xs, int64_t r0, int wave, int lane) {
  const int R = 1 << a.lg_rows;
  const int nbc = (a.F + 31) >> 5, blocks = nbc * (R >> 3);
  const bool vec = !a.cols && (a.Fs & 3) == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0;
  const uint32_t stride = (uint32_t)R * 4u;
  constexpr int U = 4;
  int rb = 0, cb = wave;
  while (cb >= nbc) cb -= nbc, ++rb;
  for (int blk = wave; blk < blocks; blk += U * kWaves) {
    f32x4 v[U];
    int row[U], col[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      row[u] = 8 * rb + (lane >> 3);
      col[u] = 32 * cb + 4 * (lane & 7);
      const bool in = blk + u * kWaves < blocks && col[u] < a.F && r0 + row[u] < a.n_rows;
      if (!(blk + u * kWaves < blocks)) row[u] = -1;
      v[u] = f32x4{0, 0, 0, 0};
      if (in) {
        const float *src = a.X + (r0 + row[u]) * a.Fs;
        if (vec) {
          v[u] = *reinterpret_cast<const f32x4 *>(src + col[u]);
        } else {
          v[u] = tile_values(a, src, col[u], a.F);
        }
      }
      cb += kWaves;
      while (cb >= nbc) cb -= nbc, ++rb;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (row[u] < 0) continue;
      const uint32_t at = xs + ((uint32_t)row[u] << 2) + (uint32_t)col[u] * stride;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (col[u] + j < a.F) *(lds_f32w *)(uintptr_t)(at + j * stride) = v[u][j];
    }
  }
}

// The workgroup's rows into a rank tile. The sorted thresholds of a few
// columns at a time pass through LDS (scratch: the chunk buffers' space) and
// every lane searches them for its own row, four columns side by side: a
// scattered LDS read costs a wave some 7 clocks where a scattered global read
// takes 64 (ranking through the caches took 84 of 191 us on 100K rows of 28
// columns with 14,600 thresholds each). A column with more thresholds than the
// scratch holds has every 2^m-th of them there and takes its last m steps in
// global memory.
__device__ __forceinline__ void load_ranks(const TileArgs &a, uint32_t xs, float *scratch, int cap, int64_t r0,
                                           uint32_t lrow, int group, int lane) {
  const int G = kThreads >> a.lg_rows;
  const bool valid = r0 + lrow < a.n_rows;
  const float *src = a.X + (r0 + (valid ? lrow : 0)) * a.Fs;
  const bool vec = !a.cols && (a.Fs & 3) == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0;
  const uint32_t stride = 2u << a.lg_rows;
  const uint32_t at0 = xs + row_off<true>(lrow);
  for (int c0 = 0; c0 < a.F;) {
    // as many columns as fit, a multiple of four unless it is the rest
    const int base = a.thr_off[c0];
    const int end = a.thr_off[min(c0 + 1 + lane, a.F)];
    const unsigned long long fit = __ballot(c0 + 1 + lane <= a.F && end - base <= cap);
    int nc = __builtin_popcountll(fit);  // (offsets do not decrease: the ballot is a run of ones)
    if (nc >= 4 && c0 + nc < a.F) nc &= ~3;
    int lg = 0;  // log2 of the sampling stride
    if (nc == 0) {
      nc = 1;
      while (((a.thr_off[c0 + 1] - base) >> lg) > cap) ++lg;
    }
    nc = __builtin_amdgcn_readfirstlane(nc);
    const int c1 = c0 + nc;
    const int total = (a.thr_off[c1] - base) >> lg;
    for (int i0 = (int)threadIdx.x; i0 < total; i0 += 16 * kThreads) {  // 16 loads in flight
      float t[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) t[u] = a.thr[base + ((min(i0 + u * kThreads, total - 1) + 1) << lg) - 1];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (i0 + u * kThreads < total) scratch[i0 + u * kThreads] = t[u];
    }
    __syncthreads();
    for (int c = c0 + 4 * group; c < c1; c += 4 * G) {
      f32x4 v = {0, 0, 0, 0};
      int lo[4], n[4], top = 0;
      uint32_t rank[4];
      if (vec && (c & 3) == 0) {
        v = *reinterpret_cast<const f32x4 *>(src + c);  // (Fs is a multiple of four)
      } else {
        v = tile_values(a, src, c, c1);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int f = min(c + j, c1 - 1);
        lo[j] = (a.thr_off[f] - base) >> lg;
        n[j] = (a.thr_off[f + 1] - a.thr_off[f]) >> lg;
        top = max(top, n[j]);
        rank[j] = 0;
      }
      for (int step = top ? 1 << (31 - __builtin_clz((unsigned)top)) : 0; step; step >>= 1) {
        float t[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) t[j] = scratch[max(lo[j] + min((int)rank[j] + step, n[j]) - 1, 0)];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if ((int)rank[j] + step <= n[j] && !(v[j] < t[j])) rank[j] += step;
      }
      if (lg) {
        const int nf = a.thr_off[c + 1] - base;  // (one column)
        rank[0] <<= lg;
        for (int step = 1 << (lg - 1); step; step >>= 1)
          if ((int)rank[0] + step <= nf && !(v[0] < a.thr[base + rank[0] + step - 1])) rank[0] += step;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c + j < c1) *(lds_u16w *)(uintptr_t)(at0 + (uint32_t)(c + j) * stride) = (uint16_t)rank[j];
    }
    __syncthreads();
    c0 = c1;
  }
}

// Leaf ids of st staged trees (first tree t0) for the workgroup's rows: eight
// lanes per row, four trees each.
__device__ __forceinline__ void flush_slots(const TileArgs &a, uint32_t stage, uint32_t sstride, int t0, int st,
                                            int64_t r0, int wave, int lane) {
  const int R = 1 << a.lg_rows, T = a.out.T;
  const int k4 = 4 * (lane & 7);
  st = min(st, T - t0);
  for (int rb = wave; rb < (R >> 3); rb += kWaves) {
    const int r = 8 * rb + (lane >> 3);
    if (k4 >= st || r0 + r >= a.n_rows) continue;
    ids4 id;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = tile_flush_tree(k4 + j, st);
      const uint32_t slot = *(lds_u16 *)(uintptr_t)(stage + k * sstride + 2u * r);
      id[j] = a.id_base < 0 ? a.leaf_id[(size_t)(t0 + k) * a.leaf_slots + slot] : a.id_base + (int)slot;
    }
    int32_t *dst = a.leaf_ids + (r0 + r) * T + t0 + k4;
    if (a.ids_vec && k4 + 4 <= st) {
      *reinterpret_cast<ids4 *>(dst) = id;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k4 + j < st) dst[j] = id[j];
    }
  }
}

// PERFECT: PerfectTreeTraversal records, else TreeTraversal. RANK: the tile
// holds 16-bit ranks and the records rank bounds. KM: sums per row (1, 2 or
// 16). ILP: trees a wave walks together.
template <bool PERFECT, bool RANK, int KM, bool VEC, int ILP>
__global__ __launch_bounds__(kThreads) void tile_kernel(TileArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int R = 1 << a.lg_rows;
  const int group = wave >> (a.lg_rows - 6);
  const uint32_t lrow = (uint32_t)tid & (uint32_t)(R - 1);
  const int64_t r0 = (int64_t)blockIdx.x << a.lg_rows;
  static_assert(PERFECT || !RANK, "rank tables are built for PTT only");
  constexpr uint32_t REC = RANK ? 4 : 8;
  const uint32_t stride = (uint32_t)R * (RANK ? 2u : 4u);
  const uint32_t xlane = lds + row_off<RANK>(lrow);
  const int chunk16 = a.nt * a.tree_bytes / 16;
  const uint32_t chunk_bytes = (uint32_t)(a.nt * a.tree_bytes);
  const u32x4 *src = reinterpret_cast<const u32x4 *>(a.recs);
  u32x4 *bufp = reinterpret_cast<u32x4 *>(smem + a.buf_off);

  u32x4 pf[kStage];
  auto fetch = [&](int c) {
#pragma unroll
    for (int i = 0; i < kStage; ++i) pf[i] = src[(size_t)c * chunk16 + min(i * kThreads + tid, chunk16 - 1)];
  };
  auto put = [&](int b) {
#pragma unroll
    for (int i = 0; i < kStage; ++i)
      if (i * kThreads + tid < chunk16) bufp[b * chunk16 + i * kThreads + tid] = pf[i];
  };
  const int c_begin = a.split ? (int)blockIdx.y * a.split : 0;
  const int c_end = a.split ? min(c_begin + a.split, a.n_chunks) : a.n_chunks;
  fetch(c_begin);
  if constexpr (RANK)
    load_ranks(a, lds, reinterpret_cast<float *>(smem + a.buf_off), a.scratch, r0, lrow, group, lane);
  else
    load_tile(a, lds, r0, wave, lane);
  put(0);
  lds_barrier();

  double acc[KM];
#pragma unroll
  for (int k = 0; k < KM; ++k) acc[k] = 0.0;
  constexpr bool vecl = VEC;  // vector leaves (KM = 2: held; more: added at once)
  float hv[ILP], hw[ILP];
  int hk[ILP];
#pragma unroll
  for (int i = 0; i < ILP; ++i) {
    hv[i] = 0.0f;
    hw[i] = 0.0f;
    hk[i] = 0;
  }
  // the values of the trees walked last, read a batch ago
  auto add_held = [&]() {
#pragma unroll
    for (int i = 0; i < ILP; ++i) {
      if (KM == 1) {
        acc[0] += (double)hv[i];
      } else if (KM == 2) {
        if (vecl) {
          acc[0] += (double)hv[i];
          acc[1] += (double)hw[i];
        } else {
          acc[0] += hk[i] == 0 ? (double)hv[i] : 0.0;
          acc[1] += hk[i] == 0 ? 0.0 : (double)hv[i];
        }
      } else {
        acc[hk[i] & (KM - 1)] += (double)hv[i];
      }
    }
  };
  const uint32_t sstride = tile_slot_stride(R);
  const uint32_t stage0 = lds + (uint32_t)a.stage_off;
  const int st = a.st_chunks * a.nt;
  const uint32_t stage_bytes = (uint32_t)st * sstride;
  int sc = 0, sb = 0;  // chunk within the flush group, staging buffer
  int pending = -1;    // first tree of the staged group still to be written
  int staged = 0;      // trees in it (the group that ends a workgroup's trees may be short)

  for (int c = c_begin; c < c_end; ++c) {
    const int b = a.bufs == 2 ? (c - c_begin) & 1 : 0;
    const bool more = c + 1 < c_end;
    fetch(more ? c + 1 : c);
    if (pending >= 0) {
      flush_slots(a, stage0 + (uint32_t)(sb ^ 1) * stage_bytes, sstride, pending, staged, r0, wave, lane);
      pending = -1;
    }
    const uint32_t buf = lds + (uint32_t)a.buf_off + (uint32_t)b * chunk_bytes;
    for (int q = 0; q < a.per; q += ILP) {
      const int tl = group * a.per + q;  // uniform
      const int t = c * a.nt + tl;
      const uint32_t tb = buf + (uint32_t)(tl * a.tree_bytes);
      uint32_t ad[ILP];
      if constexpr (PERFECT) {
        // heap step in bytes, places in path order: inc = REC << level
        uint32_t inc = REC;
        using Word = typename std::conditional<RANK, lds_u32, lds_u64>::type;
        typename std::conditional<RANK, uint32_t, uint64_t>::type rec[ILP];
        uint32_t xv[ILP];
#pragma unroll
        for (int i = 0; i < ILP; ++i) {
          ad[i] = tb + (uint32_t)(i * a.tree_bytes) + REC;
          rec[i] = *(Word *)(uintptr_t)ad[i];
        }
        auto features = [&]() {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < ILP; ++i) {
            if constexpr (RANK)
              xv[i] = *(lds_u16 *)(uintptr_t)xaddr16<true>((uint32_t)rec[i], stride, xlane);
            else
              xv[i] = *(lds_u32 *)(uintptr_t)xaddr16<false>((uint32_t)(rec[i] >> 32), stride, xlane);
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        auto step = [&](int i) {
          bool left;
          if constexpr (RANK)
            left = (uint16_t)xv[i] < (uint16_t)rec[i];
          else
            left = as_float(xv[i]) < as_float((uint32_t)rec[i]);
          ad[i] = ad[i] + inc + (left ? 0u : inc);
        };
        for (int l = 1; l < a.depth; ++l) {
          features();
#pragma unroll
          for (int i = 0; i < ILP; ++i) {
            step(i);
            rec[i] = *(Word *)(uintptr_t)ad[i];
          }
          inc <<= 1;
          asm volatile("" : "+v"(inc));
        }
        features();
#pragma unroll
        for (int i = 0; i < ILP; ++i) step(i);
        // (REC * (2^D + place) from the tree's start)
#pragma unroll
        for (int i = 0; i < ILP; ++i) ad[i] -= tb + (uint32_t)(i * a.tree_bytes) + (REC << a.depth);
      } else {
        int levels = 0;
#pragma unroll
        for (int i = 0; i < ILP; ++i) levels = max(levels, a.tree_depth[min(t + i, a.out.T - 1)]);
        uint32_t b0[ILP], b8[ILP];
        uint32_t xv[ILP];
        uint2 rec[ILP];
#pragma unroll
        for (int i = 0; i < ILP; ++i) {
          b0[i] = tb + (uint32_t)(i * a.tree_bytes);
          b8[i] = b0[i] - 8u;
          ad[i] = b0[i];
        }
#pragma unroll
        for (int i = 0; i < ILP; ++i) {
          const uint64_t w = *(lds_u64 *)(uintptr_t)ad[i];
          rec[i] = make_uint2((uint32_t)w, (uint32_t)(w >> 32));
        }
        for (int l = 0; l < levels; ++l) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < ILP; ++i) {
            xv[i] = *(lds_u32 *)(uintptr_t)xaddr16<false>(rec[i].y, stride, xlane);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < ILP; ++i) {
            // (the read after the last level is unused but in bounds)
            ad[i] = (rec[i].y >> 16) + (as_float(xv[i]) < as_float(rec[i].x) ? b8[i] : b0[i]);
            const uint64_t w = *(lds_u64 *)(uintptr_t)ad[i];
            rec[i] = make_uint2((uint32_t)w, (uint32_t)(w >> 32));
          }
        }
#pragma unroll
        for (int i = 0; i < ILP; ++i) ad[i] -= b0[i];
      }
      __builtin_amdgcn_sched_barrier(0);
      // ad: the leaf's place in its tree, in bytes of records
      const uint32_t lbase = (uint32_t)t * (uint32_t)a.leaf_slots;
      if constexpr (KM < 16 || !vecl) {
        add_held();
        // the sums are taken here, not after the loads: these take the
        // registers the values have just left (no copies, so no wait for them)
#pragma unroll
        for (int k = 0; k < KM; ++k) asm volatile("" : "+v"(acc[k]));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < ILP; ++i) {
          const uint32_t at = 4u * (lbase + (uint32_t)(i * a.leaf_slots)) + (REC == 8 ? ad[i] >> 1 : ad[i]);
          const unsigned char *lv = reinterpret_cast<const unsigned char *>(a.leafv);
          if (KM == 2 && vecl) {
            const float2 w = *reinterpret_cast<const float2 *>(lv + 2u * at);
            hv[i] = w.x;
            hw[i] = w.y;
          } else {
            hv[i] = *reinterpret_cast<const float *>(lv + at);
            if (KM > 1) hk[i] = a.tree_class[t + i];
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < ILP; ++i) {
          const float *lv = a.leafv + (size_t)(lbase + (uint32_t)(i * a.leaf_slots) + ad[i] / REC) * a.LD;
#pragma unroll
          for (int k = 0; k < KM; ++k)
            if (k < a.LD) acc[k] += (double)lv[k];
        }
      }
      if (a.leaf_ids) {
        const uint32_t at = stage0 + (uint32_t)sb * stage_bytes + (uint32_t)(sc * a.nt + tl) * sstride + 2u * lrow;
#pragma unroll
        for (int i = 0; i < ILP; ++i)
          *(lds_u16w *)(uintptr_t)(at + (uint32_t)i * sstride) =
              (uint16_t)(PERFECT ? __builtin_bitreverse32(ad[i] / REC) >> (32 - a.depth) : ad[i] / REC);
      }
    }
    if (a.bufs == 1) lds_barrier();  // every wave is done with the one buffer
    if (more) put(a.bufs == 2 ? b ^ 1 : 0);
    lds_barrier();
    if (a.leaf_ids && (++sc == a.st_chunks || !more)) {
      pending = (c + 1 - sc) * a.nt;
      staged = sc * a.nt;
      sc = 0;
      sb ^= 1;
    }
  }
  if (pending >= 0)
    flush_slots(a, stage0 + (uint32_t)(sb ^ 1) * stage_bytes, sstride, pending, staged, r0, wave, lane);
  if (KM < 16 || !vecl) add_held();

  // the groups' sums in group order
  const int G = kThreads >> a.lg_rows;
  const int64_t row = r0 + lrow;
  if (G > 1) {
    double *red = reinterpret_cast<double *>(smem);
    lds_barrier();
#pragma unroll
    for (int k = 0; k < KM; ++k)
      if (k < a.out.K) red[(size_t)(group * a.out.K + k) * R + lrow] = acc[k];
    lds_barrier();
    if (group != 0) return;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      if (k < a.out.K) {
        double v = 0.0;
        for (int g = 0; g < G; ++g) v += red[(size_t)(g * a.out.K + k) * R + lrow];
        acc[k] = v;
      }
    }
  }
  if (row >= a.n_rows) return;
  if (a.split) {
    double *dst = a.partial + ((size_t)blockIdx.y * a.n_rows + row) * a.out.K;
#pragma unroll
    for (int k = 0; k < KM; ++k)
      if (k < a.out.K) dst[k] = acc[k];
  } else {
    finish_row<KM>(a.out, acc, row);
  }
}

using TileFn = void (*)(TileArgs);

template <bool PERFECT, bool RANK, int ILP>
TileFn pick_k(int km, bool vec) {
  if (vec) return km == 2 ? tile_kernel<PERFECT, RANK, 2, true, ILP> : tile_kernel<PERFECT, RANK, 16, true, ILP>;
  return km == 1   ? tile_kernel<PERFECT, RANK, 1, false, ILP>
         : km == 2 ? tile_kernel<PERFECT, RANK, 2, false, ILP>
                   : tile_kernel<PERFECT, RANK, 16, false, ILP>;
}
template <bool PERFECT, bool RANK>
TileFn pick(int km, bool vec, int ilp) {
  return ilp == 1   ? pick_k<PERFECT, RANK, 1>(km, vec)
         : ilp == 2 ? pick_k<PERFECT, RANK, 2>(km, vec)
         : ilp == 3 ? pick_k<PERFECT, RANK, 3>(km, vec)
         : ilp == 4 ? pick_k<PERFECT, RANK, 4>(km, vec)
                    : pick_k<PERFECT, RANK, 8>(km, vec);
}

}  // namespace

int launch_tile(bool perfect, const EnsembleDev &e, const TileDev &tile, const TileDev *rank, const int32_t *leaf_id,
                int leaf_slots, int levels, const int32_t *tree_depth, const float *X, int64_t n_rows, float *scores,
                int32_t *leaf_ids, const Launch &ws, hipStream_t stream, std::string *err) {
  int dev = 0, cus = 0, lds_max = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1 ||
      hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
    *err = "hipDeviceGetAttribute failed";
    return HB_ERR_HIP;
  }
  const int64_t ws_bytes = ws.ptr && n_rows <= kTileSplitMaxRows ? ws.bytes : 0;
  if ((!tile.recs && !(rank && rank->recs)) || (!ws_bytes && n_rows < (int64_t)kTileMinRowsPerCu * cus)) return 1;
  if ((int64_t)kThreads * e.n_outputs * 8 > lds_max) return 1;
  const TileDev *tp = &tile;
  auto shape = [&](const TileDev &t) {
    if (!t.recs) return TileShape{};
    const TileSpec spec{e.n_trees, e.n_cols, e.n_outputs, levels, t.tree_bytes, t.thr != nullptr, t.n_thr, t.search_steps};
    return best_shape(spec, n_rows, leaf_ids != nullptr, ws_bytes, lds_max, cus);
  };
  TileShape p = shape(tile);
  if (rank) {
    const TileShape q = shape(*rank);
    if (q.rows && (!p.rows || q.cost < p.cost)) {
      p = q;
      tp = rank;
    }
  }
  if (!p.rows || (n_rows < (int64_t)kTileMinRowsPerCu * cus && p.parts < 2)) return 1;
  // Leaf ids of fewer than 16 trees at a time leave as short pieces of lines:
  // beyond 3M walks a leaf-wise split is then slower than the row-parallel one
  // (800 trees of 255 leaves, 50 columns, flushes of 6 trees, 6,500 rows: 68
  // against 55 us; at 3,000 rows, 28 against 42).
  if (!perfect && leaf_ids && p.parts > 1 && p.nt * p.st_chunks < 16 && n_rows * e.n_trees > 3000000) return 1;
  const TileDev &t = *tp;
  const int km = e.n_outputs == 1 ? 1 : e.n_outputs == 2 ? 2 : 16;
  TileArgs a{};
  a.X = X;
  a.n_rows = n_rows;
  a.F = e.n_cols;
  a.Fs = e.n_features;
  a.cols = e.cols;
  a.leaf_ids = leaf_ids;
  a.out = OutArgs{scores, e.n_trees, e.n_outputs, e.aggregation, e.transform, e.base_score};
  a.tree_class = e.tree_class;
  a.recs = t.recs;
  a.tree_bytes = t.tree_bytes;
  a.depth = levels;
  a.tree_depth = tree_depth;
  a.leafv = t.leafv;
  a.leaf_id = leaf_id;
  a.leaf_slots = leaf_slots;
  a.LD = e.leaf_dim;
  a.id_base = t.id_base;
  a.thr = t.thr;
  a.thr_off = t.thr_off;
  a.lg_rows = __builtin_ctz((unsigned)p.rows);
  a.nt = p.nt;
  a.per = p.nt / (kThreads / p.rows);
  a.n_chunks = (e.n_trees + p.nt - 1) / p.nt;
  a.split = p.split;
  a.partial = static_cast<double *>(ws.ptr);
  a.bufs = p.bufs;
  a.buf_off = p.buf_off;
  a.stage_off = p.stage_off;
  a.scratch = (p.lds - p.buf_off) / 4;
  a.st_chunks = p.st_chunks;
  a.ids_vec = e.n_trees % 4 == 0 && (reinterpret_cast<uintptr_t>(leaf_ids) & 15) == 0;
  const bool vec = e.leaf_dim > 1, ranked = t.thr != nullptr;
  TileFn fn = !perfect ? pick<false, false>(km, vec, p.ilp)
              : ranked ? pick<true, true>(km, vec, p.ilp)
                       : pick<true, false>(km, vec, p.ilp);
  const int64_t blocks = (n_rows + p.rows - 1) / p.rows;
  if (ws.plan) {
    auto tf = [](bool b) { return b ? "true, " : "false, "; };
    plan_line(ws.plan,
              std::string("tile_kernel<") + tf(perfect) + tf(ranked) + std::to_string(km) + ", " + tf(vec) +
                  std::to_string(p.ilp) + ">",
              blocks, p.parts, kThreads, p.lds);
    return p.parts > 1 ? split_finish(nullptr, p.parts, n_rows, a.out, ws.plan, stream, err) : HB_OK;
  }
  hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      p.lds);
  if (rc != hipSuccess) {
    *err = std::string("hipFuncSetAttribute: ") + hipGetErrorString(rc);
    return HB_ERR_HIP;
  }
  hipLaunchKernelGGL(fn, dim3((unsigned)blocks, (unsigned)p.parts), dim3(kThreads), p.lds, stream, a);
  rc = hipGetLastError();
  if (rc != hipSuccess) {
    *err = std::string("kernel launch: ") + hipGetErrorString(rc);
    return HB_ERR_HIP;
  }
  if (p.parts > 1) return split_finish(a.partial, p.parts, n_rows, a.out, nullptr, stream, err);
  return HB_OK;
}

}  // namespace hb

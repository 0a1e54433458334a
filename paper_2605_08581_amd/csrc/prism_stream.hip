// Attention for few query rows per (request, kv head): decode steps and short
// suffixes.  At most 32 packed rows share every K/V byte, so the work is below
// 32 flop per byte and the kernel is bound by how many bytes it keeps in flight
// from HBM, or, for small waves, by latency.
//
// Waves too small to fill the chip come here as well, with more rows in tiles of
// 16: the tiles of a (request, kv head) read its keys again each, from the die's
// L2, but every CU works, a chain of key steps is a quarter as long, and nothing
// has to be merged by a second launch.  us per pass, prefill kernel -> this one:
// 37 rows x 4 over 1003 cached keys, 8 kv heads, d = 128 (80 tiles) 13.6 -> 11.3,
// 64 x 4 over 300 (128 tiles) 10.3 -> 6.4, four requests of 48 over 200 keys x 4
// heads, d = 64 (48 tiles) 6.4 -> 5.0.
//
// One workgroup serves one (request, kv head, row tile, key range).  Its four waves split
// the KEYS, not the rows: wave w takes the 32-key tiles w, w+4, ... for all rows.
// No K/V byte is shared between waves, so each wave streams into LDS rings of
// its own with direct-to-LDS copies and waits for its own copies only; there is
// no barrier until the waves' partial results meet at the end.  Two tiles per
// wave are in flight or in use, 128 KB per CU at d = 128: about 100 KB on the
// way, which covers the HBM latency.  (Measured beside it at d = 128: two waves
// with four tiles each 7 % slower on 64 x 4096 keys, one wave with three or four
// tiles 4 %; two waves with two tiles, two workgroups per CU, equal there and
// 4 % slower on small batches.)
//
// With the row tile of the prefill kernel (128 rows, four waves sharing one
// tile) the same work left three of four waves without rows, took two barriers
// per tile and ran a chain of 64-key steps per workgroup.  16 requests x 300 to
// 4100 keys, 32/8 heads, d = 128 (143 MB): three launches 49 us, then one of
// 31.5 us; 64 x 4096 keys, 40 heads (4.37 GB): 771 -> 753 us.  Now, with the pages
// of one request alone read past the caches (AttnItem::read_once), 27.3 us =
// 5.2 TB/s and 694 us = 6.3 TB/s, where a plain streaming read reaches 6.5.
//
// Products are taken transposed as in the prefill kernel, with the 16x16x32
// MFMA because rows come in blocks of 16:
//   S^T = K Q^T    A = K rows from LDS, B = Q rows in registers
//   O^T = V^T P^T  A = V read transposed from LDS, B = P^T from the S^T registers
// In the 16x16 accumulator layout lane l holds column l%16 (a query row) and
// rows 4*(l/16) + r, r = 0..3 (keys for S^T, head dims for O^T).  The 32 keys of
// the second product are numbered 8*(l/16) + j: j < 4 is key 4*(l/16)+j of the
// first 16 keys, j >= 4 is key 4*(l/16)+j-4 of the second 16, which is where the
// S^T accumulators already hold them.
#include "prism_device.h"

namespace prism {

template <int D, int RB>
struct StreamShape {
  static constexpr int NW = 4;                              // waves per workgroup
  static constexpr int NS = 2;                              // tiles per wave in flight or in use
  static constexpr int kTile = 32;                          // keys per wave and step: two pages
  static constexpr int kTileBytes = 2 * kTile * D * 2;      // K then V
  static constexpr int kRows = 16 * RB;
  static constexpr int kRowPitch = D + 4;                   // floats; keeps 16 rows off one bank
  static constexpr size_t kRingBytes = (size_t)NW * NS * kTileBytes;
  static constexpr size_t kMergeBytes = (size_t)NW * kRows * (kRowPitch + 2) * sizeof(float);
  static constexpr size_t kQBytes = (size_t)kRows * D * 2;  // every wave has a copy: no barrier before its first use
  static constexpr size_t kLdsBytes = kRingBytes + NW * kQBytes;
  static_assert(kMergeBytes <= kRingBytes, "the merge works in the idle rings");
  static_assert(kLdsBytes <= 160 * 1024, "LDS of a CU");
};

// largest / sum over the four 16-lane groups that hold one query row
__device__ __forceinline__ float max_across_groups(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max_across_halves(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
}
__device__ __forceinline__ float sum_across_groups(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return sum_across_halves(__uint_as_float(a[0]) + __uint_as_float(a[1]));
}

// ONCE: items may have their cached pages to themselves (AttnItem::read_once).
template <int D, int RB, bool ONCE>
__global__ __launch_bounds__(256) void stream_attn_kernel(const AttnArgs p) {
  using Shape = StreamShape<D, RB>;
  constexpr int NW = Shape::NW, NS = Shape::NS;
  constexpr int NT = NW * 64;
  constexpr int CPR = D / 8;                     // 16-byte chunks per key row
  constexpr int ROW = D * 2;                     // bytes per key row
  constexpr int UPP = kPage * ROW / 1024;        // 1 KB copies per (page, head) block
  constexpr int KPU = 1024 / ROW;                // keys per copy
  constexpr int KK = D / 32;                     // MFMA k-steps over the head dim
  constexpr int DB = D / 16;                     // 16-wide head-dim blocks of O^T
  constexpr int TK = Shape::kTile;
  constexpr int COPIES = 2 * 2 * UPP;            // copies per tile: two pages of K and of V
  static_assert(NS * COPIES <= 63, "pending copies must fit the vmcnt counter");

  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

  // The way to the first tile, a chain of reads that miss the caches, asks for all
  // of each link at once, as in the prefill kernel; what does not depend on the
  // item is worked out while that is on its way.  (us per pass before -> after:
  // 4 requests x 300 keys x 8 heads 6.5 -> 6.2, 32 x 600 keys x 2 heads, 4 new each,
  // 11.6 -> 11.3, 16 x 300..4100 keys x 8 heads 31.4 -> 31.0.)
  pin_args(p);
  const AttnItem it = load_item(p.items, blockIdx.x);
  const Divisor G = p.group;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, g4 = lane >> 4;
  typedef __attribute__((address_space(3))) const bf16x8 *lds_b128_ptr;
  typedef __attribute__((address_space(3))) s16x4 *lds_tr_ptr;
  const uint32_t lds_base = lds_address(lds) + (uint32_t)(wave * NS * Shape::kTileBytes);
  const int lane_row = lane / CPR;
  uint32_t lane_chunk[UPP];                      // swizzled 16-byte chunk this lane fetches
#pragma unroll
  for (int i = 0; i < UPP; ++i)
    lane_chunk[i] = (uint32_t)(((lane % CPR) ^ swz<D>(i * KPU + lane / CPR)) << 4);
  // per-lane LDS addresses of the fragment reads, relative to a tile slot
  uint32_t k_lane[KK], v_lane[DB];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) k_lane[kk] = lds_base + (uint32_t)lds_off<D>(c16, 4 * kk + g4);
#pragma unroll
  for (int db = 0; db < DB; ++db)
    v_lane[db] = lds_base + (uint32_t)(TK * ROW + lds_off<D>(4 * g4 + (c16 >> 2), 2 * db + ((c16 & 3) >> 1)) +
                                       ((c16 & 1) << 3));
  const float slack = kRescaleThreshold / p.scale_log2e;
#pragma unroll
  for (int i = 0; i < UPP; ++i) __asm__ volatile("" : "+v"(lane_chunk[i]));
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) __asm__ volatile("" : "+v"(k_lane[kk]));
#pragma unroll
  for (int db = 0; db < DB; ++db) __asm__ volatile("" : "+v"(v_lane[db]));
  pin_item(it);
  if (it.req < 0) return;                        // idle padding entry
  const int P = it.prefix, S = it.suffix, T = P + S;
  const int row0 = it.row0;                      // the tile's packed rows: row0 .. row0+rows-1
  const int rows = S * G.d - row0 < Shape::kRows ? S * G.d - row0 : Shape::kRows;
  const int tok0 = G.quotient(row0);
  const ConstantPtr<int32_t> bt = constant_ptr(p.block_table + (int64_t)it.req * p.max_blocks);
  struct PageIds {
    int32_t p[2];
  };
  const int last_blk = (T - 1) / kPage;          // keys past the end are masked; any finite page will do for them
  auto pages_of = [&](int key0) -> PageIds {
    const int blk = key0 / kPage;
    return PageIds{{bt[blk < last_blk ? blk : last_blk], bt[blk + 1 < last_blk ? blk + 1 : last_blk]}};
  };
  auto key0_of = [&](int t) { return it.kv_begin + (wave + t * NW) * TK; };
  PageIds first_pages[NS];
#pragma unroll
  for (int t = 0; t < NS; ++t) first_pages[t] = pages_of(key0_of(t));
  __builtin_amdgcn_sched_barrier(0);             // on their way before the Q rows' addresses are formed

  // ---- Q rows into LDS, by the same copies as the keys and before them, so that
  // waiting for Q leaves the key copies in flight (loads into registers, which the
  // compiler waits for, would drain them: it does not see the copies).  The copy of
  // fragment (rb, kk) fetches for each lane the 16 bytes that the lane will read
  // back: row c16, dims 32kk+8*g4..+7.  The tile's first row stands in for rows past the end.
  // Q rows that do not lie on 16 bytes, which those copies do not promise to take,
  // go through registers, element by element.
  const uint32_t q_lds = lds_address(lds) + (uint32_t)(Shape::kRingBytes + wave * Shape::kQBytes);
  int limit[RB];                                 // last visible key of the lane's row
  const __bf16 *q0 = (const __bf16 *)p.q + ((int64_t)(it.q_off + tok0) * p.Hq + it.kv_head * G.d) * D;
  const i32x4 q_rows = block_resource(q0, (uint32_t)((G.quotient(row0 + rows - 1) - tok0) * p.Hq + G.d) * ROW);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = rb * 16 + c16;
    const bool valid = row < rows;
    const int from = row0 + (valid ? row : 0);
    const int tok = G.quotient(from), g = from - tok * G.d;
    limit[rb] = valid ? P + tok : -1;
    const uint32_t off = (uint32_t)(((tok - tok0) * p.Hq + g) * ROW + 16 * g4);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const uint32_t dst = q_lds + (uint32_t)((rb * KK + kk) * 1024);
      if (((uintptr_t)p.q & 15) == 0) {
        copy16_to_lds(q_rows, off + (uint32_t)(64 * kk), dst);
      } else {
        const __bf16 *from = q0 + off / 2 + 32 * kk;
        bf16x8 x;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = from[e];
        *(__attribute__((address_space(3))) bf16x8 *)(uintptr_t)(dst + (uint32_t)(lane * 16)) = x;
      }
    }
  }

  // ---- paged copies of this wave's tiles
#pragma unroll
  for (int t = 0; t < NS; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j) __asm__ volatile("" : : "s"(first_pages[t].p[j]));
  const PageSource src(p, it, ROW);
  auto copy_tile = [&](int key0, const PageIds &pages, int slot) {
#pragma unroll
    for (int pg = 0; pg < 2; ++pg) {
      const int blk = key0 / kPage + pg;
      const int pos0 = (blk < last_blk ? blk : last_blk) * kPage;
      const uint32_t dst = lds_base + (uint32_t)(slot * Shape::kTileBytes + pg * kPage * ROW);
      const int cached = src.first_new - pos0;   // rows of the page that come from the pool
      if (cached >= kPage) {
        const int valid = T - pos0 < kPage ? T - pos0 : kPage;   // the last page may hold anything past the sequence
        const i32x4 rk = src.old_rows(0, pages.p[pg], valid), rv = src.old_rows(1, pages.p[pg], valid);
        auto copy_page = [&](auto once) __attribute__((always_inline)) {
#pragma unroll
          for (int i = 0; i < UPP; ++i) {
            const uint32_t off = (uint32_t)((i * KPU + lane_row) * ROW) + lane_chunk[i];
            copy16_to_lds<decltype(once)::value>(rk, off, dst + (uint32_t)(i * 1024));
            copy16_to_lds<decltype(once)::value>(rv, off, dst + (uint32_t)(TK * ROW + i * 1024));
          }
        };
        if (ONCE && it.read_once) copy_page(std::true_type{});
        else copy_page(std::false_type{});
      } else if (cached <= 0) {
        const i32x4 rk = src.new_rows(0, pos0 - P), rv = src.new_rows(1, pos0 - P);
#pragma unroll
        for (int i = 0; i < UPP; ++i) {
          const uint32_t off = (uint32_t)(i * KPU + lane_row) * src.new_stride + lane_chunk[i];
          copy16_to_lds(rk, off, dst + (uint32_t)(i * 1024));
          copy16_to_lds(rv, off, dst + (uint32_t)(TK * ROW + i * 1024));
        }
      } else {                                   // the page where the cached prefix ends: its rows come from both
        const i32x4 ok = src.old_rows(0, pages.p[pg]), ov = src.old_rows(1, pages.p[pg]);
        const i32x4 nk = src.new_rows(0, 0, kPage - cached), nv = src.new_rows(1, 0, kPage - cached);
#pragma unroll
        for (int i = 0; i < UPP; ++i) {
          const int row = i * KPU + lane_row;
          if (row < cached) {
            const uint32_t off = (uint32_t)(row * ROW) + lane_chunk[i];
            copy16_to_lds(ok, off, dst + (uint32_t)(i * 1024));
            copy16_to_lds(ov, off, dst + (uint32_t)(TK * ROW + i * 1024));
          } else {
            const uint32_t off = (uint32_t)(row - cached) * src.new_stride + lane_chunk[i];
            copy16_to_lds(nk, off, dst + (uint32_t)(i * 1024));
            copy16_to_lds(nv, off, dst + (uint32_t)(TK * ROW + i * 1024));
          }
        }
      }
    }
  };

  // The new rows of a tile, from its ring slot to their pages, of the tokens whose
  // first packed row lies in the workgroup's row tile: every position belongs to
  // one tile of one workgroup per kv head.
  int own_lo = 0x7fffffff, own_hi = 0;
  if (p.k_new) {
    own_lo = P + G.quotient(row0 + G.d - 1);
    own_hi = P + G.quotient(row0 + rows + G.d - 1);
  }
  auto append_tile = [&](int key0, uint32_t slot) __attribute__((always_inline)) {
#pragma unroll
    for (int pg = 0; pg < 2; ++pg) {
      const int pos0 = key0 + pg * kPage;
      if (pos0 + kPage <= own_lo || pos0 >= own_hi) continue;
      const int64_t block = src.block_of(bt[pos0 / kPage]);
#pragma unroll
      for (int kv = 0; kv < 2; ++kv) {
        unsigned char *dst = (unsigned char *)(kv ? p.v_pool : p.k_pool) + block;
#pragma unroll
        for (int i = 0; i < UPP; ++i) {
          const int row = i * KPU + lane_row;
          const u32x4 data = *(__attribute__((address_space(3))) const u32x4 *)(uintptr_t)(
              lds_base + slot + (uint32_t)(kv * TK * ROW + pg * kPage * ROW + i * 1024 + lane * 16));
          if (pos0 + row >= own_lo && pos0 + row < own_hi) *reinterpret_cast<u32x4 *>(dst + row * ROW + lane_chunk[i]) = data;
        }
      }
    }
  };

  const int n_tiles = (it.kv_end - it.kv_begin + TK - 1) / TK;
  const int mine = n_tiles > wave ? (n_tiles - wave + NW - 1) / NW : 0;
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < mine) copy_tile(key0_of(t), first_pages[t], t);
  if (mine >= NS) wait_vmem<NS * COPIES>();      // Q was requested before any key
  else wait_vmem<0>();
  bf16x8 qf[RB][KK];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      qf[rb][kk] = *(lds_b128_ptr)(uintptr_t)(q_lds + (uint32_t)((rb * KK + kk) * 1024 + lane * 16));

  f32x4 oacc[DB][RB];
  float m_run[RB], l_run[RB], bound[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    m_run[rb] = bound[rb] = -1e30f;
    l_run[rb] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  for (int t = 0; t < mine; ++t) {
    const int ring = t % NS;
    const uint32_t slot = (uint32_t)(ring * Shape::kTileBytes);
    const PageIds ahead = pages_of(t + NS < mine ? key0_of(t + NS) : it.kv_begin);
    if (t + NS <= mine) wait_vmem<(NS - 1) * COPIES>();   // only later tiles' copies may still be on their way
    else wait_vmem<0>();
    if (key0_of(t) + TK > own_lo) append_tile(key0_of(t), slot);
    f32x4 s[2][RB];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) s[kb][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8 a = *(lds_b128_ptr)(uintptr_t)(k_lane[kk] + slot + (uint32_t)(kb * kPage * ROW));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          s[kb][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[rb][kk], s[kb][rb], 0, 0, 0);
      }
    }
    const int key0 = key0_of(t);
    if (key0 + TK - 1 > P + tok0) {              // some row may not see all of these keys
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (key0 + kb * 16 + 4 * g4 + r > limit[rb]) s[kb][rb][r] = -INFINITY;
    }
    // lazy running maximum, as in the prefill kernel
    float mx[RB];
    bool grow = false;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      mx[rb] = s[0][rb][0];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx[rb] = fmaxf(mx[rb], s[kb][rb][r]);
      grow |= mx[rb] > bound[rb];
    }
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const float m_new = fmaxf(m_run[rb], max_across_groups(mx[rb]));
        const float alpha = fast_exp2((m_run[rb] - m_new) * p.scale_log2e);
        bound[rb] = m_new + slack;
        m_run[rb] = m_new;
        l_run[rb] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 4; ++r) oacc[db][rb][r] *= alpha;
      }
    }
    bf16x8 pf[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float mc = m_run[rb] * p.scale_log2e;
      float sum = 0.f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float e = fast_exp2(fmaf(s[kb][rb][r], p.scale_log2e, -mc));
          sum += e;
          pf[rb][4 * kb + r] = (__bf16)e;
        }
      l_run[rb] += sum;
    }
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      union {
        s16x4 h[2];
        bf16x8 v;
      } a;
      a.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_ptr)(uintptr_t)(v_lane[db] + slot));
      a.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_ptr)(uintptr_t)(v_lane[db] + slot + (uint32_t)(kPage * ROW)));
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) oacc[db][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, pf[rb], oacc[db][rb], 0, 0, 0);
    }
    if (t + NS < mine) {
      wait_lds_reads();                          // the slot is free once this wave's reads of it are done
      copy_tile(key0_of(t + NS), ahead, ring);
    }
  }

  // ---- the waves' partial results meet in LDS
  wait_vmem<0>();
  __syncthreads();                               // every ring is idle from here on
  float *part = reinterpret_cast<float *>(lds);
  float *ml = part + (size_t)NW * Shape::kRows * Shape::kRowPitch;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int slot_row = wave * Shape::kRows + rb * 16 + c16;
    const float l_tot = sum_across_groups(l_run[rb]);
#pragma unroll
    for (int db = 0; db < DB; ++db)
      *reinterpret_cast<f32x4 *>(part + (size_t)slot_row * Shape::kRowPitch + 16 * db + 4 * g4) = oacc[db][rb];
    if (g4 == 0) {
      ml[2 * slot_row] = m_run[rb];
      ml[2 * slot_row + 1] = l_tot;
    }
  }
  __syncthreads();
  constexpr int TPR = D / 4;                     // threads per row, four dims each
  float *slot_out = it.part_slot >= 0 ? p.partials + (size_t)it.part_slot * Shape::kRows * (D + 2) : nullptr;
  for (int c = tid; c < rows * TPR; c += NT) {
    const int row = c / TPR, c4 = (c % TPR) * 4;
    float m = ml[2 * row];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, ml[2 * (w * Shape::kRows + row)]);
    float l = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int sr = w * Shape::kRows + row;
      const float e = fast_exp2((ml[2 * sr] - m) * p.scale_log2e);
      const f32x4 o = *reinterpret_cast<const f32x4 *>(part + (size_t)sr * Shape::kRowPitch + c4);
      l += e * ml[2 * sr + 1];
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] += e * o[r];
    }
    if (!slot_out) {
      store_out_row<D>(p, it.q_off, it.kv_head, G, row0 + row, c4, acc, 1.0f / l);
    } else {
      store_shared(slot_out + (size_t)row * D + c4, acc[0], acc[1]);
      store_shared(slot_out + (size_t)row * D + c4 + 2, acc[2], acc[3]);
      if (c4 == 0) store_shared(slot_out + (size_t)Shape::kRows * D + 2 * row, m, l);
    }
  }
  if (slot_out) {
    int *flag = reinterpret_cast<int *>(lds + Shape::kRingBytes);   // Q is no longer needed
    if (last_of_group(p, it.group, tid, flag)) merge_group<D, 1, 8, true>(p, it.group, G, Shape::kRows, tid, NT, 0, Shape::kRows);
  }
}

template <int D, int RB, bool ONCE>
static int launch_stream_t(const LaunchParams &p, hipStream_t st) {
  constexpr size_t lds_bytes = StreamShape<D, RB>::kLdsBytes;
  auto kernel = stream_attn_kernel<D, RB, ONCE>;
  static const hipError_t attr = hipFuncSetAttribute(
      (const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (attr != hipSuccess) return (int)attr;
  return launch_kernel(kernel, dim3((unsigned)p.num_items), dim3(StreamShape<D, RB>::NW * 64), lds_bytes, st, p.args);
}

template <int D>
static int launch_stream_d(const LaunchParams &p, hipStream_t st) {
  if (p.read_once) return p.tile_rows == 16 ? launch_stream_t<D, 1, true>(p, st) : launch_stream_t<D, 2, true>(p, st);
  return p.tile_rows == 16 ? launch_stream_t<D, 1, false>(p, st) : launch_stream_t<D, 2, false>(p, st);
}

int launch_stream(const LaunchParams &p, void *stream) {
  if (p.num_items == 0) return 0;
  hipStream_t st = (hipStream_t)stream;
  return p.d == 128 ? launch_stream_d<128>(p, st) : launch_stream_d<64>(p, st);
}

}  // namespace prism

// Device-side helpers shared by the attention kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <tuple>
#include <type_traits>

#include "prism_internal.h"

namespace prism {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

template <int D>
__device__ __forceinline__ int swz(int key) {
  if (D == 128) return ((key & 3) << 2) | ((key >> 2) & 3);
  return (((key >> 1) & 1) << 2) | ((key >> 2) & 3);
}

template <int D>
__device__ __forceinline__ int lds_off(int key, int chunk) {   // byte offset of a 16-byte chunk
  return key * (D * 2) + ((chunk ^ swz<D>(key)) << 4);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max over the two 32-lane halves of a wave, result in every lane
__device__ __forceinline__ float max_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// 16 bytes per lane from global memory straight into LDS: lane l's data lands
// at lds_base + 16*l (lds_base is wave-uniform and travels in M0).  The source
// is a buffer resource (wave-uniform base of one (page, head) block, in scalar
// registers) plus a per-lane byte offset, which keeps all address arithmetic
// off the vector ALU and makes a stray offset read zeros instead of faulting.
// Inline assembly, so that the compiler does not make later LDS reads of
// *other* slots wait for these copies; the kernels wait for them themselves
// (s_waitcnt vmcnt, and a workgroup barrier where waves share a tile) before a
// slot is read.
typedef __attribute__((ext_vector_type(4))) int32_t i32x4;
__device__ __forceinline__ i32x4 block_resource(const void *base, uint32_t bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)base;
  i32x4 r;
  r[0] = (int32_t)(uint32_t)a;
  r[1] = (int32_t)(uint32_t)((a >> 32) & 0xFFFFu);   // stride 0: a raw byte buffer
  r[2] = (int32_t)bytes;                             // offsets at or past this read as zero
  r[3] = 0x00020000;                                 // 32-bit untyped data
  return r;
}
// ONCE: rows that nothing else will ask for (no reuse in the caches).
template <bool ONCE = false>
__device__ __forceinline__ void copy16_to_lds(i32x4 rsrc, uint32_t lane_off, uint32_t lds_base) {
  // wave-uniform by construction; say so, in case the value was computed on the vector ALU
#pragma unroll
  for (int i = 0; i < 4; ++i) rsrc[i] = __builtin_amdgcn_readfirstlane(rsrc[i]);
  lds_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_base);
  // M0 (the LDS destination) is written and consumed inside this one statement.
  // The compiler rejects M0 in a clobber list (a reserved register), so the
  // kernels that copy this way use nothing for which the compiler would set
  // M0 itself (no LDS-DMA builtins, no indexed register moves, no messages);
  // tests/test_kernel_assembly.py checks the generated code for that.
  if constexpr (ONCE)
    __asm__ volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %0, 0 offen nt lds"
                     :
                     : "s"(rsrc), "v"(lane_off), "s"(lds_base)
                     : "memory");
  else
    __asm__ volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %0, 0 offen lds"
                     :
                     : "s"(rsrc), "v"(lane_off), "s"(lds_base)
                     : "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}

constexpr float kRescaleThreshold = 8.0f;   // log2 units

// Wait until at most N vector memory operations of this wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_vmem() {
  static_assert(N <= 63, "vmcnt is a 6-bit counter");
  __asm__ volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds_reads() { __asm__ volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }

// Read-only data at a wave-uniform address, by scalar loads.  Work items and
// block-table entries go this way: as vector loads they would queue behind the
// LDS copies, and waiting for one would wait for every copy before it.
template <class T>
using ConstantPtr = const T __attribute__((address_space(4))) *;
template <class T>
__device__ __forceinline__ ConstantPtr<T> constant_ptr(const T *p) {
  return (ConstantPtr<T>)(uintptr_t)p;
}
__device__ __forceinline__ AttnItem load_item(const AttnItem *items, int i) {
  ConstantPtr<int32_t> w = constant_ptr((const int32_t *)(items + i));
  AttnItem it;
  it.req = w[0]; it.kv_head = w[1]; it.row0 = w[2]; it.kv_begin = w[3]; it.kv_end = w[4];
  it.part_slot = w[5]; it.prefix = w[6]; it.suffix = w[7]; it.q_off = w[8]; it.group = w[9];
  it.read_once = w[10];
  return it;
}

// Have these in scalar registers from here on.
__device__ __forceinline__ void pin_args(const AttnArgs &p) {
  __asm__ volatile("" : : "s"(p.q), "s"(p.k_pool), "s"(p.v_pool), "s"(p.k_new), "s"(p.v_new), "s"(p.block_table),
                   "s"(p.items), "s"(p.Hq), "s"(p.Hkv), "s"(p.max_blocks), "s"(p.group.d), "s"(p.group.shift),
                   "s"(p.group.multiplier), "s"(p.scale_log2e));
}
__device__ __forceinline__ void pin_item(const AttnItem &it) {
  __asm__ volatile("" : : "s"(it.req), "s"(it.kv_head), "s"(it.row0), "s"(it.kv_begin), "s"(it.kv_end), "s"(it.part_slot),
                   "s"(it.prefix), "s"(it.suffix), "s"(it.q_off));
}

// All of a group but its arrival counter.
__device__ __forceinline__ ReduceGroup load_group(const ReduceGroup *groups, int i) {
  ConstantPtr<int32_t> w = constant_ptr((const int32_t *)(groups + i));
  ReduceGroup g;
  g.req = w[0]; g.kv_head = w[1]; g.row0 = w[2]; g.nsplit = w[3]; g.first_slot = w[4]; g.suffix = w[5]; g.q_off = w[6];
  g.arrived = 0;
  return g;
}

// ---- where the rows of one (page, kv head) block come from ------------------
// Cached positions lie in the pool.  When the call appends as well (k_new set),
// positions of the new tokens are read from the packed suffix arrays, so that
// attention does not depend on the append having happened; the page where the
// cached prefix ends inside takes rows from both.  Descriptors of new rows end
// after the request's last row: rows past the sequence arrive as zeros.
struct PageSource {
  const AttnArgs &p;
  const int P, S, row_bytes, q_off, kv_head;
  const int first_new;                           // positions from here on are packed rows
  const uint32_t new_stride;                     // bytes from one packed row of the head to the next
  __device__ __forceinline__ PageSource(const AttnArgs &args, const AttnItem &it, int row)
      : p(args), P(it.prefix), S(it.suffix), row_bytes(row), q_off(it.q_off), kv_head(it.kv_head),
        first_new(args.k_new ? it.prefix : 0x7fffffff), new_stride((uint32_t)(args.Hkv * row)) {}
  // byte offset of the (page, kv head) block in a pool
  __device__ __forceinline__ int64_t block_of(int32_t page) const {
    return ((int64_t)page * p.Hkv + kv_head) * (kPage * row_bytes);
  }
  // the first `rows` rows of a pool block, K (which = 0) or V (1)
  __device__ __forceinline__ i32x4 old_rows(int which, int32_t page, int rows = kPage) const {
    return block_resource((const unsigned char *)(which ? p.v_pool : p.k_pool) + block_of(page),
                          (uint32_t)(rows * row_bytes));
  }
  // up to `rows` packed rows from token tok on (clamped into the request's own rows)
  __device__ __forceinline__ i32x4 new_rows(int which, int tok, int rows = kPage) const {
    if (tok < 0) tok = 0;
    if (rows > S - tok) rows = S - tok;
    const int64_t first = ((int64_t)(q_off + tok) * p.Hkv + kv_head) * row_bytes;
    return block_resource((const unsigned char *)(which ? p.v_new : p.k_new) + first,
                          (uint32_t)(rows - 1) * new_stride + (uint32_t)row_bytes);
  }
};

// ---- split-KV partials between workgroups -----------------------------------
// Slot layout: fp32 O[tile_rows][D], then (m, l) per row.  Written and read with
// device-scope accesses: they go through to memory that every die sees, so the
// only ordering needed is "my stores are done" before the arrival is counted.
__device__ __forceinline__ void store_shared(float *dst, float a, float b) {
  const uint64_t v = (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32);
  __hip_atomic_store(reinterpret_cast<uint64_t *>(dst), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_shared(const float *src) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t *>(src), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

template <int D>
__device__ __forceinline__ void store_out_row(const AttnArgs &p, int q_off, int kv_head, const Divisor &G, int row, int c4,
                                              const f32x4 &acc, float scale) {
  const int tok = G.quotient(row);
  __bf16 *op = (__bf16 *)p.out + ((int64_t)(q_off + tok) * p.Hq + kv_head * G.d + (row - tok * G.d)) * D + c4;
  bf16x4 o4;
#pragma unroll
  for (int r = 0; r < 4; ++r) o4[r] = (__bf16)(acc[r] * scale);
  *reinterpret_cast<bf16x4 *>(op) = o4;
}

// Counts this workgroup's partial as written; true in the workgroup that is the
// last of its group (which leaves the counter at zero for the next call).
__device__ __forceinline__ bool last_of_group(const AttnArgs &p, int group, int tid, int *flag) {
  wait_vmem<0>();                                // this wave's partials have been acknowledged
  __syncthreads();                               // every wave's have
  if (tid == 0) {
    int32_t *arrived = &p.groups[group].arrived;
    const int32_t n = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = n + 1 == p.groups[group].nsplit;
    if (last) __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = last;
  }
  __syncthreads();
  return *flag != 0;
}

// out = sum_s e^{(m_s-m)c} O_s / sum_s e^{(m_s-m)c} l_s with m = max_s m_s (the
// associative log-sum-exp combine of softmax partials) for the rows of one
// group from row `begin` up to row `end` of the tile, by a workgroup of
// `threads`.  A thread owns four dims of R rows.  Bound by the latency of reads
// that miss the caches, so R x BATCH partials have all their reads in flight
// together.  SHARED: the partials were written by this very launch.
template <bool SHARED>
__device__ __forceinline__ float2 load_part(const float *src) {
  if constexpr (SHARED) return load_shared(src);
  else return *reinterpret_cast<const float2 *>(src);
}
template <int D, int R, int BATCH, bool SHARED>
__device__ __forceinline__ void merge_group(const AttnArgs &p, int group, const Divisor &G, int tile_rows, int tid, int threads,
                                            int begin, int end) {
  constexpr int TPR = D / 4;
  const ReduceGroup g = load_group(p.groups, group);
  const size_t slot_f = (size_t)tile_rows * (D + 2);
  const float *base = p.partials + (size_t)g.first_slot * slot_f;
  int n = g.suffix * G.d - g.row0;
  if (n > tile_rows) n = tile_rows;
  if (n > end) n = end;
  const int c4 = (tid % TPR) * 4, step = threads / TPR;
  for (int row0 = begin + tid / TPR; row0 < n; row0 += R * step) {
    float m[R], l[R];
    f32x4 acc[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      m[k] = -INFINITY;
      l[k] = 0.f;
      acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int s0 = 0; s0 < g.nsplit; s0 += BATCH) {
      float2 a[R][BATCH], x[R][BATCH], y[R][BATCH];
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int row = row0 + k * step < n ? row0 + k * step : n - 1;
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
          const float *slot = base + (s0 + i < g.nsplit ? s0 + i : g.nsplit - 1) * slot_f;
          a[k][i] = load_part<SHARED>(slot + (size_t)tile_rows * D + 2 * row);
          x[k][i] = load_part<SHARED>(slot + (size_t)row * D + c4);
          y[k][i] = load_part<SHARED>(slot + (size_t)row * D + c4 + 2);
        }
      }
#pragma unroll
      for (int k = 0; k < R; ++k) {
        float m_new = m[k];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) m_new = fmaxf(m_new, a[k][i].x);
        const float keep = fast_exp2((m[k] - m_new) * p.scale_log2e);
        m[k] = m_new;
        l[k] *= keep;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[k][r] *= keep;
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
          const float w = s0 + i < g.nsplit ? fast_exp2((a[k][i].x - m_new) * p.scale_log2e) : 0.f;
          l[k] += w * a[k][i].y;
          acc[k][0] += w * x[k][i].x;
          acc[k][1] += w * x[k][i].y;
          acc[k][2] += w * y[k][i].x;
          acc[k][3] += w * y[k][i].y;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < R; ++k)
      if (row0 + k * step < n)
        store_out_row<D>(p, g.q_off, g.kv_head, G, g.row0 + row0 + k * step, c4, acc[k], 1.0f / l[k]);
  }
}

// Wait until every MFMA issued so far has written its result (the longest one
// here takes 8 passes of 4 cycles): needed before accumulators that inline
// assembly names are read by anything but another MFMA.
__device__ __forceinline__ void mfma_drain() {
  __builtin_amdgcn_sched_barrier(0);
  __asm__ volatile("s_nop 15\n\ts_nop 3");
  __builtin_amdgcn_sched_barrier(0);
}

// f(integral_constant<int, B>) ... f(integral_constant<int, E-1>), expanded at
// compile time: the body sees its index as a constant expression.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Launch with the launch's own status as the return value: reading the
// runtime's last-error slot instead would also return, and clear, an error
// that an earlier call of the caller's left there.
template <class... Params, class... Args>
inline int launch_kernel(void (*kernel)(Params...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream,
                         Args... args) {
  static_assert(sizeof...(Params) == sizeof...(Args), "argument count");
  std::tuple<Params...> values{static_cast<Params>(args)...};
  void *ptrs[sizeof...(Params)];
  int i = 0;
  std::apply([&](auto &...v) { ((ptrs[i++] = (void *)&v), ...); }, values);
  return (int)hipLaunchKernel((const void *)kernel, grid, block, ptrs, lds_bytes, stream);
}

}  // namespace prism

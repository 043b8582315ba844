// Device side of the runtime (paper Section 5): the task bodies, the event protocol, the scheduler
// wavefronts and the three kernel templates.  Included by variants.hip, which instantiates the
// kernels, and by runtime.hip (host side), which only needs the argument structures.
//
// One persistent kernel: worker workgroups (one per CU, 512 threads = 8 wavefronts) walk their
// pre-enqueued (ahead-of-time) task list; before a task they wait until its dependent event's
// counter has reached epoch * required, after it they publish their stores and add one to the
// triggering event's counter.  Event counters only ever grow (no reset between steps).
//
// Memory ordering (the GPU has 8 XCDs with private, mutually non-coherent L2s).  Whole-cache
// write-back / invalidate fences cost tens of microseconds per hop with 256 workgroups, so the
// runtime never issues them.  Instead every datum that crosses workgroups inside the kernel
// (activations, split-KV partials, the K/V row appended this step, event counters) is written
// with agent-scope stores and read with agent-scope loads (ld_act / st_act below): such accesses
// are performed at the device coherence point, not in an XCD-private cache.  Producer side:
// agent-scope stores, every wavefront waits for its own stores to complete (vmcnt 0), workgroup
// barrier, one lane adds to the event counter.  Consumer side: one lane polls the counter,
// workgroup barrier, then agent-scope loads.  A marked tensor (kUnsetWord) needs none of it: each of its
// words says whether it has been written, the consumer's loads are its poll.  Weights, descriptors and cache rows of earlier
// steps are immutable during a step and use ordinary (non-temporal) loads.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <vector>

#include "mpk_internal.h"

namespace mpk {
const char* last_error();
size_t export_size(const HostGraph& g);
void export_graph(const HostGraph& g, void* buf);
void task_forms(const HostGraph& g, mpk_task_form* out);

// Everything that is fixed for the lifetime of a graph lives in one device-resident record that
// the kernels reach through a pointer (uniform address -> scalar loads on demand, nothing is
// pinned in registers for the whole kernel).
struct GraphConst {
  const TaskDesc* tasks;
  const EventDesc* events;
  uint32_t* counters;
  uint32_t* hier;            // counter blocks of hierarchical events
  const uint32_t* aot_off;
  const uint32_t* aot;
  const uint32_t* op_list;   // per-operator launch: task indices grouped by operator
  uint32_t* err;             // [0] error code, [1] abort flag, [2..3] detail
  const double* inv_freq;    // RoPE frequencies theta^(-2i/d), i < head_dim / 2
  uint32_t attn_shape;       // attn_shape_index of the model and its cache
  float* rope_tab;           // [2][batch][head_dim / 2] (cos, sin) of a step's rotation angles, even and odd steps, written by
                             // the embedding tasks; the copy of the other steps is put back to unset (kUnsetWord)
  uint32_t* grp_counters;    // arrival counters per (layer, sequence, KV head), monotonic
  uint64_t* trace;           // optional [n_tasks][kTraceSlots] timestamps (100 MHz), or null
  uint64_t timeout_ticks;
  uint32_t n_workers;
  uint32_t vocab, max_seq, n_q, n_kv, head_dim, batch;
  uint32_t lin_rows_max;     // largest number of weight rows (gate/up pairs count twice) of a linear task
  uint32_t lin_page_off;     // float offset of the LDS pre-load pages in the task area (0: none)
  // just-in-time launch (Section 5.2): scheduler event queues and worker task queues.  Entries
  // are 64-bit (ticket + 1) << 32 | id with tickets that only grow, so a slot is valid exactly
  // when it carries the ticket its reader expects; tails sit on their own 256-byte lines.
  uint32_t n_sched;          // scheduler wavefronts (0: every task is ahead-of-time)
  uint32_t evq_cap, wq_cap;  // powers of two
  uint64_t* evq_buf;         // [n_sched][evq_cap]
  uint32_t* evq_tail;        // [n_sched][64]
  uint32_t* sched_state;     // [n_sched][64]: [0] head ticket, [1] round-robin cursor (persist across steps)
  const uint32_t* sched_nev; // [n_sched] events a scheduler handles per step
  uint64_t* wq_buf;          // [n_workers][wq_cap]
  uint32_t* wq_tail;         // [n_workers][64]
  uint32_t* wq_head;         // [n_workers] head ticket (persists across steps)
  uint32_t start_event, terminal_event;
  // multi-token launch: written by mpk_decode_steps before the launch (stream-ordered copy)
  int32_t* tokens_out;   // [n_steps][batch] or null
  float* logits_all;     // [n_steps][batch][vocab] or null
  // paged KV cache (Section 6.1): row r of sequence b lives in page page_table[b][r >> page_shift]
  // of the layer's pool [kv_pages][n_kv][1 << page_shift][head_dim]; the table is device memory
  // that the serving task (or the caller, between launches) writes
  const int32_t* page_table;   // [batch][max_seq >> page_shift], or null
  const ServeDev* serve;       // serving state, or null
  uint32_t page_shift, kv_pages;
  int32_t serve_event;         // event the serving task triggers, -1 = none
  uint32_t mark_words;         // words of one copy of the marked tensors (0: none), copies for even and odd steps
  float* mark_base;
};

// Which instance of the attention task runs: head_dim 64 / 128, 1 / 2 / 4 / 8 query heads per KV head,
// contiguous or paged cache.
constexpr uint32_t attn_shape_index(uint32_t d, uint32_t grp, uint32_t paged) {
  return ((d == 128u ? 4u : 0u) + (grp == 8u ? 3u : grp == 4u ? 2u : grp == 2u ? 1u : 0u)) * 2u + paged;
}

// Per-step kernel arguments, passed by value.  Every device function taking it is force-inlined:
// a real call with a reference to it would make the compiler copy the struct to private memory.
// Tables that no kernel ever writes (the graph record, task and event descriptors, queues) are
// read through the constant address space: uniform reads then become scalar loads, which use
// their own counter and never queue behind (or wait for) the vector-memory weight stream.
#define MPK_CONST __attribute__((address_space(4)))
struct StepArgs {
  const MPK_CONST GraphConst* g;
  // what every wait and notification needs, by value: kernel arguments are in scalar registers
  // when the kernel starts, a field behind `g` costs a memory round trip on the critical path
  const TaskDesc* tasks;
  const EventDesc* events;
  uint32_t* counters;
  uint32_t* hier;
  uint32_t n_sched;
  uint32_t epoch;
  const int32_t* token_ids;
  const int32_t* positions;
  float* logits;
  // multi-token launch (greedy_loop graphs): the kernel runs n_steps decode steps; `step` counts
  // them and `epoch` grows with it.  positions[] stays as the host wrote it until the last step
  // (tasks run ahead of the sampling, so they take positions[b] + step).  16 bits each: the
  // struct is passed by value to every non-inlined task function and its fields sit in scalar
  // registers throughout the kernel; 16 bytes more of it slowed the single-step launch by 1 to 4 %.
  // For the same reason the output pointers of a multi-token launch and the trace buffer are in
  // the graph record instead.
  uint16_t step, n_steps;
  uint32_t flags;   // kTraceBit
};
static_assert(sizeof(StepArgs) == 80, "StepArgs grew: check the single-step launch time");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// A struct passed by value to a real (non-inlined) function travels through private memory and
// arrives in vector registers: to the compiler every field is then a per-lane value, so the
// descriptor reads behind it become vector loads and every branch on them an exec-mask branch.
// All lanes hold the same values: say so, field by field.
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename P>
__device__ __forceinline__ P uniform_ptr(P p) {
  const uint64_t v = (uint64_t)p;
  return (P)(((uint64_t)uniform_u32((uint32_t)(v >> 32)) << 32) | uniform_u32((uint32_t)v));
}
__device__ __forceinline__ StepArgs uniform_args(const StepArgs& a) {
  StepArgs u;
  u.g = uniform_ptr(a.g);
  u.tasks = uniform_ptr(a.tasks);
  u.events = uniform_ptr(a.events);
  u.counters = uniform_ptr(a.counters);
  u.hier = uniform_ptr(a.hier);
  u.n_sched = uniform_u32(a.n_sched);
  u.epoch = uniform_u32(a.epoch);
  u.token_ids = uniform_ptr(a.token_ids);
  u.positions = uniform_ptr(a.positions);
  u.logits = uniform_ptr(a.logits);
  u.step = (uint16_t)uniform_u32(a.step);
  u.n_steps = (uint16_t)uniform_u32(a.n_steps);
  u.flags = uniform_u32(a.flags);
  return u;
}

// Pointers that arrive through descriptors in memory are "generic" to the compiler, which then
// emits FLAT memory instructions: those may complete out of order, so every use has to wait for
// ALL outstanding memory operations (vmcnt(0) lgkmcnt(0)) and nothing pipelines.  Everything the
// kernels touch outside LDS is device memory: say so, and loads/stores become GLOBAL instructions
// that complete in order and can be waited for one by one.
#define MPK_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ MPK_GLOBAL T* as_global(T* p) {
  return (MPK_GLOBAL T*)p;
}
// 16-byte non-temporal load (weights, cache rows: streamed once, keep them out of the caches)
__device__ __forceinline__ u32x4 ld_stream16(const void* p) {
  return __builtin_nontemporal_load(as_global((const u32x4*)p));
}

// 16-byte non-temporal load at byte `off` of a run of memory that ends at byte `end`, with the hardware's
// range check: lanes at or past the end touch no memory and get zeros, and end = 0 is a load that costs an
// issue slot.  The pipelines below issue the same number of loads whatever there is left to fetch,
// because the compiler counts the loads in flight at compile time: behind a branch around some of them it
// waits for everything older.  (off + 16 must not wrap; p uniform.)  Matrix-core tasks, us a step against
// reading one cached line instead: 8B layers at batch 16 1283 -> 1244, odd sizes at batch 5 595 -> 574.
// Not for the vector body: such a load still takes 16 cycles of the CU's address unit, and the 36 a short
// task has no use for, times eight wavefronts, cost more than exact counts give (8B, batch 1: 2798 -> 3129).
__device__ __forceinline__ u32x4 ld_stream16_ranged(const void* p, uint32_t end, uint32_t off) {
  const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)end, 0x00020000);
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 2));   // 2: non-temporal
}

template <typename T>
__device__ __forceinline__ T ld_const_record(const T* p) {   // sizeof(T) a multiple of 16
  union {
    T rec;
    u32x4 v[sizeof(T) / 16];
  } u;
  const MPK_CONST u32x4* src = (const MPK_CONST u32x4*)p;
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 16; ++i) u.v[i] = src[i];
  return u.rec;
}
__device__ __forceinline__ TaskDesc ld_task(const StepArgs& a, uint32_t i) { return ld_const_record(a.tasks + i); }
__device__ __forceinline__ uint32_t ld_u32c(const uint32_t* p) { return *(const MPK_CONST uint32_t*)p; }

constexpr int kTraceSlots = 12;
// StepArgs::flags
constexpr uint32_t kTraceBit = 1u;      // per-task timestamps are recorded (buffer: GraphConst::trace)
constexpr uint32_t kJitterBit = 2u;     // every task starts after a pseudo-random delay (race hunting)
constexpr uint32_t kNoPreloadBit = 4u;  // no weight / cache-row request before a task's event wait
constexpr uint32_t kLoseNotifyBit = 8u; // worker 0 drops its notifications in this launch (watchdog test)
constexpr uint32_t kServeBit = 16u;     // serving launch: positions[] and token_ids[] are rewritten by the serving
                                        // task at the start of every step (absolute positions, read coherently)
constexpr uint32_t kOneStepBit = 32u;   // the launch runs ONE step (single-step entry points, a launch per step of a run):
                                        // nothing that earlier steps wrote can be stale in a cache
__device__ __forceinline__ void trace_mark(const StepArgs& a, const TaskDesc& t, int slot) {
  if ((a.flags & kTraceBit) && threadIdx.x == 0) as_global(a.g->trace)[(size_t)t.index * kTraceSlots + slot] = wall_clock64();
}

// MPK_DEBUG_JITTER: a delay of 0 .. 20 us, a hash of (task, step), before the task does anything.
// It shifts every task against every other differently in every step, so a consumer that does not
// really wait for its event, or a producer that notifies before its stores have completed, shows
// up as a wrong result instead of depending on the timing of an unloaded machine.
__device__ __forceinline__ void debug_jitter(const StepArgs& a, uint32_t task_index) {
  if (!(a.flags & kJitterBit)) return;
  if (threadIdx.x == 0) {
    uint32_t h = (task_index + 1u) * 2654435761u ^ (a.epoch * 40503u + 0x9E3779B9u);
    h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
    const uint64_t ticks = h % 2000u;   // the wall clock counts at 100 MHz
    const uint64_t t0 = wall_clock64();
    while (wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(8);
  }
  __syncthreads();
}

enum DevErr : uint32_t { DE_NONE = 0, DE_TIMEOUT = 1, DE_BAD_POSITION = 2, DE_BAD_TOKEN = 3, DE_BAD_META = 4, DE_BAD_PAGE = 5 };

// ------------------------------------------------------------------------------ device helpers
__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// fp32 -> bf16, round to nearest even; NaN stays a quiet NaN.
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
// The same sum without LDS traffic: four data-parallel-primitive steps inside each row of 16 lanes
// (lane ^ 1, lane ^ 2, mirror of 8, mirror of 16), then the four row totals.
__device__ __forceinline__ float wave_sum_dpp(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  v += dpp(v, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
  v += dpp(v, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
  v += dpp(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
  v += dpp(v, std::integral_constant<int, 0x140>{});   // row_mirror
  const int u = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(u, 0)) + __int_as_float(__builtin_amdgcn_readlane(u, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(u, 32)) + __int_as_float(__builtin_amdgcn_readlane(u, 48)));
}
// Sum of squares of a row staged 16 bytes a lane, in the order that 8 bytes a lane has: there lane i of wavefront w takes the
// pairs of inputs u * 512 + 64 w + i, u after u, and the lanes are added by wave_sum_dpp.  Sums of squares reach every
// output of a projection, and a last bit of them decides which way appended bf16 rows round: a wider load must not
// move them.  A load's lower 32 lanes hold an even u, the upper ones the next, lane l (of 32) the pairs of lanes
// 2 l and 2 l + 1: lower lane l sums for lane 2 l, upper lane l for lane 2 l + 1, after an exchange of halves.  us a step,
// four neighbouring inputs a thread / this: tiny model 41.6 / 42.1, 8B 2746 / 2755, 1B class 629 / 636.
struct SumSq {
  float s = 0.f;
  __device__ __forceinline__ void add(const float4& v) {
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.x), __float_as_uint(v.z), false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.y), __float_as_uint(v.w), false, false);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float a = __uint_as_float(x[h]), b = __uint_as_float(y[h]);
      s = fmaf(b, b, fmaf(a, a, s));
    }
  }
  __device__ __forceinline__ float sum() const {
    auto dpp = [](float x, auto ctrl) {
      return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    const auto o = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    float v = __uint_as_float(o[0]) + __uint_as_float(o[1]);   // lane ^ 1
    v += dpp(v, std::integral_constant<int, 0xB1>{});          // lane ^ 2
    v += dpp(v, std::integral_constant<int, 0x4E>{});          // mirror of 8
    v += dpp(v, std::integral_constant<int, 0x141>{});         // mirror of 16
    const int u = __float_as_int(v);
    return (__int_as_float(__builtin_amdgcn_readlane(u, 0)) + __int_as_float(__builtin_amdgcn_readlane(u, 8))) +
           (__int_as_float(__builtin_amdgcn_readlane(u, 16)) + __int_as_float(__builtin_amdgcn_readlane(u, 24)));
  }
};
// Four sums at once, each as wave_sum_dpp adds it up: every lane of the wavefront's row r of 16 lanes gets that of value r
// (sums of each row, then neighbouring rows of two values, and halves of two such pairs, put side by side by a swap and added.
// 22 vector operations; with the swaps first, which is another order, 10: 2B class at batch 2, four tokens 2110 us, now 2166).
__device__ __forceinline__ float wave_sum4(float v0, float v1, float v2, float v3) {
  auto dpp = [](float x, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  auto row_sum = [&](float v) {
    v += dpp(v, std::integral_constant<int, 0xB1>{});
    v += dpp(v, std::integral_constant<int, 0x4E>{});
    v += dpp(v, std::integral_constant<int, 0x141>{});
    v += dpp(v, std::integral_constant<int, 0x140>{});
    return __float_as_uint(v);
  };
  auto swap_add = [](auto sw) { return __uint_as_float(sw[0]) + __uint_as_float(sw[1]); };
  const float a = swap_add(__builtin_amdgcn_permlane16_swap(row_sum(v0), row_sum(v1), false, false));
  const float b = swap_add(__builtin_amdgcn_permlane16_swap(row_sum(v2), row_sum(v3), false, false));
  return swap_add(__builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false));
}
// ... and any other reduction (below: the largest value) the same way
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce_dpp(uint32_t v, Op op) {
  auto dpp = [](uint32_t x, auto ctrl) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xF, 0xF, true);
  };
  v = op(v, dpp(v, std::integral_constant<int, 0xB1>{}));
  v = op(v, dpp(v, std::integral_constant<int, 0x4E>{}));
  v = op(v, dpp(v, std::integral_constant<int, 0x141>{}));
  v = op(v, dpp(v, std::integral_constant<int, 0x140>{}));
  const int u = (int)v;
  return op(op((uint32_t)__builtin_amdgcn_readlane(u, 0), (uint32_t)__builtin_amdgcn_readlane(u, 16)),
            op((uint32_t)__builtin_amdgcn_readlane(u, 32), (uint32_t)__builtin_amdgcn_readlane(u, 48)));
}
__device__ __forceinline__ float wave_max_dpp(float v) {
  return __uint_as_float(wave_reduce_dpp(__float_as_uint(v), [](uint32_t x, uint32_t y) {
    return __float_as_uint(fmaxf(__uint_as_float(x), __uint_as_float(y)));
  }));
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// Sum over the whole workgroup; every thread gets the result.  red: >= 16 floats of LDS.
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < (int)(kThreads / 64); ++i) s += red[i];
  return s;
}

// Agent-coherent accessors for data produced and consumed by different workgroups in one launch.
__device__ __forceinline__ float ld_act(const float* p) {
  return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_act(float* p, float v) {
  __hip_atomic_store(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_act2(const float* p) {   // p 8-byte aligned
  uint64_t u = __hip_atomic_load(as_global((const uint64_t*)p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)u), __uint_as_float((uint32_t)(u >> 32)));
}
__device__ __forceinline__ void st_act2(float* p, float x, float y) {   // p 8-byte aligned
  __hip_atomic_store(as_global((uint64_t*)p), ((uint64_t)__float_as_uint(y) << 32) | __float_as_uint(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ld_relaxed(const uint32_t* p) {
  return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_relaxed64(const uint64_t* p) {
  return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_act_u32(uint32_t* p, uint32_t v) {
  __hip_atomic_store(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u32x4 ld_row16_coherent(const uint16_t* p) {   // p 16-byte aligned
  uint64_t a = __hip_atomic_load(as_global((const uint64_t*)p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint64_t b = __hip_atomic_load(as_global((const uint64_t*)p + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return u32x4{(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
}

// 16 and 8 bytes of a buffer at byte `off`, zeros past its end.  COHERENT: performed at the device's coherence point (words
// one by one, not 16 bytes at once) and never taken for an earlier load of the same place.
template <bool COHERENT>
__device__ __forceinline__ u32x4 ld_buffer16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, COHERENT ? (int)(16u | 0x80000000u) : 0));
}
__device__ __forceinline__ u32x2 ld_buffer8(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}
// Waits until at most N of this wavefront's vector-memory operations, the youngest, are in flight.
template <int N>
__device__ __forceinline__ void wait_vmem() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
  asm volatile("" ::: "memory");
}
// Waits for this wavefront's own loads and stores (and LDS operations).  A builtin and not assembly text:
// the compiler then knows that nothing is in flight any more.  Otherwise it takes the last loads of a
// task for pending in the next one, and copies into LDS (flat accesses to it, which may complete out of
// order) make it wait for everything in flight wherever it needs one load.
__device__ __forceinline__ void drain_vmem() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ float dot8(const u32x4& w, const float4& x0, const float4& x1, float acc) {
  acc = fmaf(bf16_lo(w.x), x0.x, acc);
  acc = fmaf(bf16_hi(w.x), x0.y, acc);
  acc = fmaf(bf16_lo(w.y), x0.z, acc);
  acc = fmaf(bf16_hi(w.y), x0.w, acc);
  acc = fmaf(bf16_lo(w.z), x1.x, acc);
  acc = fmaf(bf16_hi(w.z), x1.y, acc);
  acc = fmaf(bf16_lo(w.w), x1.z, acc);
  acc = fmaf(bf16_hi(w.w), x1.w, acc);
  return acc;
}

__device__ __forceinline__ void report(const StepArgs& a, uint32_t code, uint32_t d0, uint32_t d1) {
  if (atomicCAS(&a.g->err[0], 0u, code) == 0u) {
    a.g->err[2] = d0;
    a.g->err[3] = d1;
  }
}

// ------------------------------------------------------------------------------ task bodies
// cos and sin of position * inv_freq[i]: the angle is formed and reduced to [-pi, pi] in double.
__device__ __forceinline__ void rope_cs(const StepArgs& a, int32_t pos, uint32_t i, float* c, float* s) {
  double ang = (double)pos * as_global(a.g->inv_freq)[i];
  const double two_pi = 6.283185307179586476925286766559;
  ang -= two_pi * rint(ang / two_pi);
  double sd, cd;
  sincos(ang, &sd, &cd);
  *c = (float)cd;
  *s = (float)sd;
}

// T0: x[b] = E[token[b]] widened to fp32.  Eight elements a thread: the row is one round trip (an
// element at a time, loads and coherent stores took turns: 7 us for 4096 inputs, now 2).
// The task also leaves the step's rotation angles of its sequences in the rope table: they depend
// on the position alone, and every attention task of every layer that worked them out for itself (in
// double precision) spent 1 to 3 us on them ahead of its event.
__device__ __forceinline__ void body_embed(const TaskDesc& t, const StepArgs& a) {
  for (uint32_t b = t.b0; b < t.b1; ++b) {
    int32_t tok = (int32_t)ld_relaxed((const uint32_t*)a.token_ids + b);   // may come from the previous step's sampling task
    const int32_t pos = (a.flags & kServeBit) ? (int32_t)ld_relaxed((const uint32_t*)a.positions + b) : as_global(a.positions)[b] + (int32_t)a.step;
    if (tok < 0 || (uint32_t)tok >= a.g->vocab) {
      if (threadIdx.x == 0) report(a, DE_BAD_TOKEN, b, (uint32_t)tok);
      tok = 0;
    }
    const uint16_t* row = (const uint16_t*)t.w + (size_t)tok * t.K;
    float* out = t.out + (size_t)b * t.ld_out;
    for (uint32_t i = 8u * threadIdx.x; i < t.K; i += 8u * kThreads) {   // (the host checks that K is a multiple of 8)
      const u32x4 w = *as_global((const u32x4*)(row + i));
#pragma unroll
      for (int k = 0; k < 4; ++k) st_act2(out + i + 2 * k, bf16_lo(w[k]), bf16_hi(w[k]));
    }
    const uint32_t half = a.g->head_dim / 2u, i = kThreads - 1u - threadIdx.x;   // (threads without a share of a short row)
    if (i < half) {
      float cs, sn;
      rope_cs(a, pos, i, &cs, &sn);
      const uint32_t copy = a.g->batch * a.g->head_dim;
      float* tab = a.g->rope_tab + 2u * ((size_t)b * half + i);
      st_act2(tab + (a.epoch & 1u) * copy, cs, sn);
      st_act2(tab + (~a.epoch & 1u) * copy, __uint_as_float(kUnsetWord), __uint_as_float(kUnsetWord));
    }
  }
}

// T1/T8/T13: y = x * (1 / sqrt(mean(x^2) + eps)) * g, one batch row per task.
__device__ __forceinline__ void body_rmsnorm(const TaskDesc& t, float* lds) {
  const uint16_t* g = (const uint16_t*)t.w2;
  for (uint32_t b = t.b0; b < t.b1; ++b) {
    const float* x = t.in + (size_t)b * t.ld_in;
    float* y = t.out + (size_t)b * t.ld_out;
    float ss = 0.f;
    for (uint32_t i = threadIdx.x; i < t.K; i += kThreads) {
      float v = ld_act(x + i);
      ss = fmaf(v, v, ss);
    }
    ss = block_sum(ss, lds);
    float inv = 1.0f / sqrtf(ss / (float)t.K + t.f0);
    for (uint32_t i = threadIdx.x; i < t.K; i += kThreads) st_act(y + i, ld_act(x + i) * inv * bf16_to_f32(as_global(g)[i]));
  }
}

struct EventProbe {   // a look at an event whose loads may still be in flight
  uint32_t seen = 0, need = 1;
};
__device__ __forceinline__ EventProbe probe_event(const StepArgs& a, int32_t e, int lane);
__device__ __forceinline__ bool probe_reached(const EventProbe& p);
__device__ __forceinline__ bool wait_event(const StepArgs& a, int32_t e, uint32_t* s_flag);
__device__ __forceinline__ bool wait_event(const StepArgs& a, int32_t e, uint32_t* s_flag, const EventProbe& probe);
__device__ __forceinline__ StepArgs published_args();

// ------------------------------------------------------------------------------ marked tensors
// (see kUnsetWord.)  Loads of a marked tensor are repeated until none of them finds an unset word; mark_wait says
// whether to go round again.  What bounds a hop between two operators is the number of trips to the
// coherence point that follow one another: five with an event (store, its acknowledgement, notification, poll,
// input), two here.  us a step, events / marked: tiny model 57.1 / 42.6, 1B class at batch 1 784 / 747, 8B 2788 / 2758,
// 2B class at batch 2, four tokens 2700 / 2434, 70B layers 1804 / 1795.
// For batch 1 and 2 only: at batch 8 a worker's input is 128 KB, and 256 workers that load it before it is
// complete, and look at every word, take more from the producers than the hop gives (8B layers at batch 8 1078 -> 1155,
// 4B class at batch 4 811 -> 893).
__device__ __forceinline__ float mark_clean(float v) {   // (no arithmetic gives this pattern as far as is known: made certain)
  return __float_as_uint(v) == kUnsetWord ? __uint_as_float(0x7FC00000u) : v;
}
__device__ __forceinline__ bool mark_unset(float v) { return __float_as_uint(v) == kUnsetWord; }
__device__ __forceinline__ uint32_t mark_top(float v) { return __float_as_uint(v); }
__device__ __forceinline__ uint32_t mark_top(const float2& v) { return max(__float_as_uint(v.x), __float_as_uint(v.y)); }
// Puts a word of the other copy back to unset (two words: p 8-byte aligned).
__device__ __forceinline__ void mark_reset(float* p, int32_t twin) {
  if (twin) st_act_u32((uint32_t*)(p + (ptrdiff_t)twin * 64), kUnsetWord);
}
__device__ __forceinline__ void mark_reset2(float* p, int32_t twin) {
  const float u = __uint_as_float(kUnsetWord);
  if (twin) st_act2(p + (ptrdiff_t)twin * 64, u, u);
}
// Control word of the LDS: set by a wavefront that gives up waiting (the step is being aborted).
constexpr uint32_t kLdsAbortAt = 8;
// (its address space spelt out: a volatile access is a flat one otherwise, behind which the compiler waits for everything in flight)
typedef volatile __attribute__((address_space(3))) uint32_t lds_word_t;
__device__ __forceinline__ lds_word_t& abort_word() {
  extern __shared__ __align__(16) float dyn_lds[];
  return ((lds_word_t*)dyn_lds)[kLdsAbortAt];
}
struct MarkWait {
  uint32_t tries = 0;
  uint64_t t0 = 0;
};
// The whole wavefront calls it.  True: some lane has found an unset word, load again.  False: every lane has what it
// asked for, or the step is being aborted: mark_aborted then says so to every wavefront of the workgroup
// behind the next barrier, and the task ends by itself (mark_report).
__device__ __forceinline__ bool mark_wait(const StepArgs& a, bool unset, MarkWait& w) {
  if (!__any(unset)) return false;
  if (__builtin_expect((++w.tries & 255u) == 0, 0)) {
    const uint64_t now = wall_clock64();
    if (w.tries == 256u) w.t0 = now;
    if (now - w.t0 > a.g->timeout_ticks || __builtin_amdgcn_readfirstlane(ld_relaxed(a.g->err + 1)) != 0) {
      abort_word() = 1u;
      return false;
    }
  }
  return true;
}
__device__ __forceinline__ bool mark_aborted() {
  return __builtin_amdgcn_readfirstlane(abort_word()) != 0;
}

// A task has given up on its inputs: the watchdog's report, unless the step was being aborted already.
__device__ __noinline__ void mark_report(uint32_t event) {
  const StepArgs a = published_args();
  if (threadIdx.x == 0 && ld_relaxed(a.g->err + 1) == 0) {
    report(a, DE_TIMEOUT, event, blockIdx.x);
    __hip_atomic_store(as_global(a.g->err + 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// ------------------------------------------------------------------------------ linear tasks
// T2/T6/T9/T11/T14: y[b][c] = sum_j W[c][j] x[b][j] for output columns [c0, c1), all batch rows
// at once, with optional fused stages: RMSNorm of the input (TF_PRO_NORM), residual add
// (TF_EPI_RESID), silu(gate) * up (TF_GATEUP: column c needs weight rows c and F + c).
//
// Weight rows of a task ("ring rows": one per column, or the (gate, up) pair of each column) are
// split into 8 contiguous ranges, one per wavefront.  A wavefront walks its rows in pairs and
// every pair in segments of 4096 input elements; one (pair, segment) is a half block of
// 2 rows x 8 stages, a stage being 64 lanes x 16 bytes = 512 elements: 16 sixteen-byte loads per
// lane.  A wavefront owns two half-block buffers (32 KB, 256 KB per CU) and uses them in turn: it
// consumes one, requests that buffer's next half block at once, and turns to the other.  The
// compiler's count of the loads in flight does not survive the loop's back edge (it waits for
// both buffers before the first use of either), so a wavefront still drains its queue once per
// pair of half blocks; the eight wavefronts of a CU drift apart and cover for each other.
// Against ONE buffer of twice the size, requested whole and then consumed whole: the first
// buffer's request goes out half a block earlier, and a task with two rows per wavefront (the O
// and down projections of the 8B shape) pre-loads two segments instead of one.
//
// Cross-task pipelining (paper Section 5.3).  Weights never depend on an event, so a task
// requests its first two half blocks (256 KB per CU) BEFORE it waits for its dependent event:
// they stream in while the input vector is still being produced elsewhere.  At the end of a task
// wavefront 0 alone applies the epilogue, writes the outputs with coherent stores and waits for
// exactly those stores; the other wavefronts wait at a barrier meanwhile, and only then walk into
// the worker's next task and issue its first requests, while wavefront 0 notifies the triggering
// event, requests its own share and polls the next event.  (The others must not run ahead: all
// wavefronts of a CU share its path to memory, and output stores queued behind their requests
// were acknowledged up to 10 us late.)
// The buffers are local to a task on purpose: carried around the task loop instead, the
// compiler moves parts of them to scratch memory, and a scratch access in the middle of a request
// waits for every load issued before it.
constexpr int kHalfRows = 2, kRingStages = 8;
constexpr uint32_t kSegLen = 512u * kRingStages;   // input elements per half-block row
struct HalfRing {
  u32x4 s[kHalfRows][kRingStages];
};

__device__ __forceinline__ void ring_clear(HalfRing& ring) {
#pragma unroll
  for (int i = 0; i < kHalfRows; ++i)
#pragma unroll
    for (int u = 0; u < kRingStages; ++u) ring.s[i][u] = u32x4{0, 0, 0, 0};
}

// Short rows are packed: with K <= 2048 (1024) inputs, two (four) weight rows share one of the half block's
// rows, four (two) stages each, and the staged input is in LDS as often, so that loads and multiplies are
// those of one row of 4096.  (A row of 2048 alone left half of every half block's loads to repeat its last 16 bytes.)
// Sums are kept per two stages and handed on within a weight row (lin_chain).  us a step: 1B class at batch 1 702 ->
// 630 (gate/up phase of a layer 15.2 -> 11.8 us), 2B class at batch 2, four tokens 2190 -> 2135.
//
// A kernel set of its own for models with packed tasks: where none is, the choice costs every task 0.3 us (8B at
// batch 1 2736 -> 2789 us a step, tiny model 42.0 -> 44.7).
//
// Wavefront-uniform view of one linear task for one wavefront.
template <bool PACKED>
struct LinGeom {
  const uint16_t* W;
  uint32_t K, c0, F, gateup;
  uint32_t r0, r1;    // ring rows [r0, r1) of this wavefront within the task
  uint32_t nseg;      // segments per row
  uint32_t packed;    // weight rows per row of a half block: 1, 2 or 4
  __device__ __forceinline__ uint32_t pack() const { return PACKED ? packed : 1u; }
};

template <bool PACKED>
__device__ __forceinline__ LinGeom<PACKED> lin_geom(const TaskDesc& t, uint32_t wave) {
  LinGeom<PACKED> g;

  g.W = (const uint16_t*)t.w;
  g.K = t.K;
  g.c0 = t.c0;
  g.F = t.p0;
  g.gateup = (t.flags & TF_GATEUP) ? 1u : 0u;
  const uint32_t R = (t.c1 - t.c0) << g.gateup;
  g.packed = PACKED ? lin_pack(t.K, R) : 1u;
  constexpr uint32_t NW = kThreads / 64;
  // rows are dealt in pairs, packed ones in fours or eights (a half block holds as many; a (gate, up) pair stays in
  // one wavefront): every wavefront gets floor(pairs / 8) of them and the first pairs % 8 wavefronts one more, so
  // that a tile of any size -- tiles sized by worker speed are seldom multiples of 16 rows --
  // loads the wavefronts to within one pair of each other
  const uint32_t per = 2u * g.pack(), psh = g.pack() == 4u ? 3u : g.pack();   // (per = 1 << psh)
  const uint32_t P = (R + per - 1u) >> psh, base = P / NW, extra = P % NW;
  const uint32_t p0 = wave * base + min(wave, extra), p1 = p0 + base + (wave < extra ? 1u : 0u);
  g.r0 = min(per * p0, R);
  g.r1 = min(per * p1, R);
  g.nseg = (t.K + kSegLen - 1u) / kSegLen;
  return g;
}

// Position of a wavefront in its sequence of half blocks: rows [row0, row0 + 2 pack) x segment `seg`,
// segments of a pair first.  Two of them walk the sequence: one requests, one consumes.
struct LinCursor {
  uint32_t row0, seg;
};
template <bool PACKED>
__device__ __forceinline__ bool lin_valid(const LinGeom<PACKED>& g, const LinCursor& c) { return c.row0 < g.r1; }
template <bool PACKED>
__device__ __forceinline__ void lin_advance(const LinGeom<PACKED>& g, LinCursor& c) {
  if (++c.seg == g.nseg) {
    c.seg = 0;
    c.row0 += kHalfRows * g.pack();
  }
}

// The half block at a cursor.  Weight row s (below pack) of half-block row i: without gate/up ring row row0 + i pack + s;
// with it row0 + 2 s + i, so that i = 0 are gate rows and i = 1 their up rows.  Either way the weight rows of a
// half-block row follow one another in memory.
struct LinHalf {
  const uint16_t* p[kHalfRows];   // weight row 0, segment start (a half-block row without any repeats the first)
  uint32_t n[kHalfRows];          // weight rows there are (at least 1)
  uint32_t row0, nrows, seg, seglen;   // (nrows: ring rows, of unpacked ones)
};

template <bool PACKED>
__device__ __forceinline__ LinHalf lin_half(const LinGeom<PACKED>& g, const LinCursor& c) {
  LinHalf B;
  B.seg = c.seg;
  B.row0 = c.row0;
  B.seglen = min(kSegLen, g.K - c.seg * kSegLen);
  const uint32_t left = g.r1 - c.row0;   // ring rows
  B.nrows = min(left, (uint32_t)kHalfRows);
#pragma unroll
  for (int i = 0; i < kHalfRows; ++i) {
    uint32_t wrow;
    if constexpr (!PACKED) {
      const uint32_t r = c.row0 + min((uint32_t)i, B.nrows - 1u);
      wrow = g.gateup ? (g.c0 + (r >> 1) + ((r & 1u) ? g.F : 0u)) : g.c0 + r;
      B.n[i] = 1u;
    } else if (g.gateup) {   // (pairs are never cut: left is even)
      wrow = g.c0 + (c.row0 >> 1) + (i ? g.F : 0u);
      B.n[i] = min(g.pack(), left >> 1);
    } else {
      const bool there = left > (uint32_t)i * g.pack();
      wrow = g.c0 + c.row0 + (there ? (uint32_t)i * g.pack() : 0u);
      B.n[i] = min(g.pack(), there ? left - (uint32_t)i * g.pack() : left);
    }
    B.p[i] = g.W + (size_t)wrow * g.K + c.seg * kSegLen;
  }
  return B;
}

// This lane's element of stage u of half-block row i: past the end of a short segment (or of a packed row) the row's last
// 16 bytes (the staged input is zero there), for a weight row that does not exist the last one that does -- so every
// lane takes part in every load.
template <bool PACKED>
__device__ __forceinline__ const uint16_t* lin_lane(const LinGeom<PACKED>& g, const LinHalf& B, int i, int u, int lane) {
  const uint32_t sh = g.pack() == 1u ? 3u : (g.pack() == 2u ? 2u : 1u);   // 1 << sh stages a weight row
  const uint32_t o = min(((uint32_t)u & ((1u << sh) - 1u)) * 512u + (uint32_t)lane * 8u, B.seglen - 8u);
  return B.p[i] + min((uint32_t)u >> sh, B.n[i] - 1u) * g.K + o;
}
template <bool PACKED>
__device__ __forceinline__ bool lin_full(const LinGeom<PACKED>& g, const LinHalf& B) {   // 4096 inputs in a row of memory, twice
  return B.seglen * g.pack() == kSegLen && B.n[0] == g.pack() && B.n[1] == g.pack();
}
// Stages of a half block that hold inputs: past the end of a short row (or of a long row's last segment) there are only
// zeros to multiply by.  A projection of 256 inputs spent 0.6 of its 3.6 us on those, one of 2048 in tasks of a few rows 0.3 of 3.3.  us a
// step with all stages / without: tiny model 41.9 / 36.9, 1B class 637 / 631, 2B class at batch 2, four tokens 2165 / 2113, mixture of
// experts at batch 1 839 / 819.
template <bool PACKED>
__device__ __forceinline__ uint32_t lin_stages(const LinGeom<PACKED>& g, const LinHalf& B) {
  return g.pack() > 1u ? (uint32_t)kRingStages : (B.seglen + 511u) / 512u;
}
// f(0) .. f(n - 1), and up to the next power of two that is at least LEAST.
template <int LEAST, class F>
__device__ __forceinline__ void lin_each_stage(uint32_t n, F&& f) {
  static_for<0, LEAST>(f);
  if constexpr (LEAST < kRingStages) {
    if (n > (uint32_t)LEAST) {
      static_for<LEAST, 2 * LEAST>(f);
      if constexpr (2 * LEAST < kRingStages) {
        if (n > 2u * LEAST) {
          static_for<2 * LEAST, 4 * LEAST>(f);
          if constexpr (4 * LEAST < kRingStages) {
            if (n > 4u * LEAST) static_for<4 * LEAST, 8 * LEAST>(f);
          }
        }
      }
    }
  }
}
// Requests a half block, stage by stage.
template <int LEAST, bool PACKED>
__device__ __forceinline__ void lin_request(const LinGeom<PACKED>& g, const LinHalf& B, HalfRing& ring, int lane) {
  if (lin_full(g, B)) {   // one base address per row, constant stage offsets
#pragma unroll
    for (int u = 0; u < kRingStages; ++u)
#pragma unroll
      for (int i = 0; i < kHalfRows; ++i) ring.s[i][u] = ld_stream16(B.p[i] + lane * 8 + u * 512);
  } else {
    lin_each_stage<LEAST>(lin_stages(g, B), [&](auto uc) {
      constexpr int u = decltype(uc)::value;
#pragma unroll
      for (int i = 0; i < kHalfRows; ++i) ring.s[i][u] = ld_stream16(lin_lane(g, B, i, u, lane));
    });
  }
}

// Sums of a half-block row: one, or (packed kernels) one for every two stages.  A weight row of more stages than two goes on
// with the sum of the stages before, as it would in a half-block row of its own: what is packed and how
// does not change the order in which a row is added up.  A row's sum is the one of its last stages.
template <int NB, int NG>
__device__ __forceinline__ void lin_chain(int u, uint32_t pack, float (&acc)[kHalfRows][NG][NB]) {
  if constexpr (NG > 1) {
    static_assert(NG * 2 == kRingStages, "two stages a sum");
    if (u & 1) return;
    const bool goes_on = u == 0 || u == 4 ? pack == 1u : pack <= 2u;   // (u == 0: segments of a long row)
    const int q = u / 2, from = (q + NG - 1) % NG;
#pragma unroll
    for (int i = 0; i < kHalfRows; ++i)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[i][q][b] = goes_on ? acc[i][from][b] : 0.f;
  }
}
// Adds the half block's partial dot products to acc; w(i, u): this lane's weights of stage u of half-block row i.
template <int LEAST, int NB, int NG, class Weights>   // NG: sums per half-block row, of 8 / NG stages each
__device__ __forceinline__ void lin_consume_from(const LinHalf& B, Weights w, const float* xs, uint32_t Kp,
                                                 int lane, uint32_t pack, uint32_t stages, float (&acc)[kHalfRows][NG][NB]) {
  lin_each_stage<LEAST>(stages, [&](auto uc) {
    constexpr int u = decltype(uc)::value;
    lin_chain<NB, NG>(u, pack, acc);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float4* xp = (const float4*)(xs + (size_t)b * Kp + B.seg * kSegLen + u * 512 + lane * 8);
      const float4 x0 = xp[0], x1 = xp[1];
#pragma unroll
      for (int i = 0; i < kHalfRows; ++i) acc[i][u * NG / kRingStages][b] = dot8(w(i, u), x0, x1, acc[i][u * NG / kRingStages][b]);
    }
  });
  if constexpr (NG > 1) {   // (a row's sum is that of the last stages)
    if (stages <= 4u) {
#pragma unroll
      for (int i = 0; i < kHalfRows; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[i][NG - 1][b] = LEAST <= 2 && stages <= 2u ? acc[i][0][b] : acc[i][1][b];
    }
  }
}
template <int LEAST, int NB, int NG>
__device__ __forceinline__ void lin_consume(const LinHalf& B, const HalfRing& ring, const float* xs, uint32_t Kp,
                                            int lane, uint32_t pack, uint32_t stages, float (&acc)[kHalfRows][NG][NB]) {
  lin_consume_from<LEAST, NB, NG>(B, [&](int i, int u) -> const u32x4& { return ring.s[i][u]; }, xs, Kp, lane, pack, stages, acc);
}

// LDS pre-load pages (paper Section 5.3: data of a task that has not started yet is pre-loaded into
// shared-memory pages).  One page per wavefront holds one half block in the layout of a HalfRing:
// [row 0..1][stage 0..7][lane] x 16 bytes.  The loads go from device memory straight into LDS (no
// registers), so a page can be filled by one task and consumed by the worker's next one.
// LEAST: that of the multiplies, which read every stage of the page that it makes them take (whatever the LDS holds in a stage
// that nobody has filled may read as NaN, and 0 x NaN is NaN).
typedef __attribute__((address_space(3))) void* lds_ptr_t;
template <int LEAST, bool PACKED>
__device__ __forceinline__ void lin_request_page(const LinGeom<PACKED>& g, const LinHalf& B, u32x4* page, int lane) {
  lin_each_stage<LEAST>(lin_stages(g, B), [&](auto uc) {
    constexpr int u = decltype(uc)::value;
#pragma unroll
    for (int i = 0; i < kHalfRows; ++i)
      __builtin_amdgcn_global_load_lds(as_global((const u32x4*)lin_lane(g, B, i, u, lane)), (lds_ptr_t)(page + (i * kRingStages + u) * 64), 16, 0, 0);
  });
}
template <int LEAST, int NB, int NG>
__device__ __forceinline__ void lin_consume_page(const LinHalf& B, const u32x4* page, const float* xs, uint32_t Kp,
                                                 int lane, uint32_t pack, uint32_t stages, float (&acc)[kHalfRows][NG][NB]) {
  lin_consume_from<LEAST, NB, NG>(B, [&](int i, int u) { return page[(i * kRingStages + u) * 64 + lane]; }, xs, Kp, lane, pack, stages, acc);
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() carries a release fence, for
// which the compiler drains the vector-memory queue (s_waitcnt vmcnt(0)): with a pre-load of
// the next task in flight that would stall every wavefront, and the event notification behind
// it, until the whole pre-load has landed.  What the barriers of a linear task publish lives in
// LDS; data for other workgroups is published by wavefront 0 with its own wait.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ void signal_from_wave0(const StepArgs& a, const TaskDesc& t, int lane);
__device__ __forceinline__ void notify_task(const StepArgs& a, const TaskDesc& t);
__device__ __forceinline__ void notify_event(const StepArgs& a, int32_t e);
__device__ __forceinline__ void poll_event_wave0(const StepArgs& a, int32_t e, uint32_t* s_flag, int lane);
__device__ __forceinline__ void poll_event_or_jit_wave0(const StepArgs& a, int32_t e, uint32_t* s_flag, int lane, uint32_t jit_head);
// Hybrid launch (Section 5.2): a worker may start the linear task at the head of its ahead-of-time
// queue before that task's event is activated (so the weights are requested early), provided it
// keeps an eye on its just-in-time queue while it waits: a worker that blocked regardless could
// sit on the very tasks the awaited event depends on.  When a just-in-time task arrives first,
// the linear task gives up (kLinPreempted, task index in s_flag[1]); the worker runs that task and
// starts the linear task again.  (Running it from inside the wait would keep the pre-loaded
// weights live across a call: the compiler then moves them to scratch memory for good.)
// NoJit: all-ahead-of-time kernels, nothing to watch.
constexpr uint32_t kLinAbort = 0, kLinDone = 1, kLinPreempted = 2;
struct NoJit {
  static constexpr bool enabled = false, marks = false;
  uint32_t jit_head = 0;
  uint32_t n_next = 0, next[2] = {0, 0};   // the worker's next tasks, see warm_descriptors
};
struct NoJitMarks : NoJit {   // ... and the task's descriptor may be a marked one
  static constexpr bool marks = true;
};
struct JitWatch {
  static constexpr bool enabled = true, marks = false;
  uint32_t jit_head;   // the worker's consumer ticket of its just-in-time queue
};
// The first look at an event, by the first wavefront and ahead of the task's weight requests: loads
// complete in the order they were issued, so a poll behind the requests comes back behind the weights -- 3
// to 5 us when every compute unit asks for its share at once, which is what happens after an operator's
// last tasks.  The worker that finished last finds the event activated and stages its input behind
// the weights at once instead of a round trip after them.  With the exact load counts that it needs
// (drain_vmem), us a step: 8B layers at batch 8 1117 -> 1069, at batch 16 1245 -> 1195, 4B class 859 -> 828.
// (Input ahead of the weights where the event is active, behind a barrier that shares the probe: 1154 at
// batch 8 -- everybody's weights leave a round trip later.)
template <class Svc>
__device__ __forceinline__ EventProbe linear_probe(const StepArgs& a, int32_t wait_ev, uint32_t wave, int lane) {
  EventProbe p;   // (not reached)
  if (!Svc::enabled && wait_ev >= 0 && wave == 0) p = probe_event(a, wait_ev, lane);
  return p;
}
// Brings the records that the worker's next task starts and ends with -- its descriptor and those of
// its two events, six lines -- into the scalar cache.  Cold, a task pays a chain of three misses
// before its first request and another before its notification, 0.7 us each, on the path from
// one operator to the next.  One wavefront does it while the first one polls for this task's event.
// (us a step: 8B at batch 1 2830 -> 2799, 1B class 793 -> 788, serving burst 9515 -> 9378.)
__device__ __forceinline__ void warm_descriptors(const StepArgs& a, uint32_t ti) {
  const MPK_CONST TaskDesc* td = (const MPK_CONST TaskDesc*)(a.tasks + ti);
  const int32_t dep = td->dep_event, trig = td->trig_event;
  const uint32_t last = *((const MPK_CONST uint32_t*)td + 31);
  uint32_t v[4] = {0, 0, 0, 0};
  if (dep >= 0) {
    const MPK_CONST uint32_t* e = (const MPK_CONST uint32_t*)(a.events + dep);
    v[0] = e[0];
    v[1] = e[23];   // (96 bytes, 32-byte aligned: at most two lines)
  }
  if (trig >= 0) {
    const MPK_CONST uint32_t* e = (const MPK_CONST uint32_t*)(a.events + trig);
    v[2] = e[0];
    v[3] = e[23];
  }
  asm volatile("; descriptors of a later task" :: "s"(last), "s"(v[0]), "s"(v[1]), "s"(v[2]), "s"(v[3]));
}
template <class Svc>
__device__ __forceinline__ void warm_next(const StepArgs& a, const Svc& svc) {
  if (svc.n_next > 0) warm_descriptors(a, svc.next[0]);
  if (svc.n_next > 1) warm_descriptors(a, svc.next[1]);
}
// The wait of a linear task for its dependent event: kLinDone (activated), kLinAbort, kLinPreempted.
template <class Svc>
__device__ __forceinline__ uint32_t linear_wait(const StepArgs& a, int32_t wait_ev, uint32_t* s_flag, uint32_t wave, int lane,
                                                const Svc& svc, const EventProbe& probe) {
  if (wave == 0) {
    if constexpr (Svc::enabled) {
      poll_event_or_jit_wave0(a, wait_ev, s_flag, lane, svc.jit_head);
    } else {
      if (!probe_reached(probe)) poll_event_wave0(a, wait_ev, s_flag, lane);
      else if (lane == 0) *s_flag = 1;
    }
  }
  if constexpr (!Svc::enabled) {
    if (wave == 1) warm_next(a, svc);
  }
  lds_barrier();
  return __builtin_amdgcn_readfirstlane(*s_flag);   // (uniform; tell the compiler)
}

// LDS layout of a linear task (floats): xs [NB][K rounded up to 4096] | outbuf [max ring rows][NB]
// | resid [max columns][NB] | ssq [8][NB]; the two middle regions are sized by the compiler from
// the largest task of the graph (GraphConst::lin_rows_max).
//
// Runs task `t`.  wait_ev >= 0: wait for that event first (persistent kernel).  Returns whether
// the step is still alive (false: watchdog / abort).
template <int NB, bool MEGA, class Svc = NoJit, bool DEEP = false, bool PACKED = false>
__device__ __forceinline__ uint32_t linear_task(const TaskDesc& t, const StepArgs& a, float* lds, int32_t wait_ev,
                                                uint32_t* s_flag, const Svc& svc = Svc{}, uint32_t next_ti = 0) {
  // Batch 1: what is worked out from the lane number is worked out again in every task.  Otherwise the compiler
  // keeps some thirty such values in registers across the walk's calls of the task functions, and how well
  // this body does then hangs on which registers those happen to use (189 instead of 256 registers and
  // 2 spilled ones; us a step: 8B 2818 -> 2794, 1B class 795 -> 785).  Not with two rows (2725 -> 2731) or a
  // third buffer (long streams: gate/up of the 70B shape 143 -> 151 us a layer, the step unchanged).
  uint32_t tid = threadIdx.x;
  if constexpr (NB == 1 && !DEEP) asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: geometry stays scalar
  const uint32_t K = t.K, nb = t.b1 - t.b0, ncols = t.c1 - t.c0;
  // pages exist only in the all-ahead-of-time persistent kernel at batch 1 (the compiler sets the flags)
  constexpr bool kPages = MEGA && NB == 1 && !Svc::enabled;
  u32x4* page = (u32x4*)(lds + a.g->lin_page_off) + (size_t)wave * (kLinPageFloats / 4);
  const bool page_ready = kPages && (t.flags & TF_PAGE_READY), page_next = kPages && (t.flags & TF_PAGE_NEXT);
  const uint32_t Kp = (K + kSegLen - 1u) / kSegLen * kSegLen;
  const uint32_t rows_max = a.g->lin_rows_max;
  float* xs = lds;                                   // [NB][Kp]
  float* outbuf = xs + (size_t)NB * Kp;              // [rows_max][NB]
  float* res_lds = outbuf + (size_t)rows_max * NB;   // [rows_max][NB]
  float* ssq = res_lds + (size_t)rows_max * NB;      // [8][NB]
  constexpr int NG = PACKED ? 4 : 1;
  // How finely the stages of a short half block are left out.  Requests behind branches cannot be counted (see
  // ld_stream16_ranged), and packed kernels of one row are better off with all of them (1B class at batch 1 639 us a step with
  // requests left out, 628 without; multiplies left out one stage, two and four at a time 640, four only 628).
  constexpr int kLeast = PACKED && NB == 1 ? 4 : 1, kLeastAsked = PACKED && NB == 1 ? kRingStages : 1;
  const auto g = lin_geom<PACKED>(t, wave);
  HalfRing h0, h1;   // local to the task: nothing is live around the task loop, so they stay in registers
  ring_clear(h0);
  ring_clear(h1);
  const bool in_marked = Svc::marks && (t.flags & TF_IN_MARKED), in2_marked = Svc::marks && (t.flags & TF_IN2_MARKED);
  const bool preload = !(a.flags & kNoPreloadBit);   // off: the ablation of Section 6.5, Fig. 10
  const bool pro_norm = t.flags & TF_PRO_NORM;
  // ---- the input rows: 16 bytes a load, kSlices loads a lane and row in flight (12288 inputs in one round trip)
  constexpr uint32_t kSlices = 6, kSlice = 4u * kThreads, kChunk = kSlices * kSlice;   // (inputs)
  // this lane's inputs of a slice: 512 bytes of one half of it for the lower 32 lanes, of the other half for the upper (see SumSq)
  const uint32_t xat = kLinWaveInputs * wave + 4u * ((uint32_t)lane & 31u) + (kSlice / 2u) * ((uint32_t)lane >> 5);
  u32x4 xin[NB][kSlices];
  auto x_load = [&](uint32_t i0) {
#pragma unroll
    for (uint32_t b = 0; b < (uint32_t)NB; ++b) {
      // (a row that does not exist is an empty buffer: zeros)
      const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(uniform_ptr(t.in + (size_t)(t.b0 + b) * t.ld_in)), 0, b < nb ? (int)(4u * K) : 0, 0x00020000);
#pragma unroll
      for (uint32_t u = 0; u < kSlices; ++u)
        if (i0 + u * kSlice < K) xin[b][u] = ld_buffer16<true>(r, 4u * (i0 + u * kSlice + xat));
    }
  };
  // Every word of the loaded chunk has been written (wavefront-uniform).
  auto x_complete = [&](uint32_t i0) {
    uint32_t top = 0;
#pragma unroll
    for (uint32_t b = 0; b < (uint32_t)NB; ++b)
#pragma unroll
      for (uint32_t u = 0; u < kSlices; ++u)
        if (i0 + u * kSlice < K) top = max(top, max(max(xin[b][u].x, xin[b][u].y), max(xin[b][u].z, xin[b][u].w)));
    return !__any(top == kUnsetWord);
  };
  // A marked input is asked for three times: ahead of everything, between the two half blocks and behind them.  The
  // loads of a compute unit come back in the order they were issued, those of other wavefronts included: behind both
  // half blocks the input of a worker that is late anyway would be there 3 to 5 us after it could have
  // been, and a worker that is early by a fraction of a microsecond finds it on the second try.
  // (As compiled every look waits for more than its input.  x_complete stands behind the join of several paths, where the compiler
  // cannot count the loads in flight and waits for all of them, right behind the exact wait: the first look comes back
  // with the whole first half block, and the second half block leaves a round trip later than it could.)
  bool x_ok = false;
  if (in_marked && preload) x_load(0u);
  // the residual slice of this tile (tile-local, small): its round trip overlaps the staging
  const bool resid = t.flags & TF_EPI_RESID;
  float resv = 0.f;
  const float* resp = t.in2;
  auto out_row = [&](uint32_t i) { return NB == 1 ? 0u : (i >= ncols ? 1u : 0u); };   // output i of the tile: row, column
  auto out_col = [&](uint32_t i) { return NB == 1 ? i : (i >= ncols ? i - ncols : i); };
  if (resid && tid < nb * ncols) {
    const uint32_t bb = out_row(tid), cc = out_col(tid);
    resp += (size_t)(t.b0 + bb) * t.ld_out + t.c0 + cc;
    if (in2_marked) resv = ld_act(resp);
  }
  // the first gains of a folded RMSNorm are weights: requested before the event, so that the staging is one
  // round trip (the input) instead of two
  constexpr uint32_t kGainPre = 2;   // slices: the first 4096 inputs
  const auto gain = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(uniform_ptr((const uint16_t*)t.w2)), 0, pro_norm ? (int)(2u * K) : 0, 0x00020000);
  u32x2 gpre[kGainPre];
#pragma unroll
  for (uint32_t u = 0; u < kGainPre; ++u) {
    gpre[u] = u32x2{0u, 0u};
    if (pro_norm && u * kSlice < K) gpre[u] = ld_buffer8(gain, 2u * (u * kSlice + xat));
  }
  LinCursor rq{g.r0, 0u};   // next half block to request
  if (page_ready && lin_valid(g, rq)) lin_advance(g, rq);   // the first one is in this wavefront's page already
  // (every request site ends in an (empty) assembly statement of its own: otherwise the compiler
  // may merge the identical last loads of two sites into one whose destination is chosen at run
  // time, and a buffer addressed that way is moved from registers to scratch memory)
  // (the exact waits are builtins, one on each path: the compiler's own count of the loads in flight does not survive the
  // branches around the requests.  They are no condition of right results: a short row's half block is fewer loads than
  // they count, and the compiler waits by itself for what it reads.)
  if (preload && lin_valid(g, rq)) {
    lin_request<kLeastAsked>(g, lin_half(g, rq), h0, lane);
    lin_advance(g, rq);
    asm volatile("; first half block requested" ::: "memory");
    if (in_marked) wait_vmem<2 * kRingStages>();
  } else if (in_marked) {
    wait_vmem<0>();
  }
  if (in_marked && preload) {
    x_ok = x_complete(0u);
    if (!x_ok) x_load(0u);
  }
  const bool two = preload && lin_valid(g, rq);
  if (two) {
    lin_request<kLeastAsked>(g, lin_half(g, rq), h1, lane);
    lin_advance(g, rq);
    asm volatile("; second half block requested" ::: "memory");
  }
  // DEEP: a third buffer -- 384 KB per CU requested before the event and a deeper queue while
  // streaming.  A kernel variant of its own, picked for models whose linear tasks are large (70B
  // shape: -3 % per step); small tasks are bound by the hops between operators, where a bigger
  // burst ahead of the event poll and the input loads only delays those (8B shape: +3 %), and the
  // mere presence of the third buffer in the kernel costs the small shape 2 %.
  constexpr bool kThird = DEEP;
  HalfRing h2;
  bool three = false;
  if (kThird) {
    ring_clear(h2);
    three = preload && lin_valid(g, rq);
    if (three) {
      lin_request<kLeastAsked>(g, lin_half(g, rq), h2, lane);
      lin_advance(g, rq);
      asm volatile("; third half block requested" ::: "memory");
    }
  }
  if (in_marked && preload && !x_ok) {
    if (kThird && three) wait_vmem<4 * kRingStages>();
    else if (two) wait_vmem<2 * kRingStages>();
    else wait_vmem<0>();
    x_ok = x_complete(0u);
  }
  if (page_next) {
    // this task is short and has a long wait ahead: the first half block of every wavefront's
    // share of the worker's NEXT task goes into the pages now, two tasks ahead of its use
    const TaskDesc tn = ld_task(a, next_ti);
    const auto gn = lin_geom<PACKED>(tn, wave);
    const LinCursor cn{gn.r0, 0u};
    if (lin_valid(gn, cn)) lin_request_page<kLeast>(gn, lin_half(gn, cn), page, lane);
  }
  // ---- dependent event: wavefront 0 polls, the others wait at the barrier
  if (wait_ev >= 0) {
    const uint32_t w = linear_wait(a, wait_ev, s_flag, wave, lane, svc, EventProbe{});
    if (w != kLinDone) return w;   // aborted, or pre-empted by a just-in-time task: the requested weights are dropped
  } else if constexpr (Svc::marks) {
    if (wave == 1) warm_next(a, svc);
  }
  trace_mark(a, t, 1);
  if (!preload) {   // pre-loading switched off: the first requests go out only now
    if (lin_valid(g, rq)) {
      lin_request<kLeastAsked>(g, lin_half(g, rq), h0, lane);
      lin_advance(g, rq);
      asm volatile("; first half block requested after the event" ::: "memory");
    }
    if (lin_valid(g, rq)) {
      lin_request<kLeastAsked>(g, lin_half(g, rq), h1, lane);
      lin_advance(g, rq);
      asm volatile("; second half block requested after the event" ::: "memory");
    }
    if (kThird && lin_valid(g, rq)) {
      lin_request<kLeastAsked>(g, lin_half(g, rq), h2, lane);
      lin_advance(g, rq);
      asm volatile("; third half block requested after the event" ::: "memory");
    }
  }
  // ---- stage the input rows in LDS.  With TF_PRO_NORM the gain is folded in here (x * g) and
  // the row's 1/rms factor is applied to the finished dot products: W (x g inv) = inv * W (x g).
  if (resid && !in_marked && tid < nb * ncols) resv = ld_act(resp);
  SumSq ss[NB];
  for (uint32_t i0 = 0; i0 < Kp; i0 += kChunk) {
    if (i0 || !x_ok) {
      MarkWait mw;
      x_load(i0);
      while (in_marked && mark_wait(a, !x_complete(i0), mw)) x_load(i0);
    }
#pragma unroll
    for (uint32_t u = 0; u < kSlices; ++u) {
      const uint32_t i = i0 + u * kSlice + xat;
      if (i0 + u * kSlice >= Kp) continue;
      float gn[4] = {1.f, 1.f, 1.f, 1.f};
      if (pro_norm) {
        const u32x2 g2 = (i0 == 0 && u < kGainPre) ? gpre[u < kGainPre ? u : 0] : ld_buffer8(gain, 2u * i);
        gn[0] = bf16_lo(g2.x); gn[1] = bf16_hi(g2.x); gn[2] = bf16_lo(g2.y); gn[3] = bf16_hi(g2.y);
      }
#pragma unroll
      for (uint32_t b = 0; b < (uint32_t)NB; ++b) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i0 + u * kSlice < K) v = __builtin_bit_cast(float4, xin[b][u]);
        if (pro_norm) {
          if (i0 + u * kSlice < K) ss[b].add(v);
          v.x *= gn[0]; v.y *= gn[1]; v.z *= gn[2]; v.w *= gn[3];
        }
        if (g.pack() == 1u) {
          if (i < Kp) *(float4*)(xs + (size_t)b * Kp + i) = v;
        } else if (i < kSegLen / g.pack()) {   // (zeros past the input's end)
          for (uint32_t s = 0; s < kSegLen; s += kSegLen / g.pack()) *(float4*)(xs + (size_t)b * Kp + s + i) = v;
        }
      }
    }
  }
  if (pro_norm) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float v = ss[b].sum();
      if (lane == 0) ssq[wave * NB + b] = v;
    }
  }
  if (resid) {
    MarkWait mw;
    if (in2_marked)   // (written long ago: it is an input of this task's producers' producers)
      while (mark_wait(a, mark_unset(resv), mw))
        if (mark_unset(resv)) resv = ld_act(resp);
    // (not marked: complete only now that this wavefront has seen input; without any it has no output here, see lin_resid_seen)
    if (in_marked && !in2_marked && tid < nb * ncols) resv = ld_act(resp);
    if (tid < nb * ncols) res_lds[tid] = resv;
    for (uint32_t i0 = kThreads; i0 < nb * ncols; i0 += kThreads) {   // more than 512 outputs per task: rare
      const uint32_t i = i0 + tid, bb = out_row(i), cc = out_col(i);
      const float* p = t.in2 + (size_t)(t.b0 + bb) * t.ld_out + t.c0 + cc;
      float v = i < nb * ncols ? ld_act(p) : 0.f;
      if (in2_marked)
        while (mark_wait(a, mark_unset(v), mw))
          if (mark_unset(v)) v = ld_act(p);
      if (i < nb * ncols) res_lds[i] = v;
    }
  }
  lds_barrier();
  trace_mark(a, t, 2);
  // ---- stream this wavefront's rows: the two buffers in turn
  {
    float acc[kHalfRows][NG][NB];
#pragma unroll
    for (int i = 0; i < kHalfRows; ++i)
#pragma unroll
      for (int q = 0; q < NG; ++q)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[i][q][b] = 0.f;
    // the rows are complete with their last segment: reduce across lanes, results to LDS
    auto finish = [&](const LinHalf& B) {
      if (B.seg + 1 != g.nseg) return;
      if (g.pack() == 1u) {
#pragma unroll
        for (int i = 0; i < kHalfRows; ++i)
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            const float v = wave_sum_dpp(acc[i][NG - 1][b]);
            if (lane == 0 && (uint32_t)i < B.nrows) outbuf[(size_t)(B.row0 + i) * NB + b] = v;
          }
      } else if constexpr (PACKED) {
        auto out4 = [&](float v, uint32_t i, uint32_t s, int b) {   // (a row of 16 lanes has weight row s of half-block row i)
          const uint32_t r = B.row0 + (g.gateup ? 2u * s + i : i * g.pack() + s);
          if ((lane & 15) == 0 && r < g.r1) outbuf[(size_t)r * NB + b] = v;
        };
        const uint32_t k = (uint32_t)lane >> 4;   // the row of lanes has value k of a wave_sum4
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          if (g.pack() == 2u) {
            out4(wave_sum4(acc[0][1][b], acc[0][3][b], acc[1][1][b], acc[1][3][b]), k >> 1, k & 1u, b);
          } else {
            out4(wave_sum4(acc[0][0][b], acc[0][1][b], acc[0][2][b], acc[0][3][b]), 0u, k, b);
            out4(wave_sum4(acc[1][0][b], acc[1][1][b], acc[1][2][b], acc[1][3][b]), 1u, k, b);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < kHalfRows; ++i)
#pragma unroll
        for (int q = 0; q < NG; ++q)
#pragma unroll
          for (int b = 0; b < NB; ++b) acc[i][q][b] = 0.f;
    };
    LinCursor cs{g.r0, 0u};
    if (page_ready && lin_valid(g, cs)) {   // (requested a whole task ago: long since landed)
      const LinHalf B = lin_half(g, cs);
      lin_consume_page<kLeast, NB, NG>(B, page, xs, Kp, lane, g.pack(), lin_stages(g, B), acc);
      finish(B);
      lin_advance(g, cs);
    }
    while (lin_valid(g, cs)) {
      {
        const LinHalf B = lin_half(g, cs);
        lin_consume<kLeast, NB, NG>(B, h0, xs, Kp, lane, g.pack(), lin_stages(g, B), acc);
        finish(B);
        lin_advance(g, cs);
      }
      if (lin_valid(g, rq)) {
        lin_request<kLeastAsked>(g, lin_half(g, rq), h0, lane);
        lin_advance(g, rq);
        asm volatile("; first buffer requested again" ::: "memory");
      }
      if (!lin_valid(g, cs)) break;
      {
        const LinHalf B = lin_half(g, cs);
        lin_consume<kLeast, NB, NG>(B, h1, xs, Kp, lane, g.pack(), lin_stages(g, B), acc);
        finish(B);
        lin_advance(g, cs);
      }
      if (lin_valid(g, rq)) {
        lin_request<kLeastAsked>(g, lin_half(g, rq), h1, lane);
        lin_advance(g, rq);
        asm volatile("; second buffer requested again" ::: "memory");
      }
      if (kThird) {
        if (!lin_valid(g, cs)) break;
        {
          const LinHalf B = lin_half(g, cs);
          lin_consume<kLeast, NB, NG>(B, h2, xs, Kp, lane, g.pack(), lin_stages(g, B), acc);
          finish(B);
          lin_advance(g, cs);
        }
        if (lin_valid(g, rq)) {
          lin_request<kLeastAsked>(g, lin_half(g, rq), h2, lane);
          lin_advance(g, rq);
          asm volatile("; third buffer requested again" ::: "memory");
        }
      }
    }
  }
  // 1/rms by the wavefront with the fewest rows, beside the others' last ones (the sums are complete since the last barrier).
  // Behind the barrier, with the epilogue's divisions by the tile's width, it was 0.1 to 0.2 us of every hop: tiny model 36.4
  // -> 35.5 us a step, 2B class at batch 2, four tokens 2111 -> 2090, 8B 2744 -> 2739.
  if (pro_norm && wave == kThreads / 64u - 1u) {
    float inv_rms[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float ss = 0.f;
#pragma unroll
      for (int w = 0; w < (int)(kThreads / 64); ++w) ss += ssq[w * NB + b];
      inv_rms[b] = 1.0f / sqrtf(ss / (float)K + t.f0);
    }
    if (lane == 0)
#pragma unroll
      for (int b = 0; b < NB; ++b) ssq[b] = inv_rms[b];
  }
  lds_barrier();
  trace_mark(a, t, 3);
  // ---- wavefront 0: epilogue, outputs, notification, then its own share of the pre-load
  const bool out_marked = Svc::marks && (t.flags & TF_OUT_MARKED);
  const bool aborted = in_marked && mark_aborted();   // (before the last barrier: the flag is then everybody's)
  if (wave == 0) {
    float* outp = (t.flags & TF_OUT_LOGITS) ? a.logits : t.out;
    float inv_rms[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) inv_rms[b] = pro_norm ? ssq[b] : 1.0f;
    for (uint32_t i = lane; i < ncols * nb; i += 64) {
      const uint32_t cc = out_col(i), bb = out_row(i);
      float inv = inv_rms[0];
#pragma unroll
      for (int b = 1; b < NB; ++b) inv = (bb == (uint32_t)b) ? inv_rms[b] : inv;
      float v;
      if (g.gateup) {
        const float gte = outbuf[(size_t)(2 * cc) * NB + bb] * inv, up = outbuf[(size_t)(2 * cc + 1) * NB + bb] * inv;
        v = gte / (1.0f + expf(-gte)) * up;
      } else {
        v = outbuf[(size_t)cc * NB + bb] * inv;
      }
      if (t.flags & TF_EPI_RESID) v = res_lds[bb * ncols + cc] + v;
      st_act(outp + (size_t)(t.b0 + bb) * t.ld_out + t.c0 + cc, out_marked ? mark_clean(v) : v);
    }
    if (out_marked)
      for (uint32_t i = lane; i < ncols * nb; i += 64) mark_reset(outp + (size_t)(t.b0 + out_row(i)) * t.ld_out + t.c0 + out_col(i), t.twin);
    if (MEGA && !(out_marked && t.trig_event < 0)) {   // wait for exactly these stores
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      drain_vmem();
      trace_mark(a, t, 7);
    }
  }
  if (MEGA) {
    // Wavefronts 1..7 issue the next task's requests only now.  Ordering inside ONE wavefront is
    // not enough: all wavefronts of a CU share its path to memory, and behind 224 freshly issued
    // 1 KB loads the few output stores of wavefront 0 were acknowledged up to 10 us late (in-kernel
    // trace), which delays the event for every consumer -- the hop is the critical path, the
    // pre-load has slack.  (Releasing them once the stores have been issued, not acknowledged, was
    // measured too: 0.6 % slower per step on the 8B shape.)
    lds_barrier();
    if (wave == 0) {
      if (t.trig_event >= 0 && lane == 0) notify_task(a, t);
      trace_mark(a, t, 4);
    }
  }
  return aborted ? kLinAbort : kLinDone;
}

// ------------------------------------------------------------------------------ linear tasks, batch 3..16
// The same operator for 3 to 16 batch rows, on the matrix cores.  At batch 8 the vector ALUs
// would need about as many cycles for the multiply-adds as HBM needs to deliver the weights; one
// v_mfma_f32_16x16x32_bf16 does 16 weight rows x 32 inputs x 16 batch columns at once.
//   A operand = weights: lane l holds row (l % 16) of a 16-row tile and 8 of the 32 inputs of the
//     multiply: 16 bytes straight from HBM, no conversion (loaded as 8 rows x 128 bytes per
//     instruction and put in place by one DPP move per register: see mfma_job_packed).
//   B operand = activations: lane l holds batch column (l % 16), the same 8 inputs, as bf16.
//     Activations are fp32: x is split into THREE bf16 terms, hi = bf16(x), mid = bf16(x - hi),
//     lo = bf16(x - hi - mid).  Each conversion rounds to nearest and each remainder is exact in
//     fp32, so hi + mid + lo = x exactly (8 + 8 + 8 significand bits; finite x below bf16's largest and above
//     its subnormals), every product with a bf16 weight is exact, and what is rounded are the fp32 sums.
//     Their error against 64 bits is no larger than the vector body's (4B class at batch 4, logits:
//     1.47e-6 there, 1.30e-6 here).
//     (Two terms leave x to 2^-18: logits near zero then miss the element-wise bound.)
//   D: lane l holds batch column (l % 16), tile rows 4 (l / 16) .. + 3.
// The input is staged in LDS as fp32, whole when it fits (4096 inputs up to batch 8, 2048 above;
// longer inputs in chunks of that size), the row stride padded (mfma_row_pad) so that the lanes of a
// fragment spread over the banks; the wavefronts split it into the three terms as they go,
// so no barrier separates the staging of one part from the multiplies of another.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t pack_bf16_rne(float x, float y) {   // the hardware's packed conversion
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x, y}, bf16x2));
}
// (x, y) -> packed bf16 pairs hi, mid, lo with hi + mid + lo = (x, y) exactly
__device__ __forceinline__ void split_hi_mid_lo(float x, float y, uint32_t* hi, uint32_t* mid, uint32_t* lo) {
  const uint32_t h = pack_bf16_rne(x, y);
  const float rx = x - bf16_lo(h), ry = y - bf16_hi(h);
  const uint32_t m = pack_bf16_rne(rx, ry);
  *hi = h;
  *mid = m;
  *lo = pack_bf16_rne(rx - bf16_lo(m), ry - bf16_hi(m));
}

// Geometry of one matrix-core job: K inputs x nb staged rows x nrt 16-row weight tiles (nrt <= 32).
// Uniform over the wavefront (wave comes from readfirstlane).
//
// The input stays in LDS as fp32, a chunk of up to mfma_kchunk(nb) inputs at a time (the whole of
// it for every operator of the benchmark shapes), so that there is one staging pass and no
// barrier inside the multiply loop; each wavefront turns the 8 inputs x 1 row a lane needs for a
// multiply into the three bf16 terms on the fly.
//
// The 8 wavefronts form rg row groups x ks K slices (rg = 1, 2, 4 or 8, the smallest with
// 4 rg >= nrt).  Wavefront (slice s, group g) owns row tiles g, g + rg, g + 2 rg, g + 3 rg (those
// below nrt: nrtw of them) and, in every chunk, the s-th of ks nearly equal runs of 64-input
// "k-groups".  It works in rounds of 8 weight fragments (32 inputs x 16 rows, 1 KB each) = 4 slot
// groups of kMfmaFrags = 2 fragments, two rounds in flight (16 KB per wavefront, 32 MB over the
// chip: rounds of twice the size keep 64 MB in flight, which HBM does not need and which stands in
// the way of every store acknowledgement, counter update and poll of the hops between operators
// -- 8B shape at batch 8: 5.27 -> 5.10 ms per step; rounds of half the size starve: 5.93);
// slot group q always adds into accumulator q:
//   nrtw >= 3: one k-group per round, slot group q = row tile q of the wavefront
//   nrtw == 2: two k-groups per round, slot group q = (k-group q / 2, row tile q % 2)
//   nrtw == 1: four k-groups per round, slot group q = k-group q
// so the fragments of a k-group's inputs are converted once and used by all row tiles of the
// round.  The epilogue adds the accumulators of a row tile over slot groups and slices in a
// fixed order (mfma_dot).
constexpr uint32_t kMfmaFrags = 2;
struct MfmaGeom {
  uint32_t K, nb, nrt;
  uint32_t rg, rgsh, ks;   // row groups (= 1 << rgsh) x K slices = 8
  uint32_t my_g, my_s;
  uint32_t nrtw;         // row tiles of this wavefront: 0 .. 4
  uint32_t kgsh;         // k-groups per round: 1 << kgsh = 1, 2 or 4
};
__device__ __forceinline__ uint32_t mfma_group_tiles(uint32_t nrt, uint32_t rgsh, uint32_t g) {
  return g < nrt ? min(4u, (nrt - g + (1u << rgsh) - 1u) >> rgsh) : 0u;
}
__device__ __forceinline__ MfmaGeom mfma_geom(uint32_t K, uint32_t nb, uint32_t nrt, uint32_t wave) {
  MfmaGeom G;
  G.K = K; G.nb = nb; G.nrt = nrt;
  const uint32_t rgsh = (nrt > 4u ? 1u : 0u) + (nrt > 8u ? 1u : 0u) + (nrt > 16u ? 1u : 0u), rg = 1u << rgsh;
  G.rg = rg;
  G.rgsh = rgsh;
  G.ks = 8u >> rgsh;
  G.my_g = wave & (rg - 1u);
  G.my_s = wave >> rgsh;
  G.nrtw = mfma_group_tiles(nrt, rgsh, G.my_g);
  G.kgsh = G.nrtw >= 3u ? 0u : (G.nrtw == 2u ? 1u : 2u);
  return G;
}

// 8 consecutive fp32 inputs of one staged row -> packed bf16 terms hi, mid, lo (4 words each)
__device__ __forceinline__ void split8(const float4& p, const float4& q, u32x4* hi, u32x4* mid, u32x4* lo) {
  uint32_t h[4], m[4], l[4];
  split_hi_mid_lo(p.x, p.y, &h[0], &m[0], &l[0]);
  split_hi_mid_lo(p.z, p.w, &h[1], &m[1], &l[1]);
  split_hi_mid_lo(q.x, q.y, &h[2], &m[2], &l[2]);
  split_hi_mid_lo(q.z, q.w, &h[3], &m[3], &l[3]);
  *hi = u32x4{h[0], h[1], h[2], h[3]};
  *mid = u32x4{m[0], m[1], m[2], m[3]};
  *lo = u32x4{l[0], l[1], l[2], l[3]};
}
__device__ __forceinline__ u32x4 select4(bool c, const u32x4& x, const u32x4& y) {
  return u32x4{c ? x.x : y.x, c ? x.y : y.y, c ? x.z : y.z, c ? x.w : y.w};
}
// `src` of the lane N before this one in its row of 16 lanes (N = 0: of this lane), in the lanes of the fours of a row that
// BANKS names (bit k: lanes 4 k .. 4 k + 3); `old` in the others.
template <int N, int BANKS>
__device__ __forceinline__ uint32_t row_lanes(uint32_t old, uint32_t src) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)src, N ? 0x120 + N : 0xE4, 0xF, BANKS, false);
}
// The activation operands of a k-group's two multiplies (U = 0, 1), with PACK terms side by side in the columns, from the
// group's 16 inputs that the multiplies want of this lane's row: at `src` those that this lane splits, and their gains if `norm`.
// Every number is split once: the 16 / PACK-fold lanes that hold one row in different column groups share its 16 inputs and
// hand the terms round.
//   PACK 2: columns 0..7 (hi) split the first multiply's 8 inputs, columns 8..15 (mid) the second's
//   PACK 3: column group q of four splits inputs 4 q .. 4 q + 3 of the 16
// (Splitting all 16 in every lane and keeping one term was 128 vector instructions a k-group and wavefront, now 76 and
// 54, and as many reads of the LDS more; two wavefronts share a SIMD, and a projection of 4096 inputs has 8 k-groups a wavefront
// between its input and its last multiply.)
// us a step before / after: 4B class at batch 4 794 / 746, 8B layers at batch 8 1037 / 1005, serving burst 8512 / 8170, odd
// sizes at batch 5 494 / 463, mixture of experts at batch 1 860 / 837; the operands, and so the results, are the same bits.
constexpr uint32_t mfma_split_at(int pack, uint32_t col) { return pack == 2 ? 8u * (col >> 3) : pack == 3 ? 4u * (col >> 2) : 0u; }
template <int PACK>
struct MfmaOperands {
  u32x4 first[2], second[2], third[2];   // (second: PACK 1 and 2; third: PACK 1)
  __device__ __forceinline__ void load(const float* src, const uint16_t* gain, bool norm) {
    constexpr int N = PACK == 1 ? 2 : 1;   // runs of 8 (PACK 3: 4) inputs of this lane's own
#pragma unroll
    for (int U = 0; U < N; ++U) {
      float4 x0 = *(const float4*)(src + 8 * U), x1 = x0;
      if (PACK != 3) x1 = *(const float4*)(src + 8 * U + 4);
      if (norm) {
        u32x4 gg;
        if (PACK != 3) {
          gg = *(const u32x4*)(gain + 8 * U);
        } else {
          const u32x2 g2 = *(const u32x2*)gain;
          gg = u32x4{g2.x, g2.y, 0u, 0u};
        }
        x0.x *= bf16_lo(gg.x); x0.y *= bf16_hi(gg.x); x0.z *= bf16_lo(gg.y); x0.w *= bf16_hi(gg.y);
        if (PACK != 3) { x1.x *= bf16_lo(gg.z); x1.y *= bf16_hi(gg.z); x1.z *= bf16_lo(gg.w); x1.w *= bf16_hi(gg.w); }
      }
      if (PACK != 3) {
        u32x4 h, m, l;
        split8(x0, x1, &h, &m, &l);
        if (PACK == 1) {
          first[U] = h; second[U] = m; third[U] = l;
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            first[0][k] = row_lanes<8, 0xC>(h[k], m[k]);    // hi of its own half | mid of the other lane's
            first[1][k] = row_lanes<8, 0x3>(m[k], h[k]);
            second[0][k] = l[k];                            // (the second multiply's columns 8..15 are not results)
            second[1][k] = row_lanes<8, 0xF>(l[k], l[k]);
          }
        }
      } else {
        uint32_t h[2], m[2], l[2];
        split_hi_mid_lo(x0.x, x0.y, &h[0], &m[0], &l[0]);
        split_hi_mid_lo(x0.z, x0.w, &h[1], &m[1], &l[1]);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          // words k and 2 + k of a multiply come from column groups 2 U and 2 U + 1; columns 12..15 repeat lo
          first[0][k] = row_lanes<4, 0x2>(row_lanes<0, 0x1>(row_lanes<8, 0xF>(l[k], l[k]), h[k]), m[k]);
          first[0][2 + k] = row_lanes<0, 0x2>(row_lanes<12, 0x1>(row_lanes<4, 0xF>(l[k], l[k]), h[k]), m[k]);
          first[1][k] = row_lanes<12, 0x2>(row_lanes<8, 0x1>(l[k], h[k]), m[k]);
          first[1][2 + k] = row_lanes<8, 0x2>(row_lanes<4, 0x1>(row_lanes<12, 0xF>(l[k], l[k]), h[k]), m[k]);
        }
      }
    }
  }
};

// A pair of loads of 8 rows x 128 bytes (lane l: row l % 8 of rows 0..7 / 8..15, 16-byte block l / 8)
// -> the two matrix operands of the pair (lane = row + 16 x input group), in place; the derivation
// is in mfma_job_packed.
__device__ __forceinline__ void pair_to_operands(u32x4& l0, u32x4& l1) {
  auto ror8 = [](uint32_t old, uint32_t src, auto bank) {   // lanes of `bank`: src of the lane 8 further in its row of 16
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)src, 0x128, 0xF, decltype(bank)::value, false);
  };
  const u32x4 a = l0, b = l1;
  l0 = u32x4{ror8(a.x, b.x, std::integral_constant<int, 0xC>{}), ror8(a.y, b.y, std::integral_constant<int, 0xC>{}),
             ror8(a.z, b.z, std::integral_constant<int, 0xC>{}), ror8(a.w, b.w, std::integral_constant<int, 0xC>{})};
  l1 = u32x4{ror8(b.x, a.x, std::integral_constant<int, 0x3>{}), ror8(b.y, a.y, std::integral_constant<int, 0x3>{}),
             ror8(b.z, a.z, std::integral_constant<int, 0x3>{}), ror8(b.w, a.w, std::integral_constant<int, 0x3>{})};
}

// One job: out[r][b] partial tiles = W rows x staged input rows, left in LDS.
//   wbase, row_off(rt) : weight rows start at wbase (uniform) + row_off(rt) bytes, row_off = this
//                  lane's row of 16-row tile rt (32 bits: a scalar base and one vector offset per
//                  load, no address pairs to keep); loads are clamped to the end of the row
//   row_bytes(b) : byte of t.in at which fp32 input row b starts (uniform; read with coherent loads), b < nb
//   probe_fn()   : called before any request: the first look at the event, handed to wait_fn
//   wait_fn(p)   : called after the first two rounds of weights have been requested (cross-task
//                  pre-loading, Section 5.3: 16 KB per wavefront, 32 MB over the chip); returns
//                  kLinDone to go on
// LDS: x [nb][xstride] f32 at `lds`, reused at the end for the per-wavefront partial tiles
// part[8][4][16][16] f32, then the chunk's RMSNorm gains [Kc] bf16; ssq [8][16] f32 (sums of squares per wavefront and row, when pro_norm).
// On return (kLinDone) every thread may read part and ssq.
// PACK: how many of the three terms one multiply covers.  The multiply has 16 batch columns; up
// to 8 staged rows leave half of them free, so columns 0..7 take the hi term and columns 8..15
// the mid term of the same rows (PACK 2: two multiplies per fragment, the lo term alone in the
// second, on accumulators of its own); up to 4 staged rows take hi | mid | lo in columns 0..3 |
// 4..7 | 8..11 (PACK 3: one multiply).  The column groups are added up once, at the end.
template <int PACK, class RowOff, class RowBytes, class Probe, class Wait>
__device__ __forceinline__ uint32_t mfma_job_packed(const StepArgs& a, const TaskDesc& t, float* lds, float* ssq, const MfmaGeom& G,
                                                    const uint16_t* wbase, RowOff row_off, RowBytes row_bytes, bool pro_norm,
                                                    const uint16_t* gain, Probe probe_fn, Wait wait_fn) {
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t K = G.K, nb = G.nb, nrt = G.nrt;
  constexpr uint32_t Kc = mfma_kchunk(PACK == 1 ? 16u : PACK == 2 ? 8u : 4u), xstride = Kc + mfma_row_pad(PACK);   // inputs per chunk, floats between staged rows
  static_assert(mfma_kchunk(1) == mfma_kchunk(4) && mfma_kchunk(5) == mfma_kchunk(8) && mfma_kchunk(9) == mfma_kchunk(16), "the chunk follows from the packing");
  // (Every quotient below is by a power of two, and a shift: the compiler does not know it of a variable, and a
  // division is some thirty instructions, several of them in every round.)
  const uint32_t nchunk = (K + Kc - 1u) / Kc, kgsh = G.kgsh, kgpr = 1u << kgsh, ssh = 3u - G.rgsh;   // K slices: 1 << ssh
  const uint32_t nrtw = G.nrtw;
  float* xs = lds;
  float* part = lds;
  const uint32_t frow = lane & 15u, fk = (uint32_t)(lane >> 4) * 8u;
  constexpr uint32_t FR = kMfmaFrags, KG = 32u * FR;   // fragments per slot group, inputs per k-group
  // slot group q of a round: k-group offset inside the round, byte offset of its row tile's row
  const uint32_t sh = 2u - kgsh;   // q >> sh = k-group offset
  // How the weights are loaded.  A multiply wants lane (i = l % 16, j = l / 16) to hold 8 inputs of
  // tile row i, the same 8 for all i.  Loaded that way an instruction touches 16 rows x 64 bytes --
  // half lines, which streams 12 % slower than whole lines (5.9 against 6.7 TB/s in isolation).
  // So the two fragments of a k-group (64 inputs = 128 bytes of a row) are loaded as two
  // instructions of 8 rows x 128 bytes: load h (h = 0, 1), lane l: row 8 h + l % 8, inputs
  // 8 (l / 8) .. + 7 of the k-group.  Lane (i, j) then holds, of load 0: row i % 8, input block 2 j
  // (i < 8) or 2 j + 1 (i >= 8); of load 1: row 8 + i % 8, the same blocks.  One DPP move per
  // register (rotate the row of 16 lanes by 8, written to half of its lanes) turns the pair into
  //   first operand : row i, block 2 j      = load 0 (i < 8) | load 1 rotated (i >= 8)
  //   second operand: row i, block 2 j + 1  = load 0 rotated (i < 8) | load 1 (i >= 8)
  // and the activations follow: the multiplies of a k-group take input blocks (0, 2, 4, 6) and
  // (1, 3, 5, 7) instead of (0 .. 3) and (4 .. 7) -- any split of the 64 inputs will do as long as
  // both operands use the same one.
  static_assert(kMfmaFrags == 2, "the load pattern pairs the two fragments of a k-group");
  const uint32_t lrow = lane & 7u, lk = (uint32_t)(lane >> 3) * 8u;   // a load's row (+ 8 h) and first input
  uint32_t wq[4][2];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t j = kgpr == 4u ? 0u : (kgpr == 2u ? (uint32_t)q & 1u : (uint32_t)q);
    const uint32_t rt = min(G.my_g + G.rg * j, nrt - 1u);
    wq[q][0] = row_off(rt, lrow);
    wq[q][1] = row_off(rt, 8u + lrow);
  }
  // load h of the k-group at input k of the rows at byte offsets ro: this lane's 8 inputs start at
  // k + lk, or are the row's last 8 when that lies past its end (their staged inputs are zeros).  Not
  // real: a range of no bytes (a matrix is a multiple of 16 bytes below 4 GB, so a real load's end does not wrap)
  constexpr uint32_t kRange = 0xFFFFFFF0u;
  const uint16_t* wb = uniform_ptr(wbase);
  auto ld_frag = [&](uint32_t ro, uint32_t k, bool real) {
    return ld_stream16_ranged(wb, real ? kRange : 0u, ro + 2u * min(k + lk, K - 8u));
  };
  // the wavefront's run of k-groups in chunk c; a chunk takes an even number of round slots
  // (>= 2), so that even slots always use fragment buffer A and odd ones B
  auto chunk_kgs = [&](uint32_t c) { return (min(Kc, K - c * Kc) + KG - 1u) / KG; };
  auto run_lo = [&](uint32_t c) { return (G.my_s * chunk_kgs(c)) >> ssh; };
  auto run_hi = [&](uint32_t c) { return nrtw ? ((G.my_s + 1u) * chunk_kgs(c)) >> ssh : 0u; };
  auto slots = [&](uint32_t c) {
    const uint32_t lo = run_lo(c), hi = run_hi(c);
    const uint32_t n = hi > lo ? (hi - lo + kgpr - 1u) >> kgsh : 0u;
    return max(2u, (n + 1u) & ~1u);
  };
  // requests the 4 FR kilobytes of round slot (c, i) into buf; buf[FR Q + u] = load u of slot
  // group Q's k-group (rows 8 u .. 8 u + 7 of the tile, see above; two fragments after the
  // exchange in step).  Always that many loads, no branch (see ld_stream16_ranged).  A slot group that
  // does not exist (past the end of the run, or no row tile) is a load past the range.  (All lanes of all
  // wavefronts of an XCD used to read the matrix' first 16 bytes instead: up to 4096 requests for one
  // line at the end of every task, ahead of its output stores.)
  auto request_round = [&](u32x4* buf, uint32_t c, uint32_t i, bool wanted = true) {
    const uint32_t cc = min(c, nchunk - 1u);
    const uint32_t kg0 = run_lo(cc) + i * kgpr, hi = c < nchunk ? run_hi(cc) : 0u;
    const uint32_t k0 = cc * Kc;
    static_for<0, 4>([&](auto Qc) {
      constexpr uint32_t Q = (uint32_t)decltype(Qc)::value;
      const uint32_t kg = kg0 + (Q >> sh);
      const bool ok = wanted && kg < hi && (kgpr == 1u ? Q < nrtw : true);
#pragma unroll
      for (int u = 0; u < (int)FR; ++u) buf[FR * Q + u] = ld_frag(wq[Q][u], k0 + kg * KG, ok);
    });
  };
  // RMSNorm gains of a chunk, bf16, copied to LDS behind the staged rows (weights: chunk 0's are
  // requested before the event).  All copies into LDS here go from device memory straight to LDS
  // (no registers): 16 bytes per lane, a wavefront's 64 lanes land side by side.
  uint16_t* gl = (uint16_t*)(xs + (size_t)nb * xstride);   // [Kc]
  auto request_gains = [&](uint32_t c) {
    const uint32_t k0 = c * Kc, klen = min(Kc, K - k0), col = 8u * threadIdx.x;
    // (a buffer load: the compiler takes a global load into LDS for a flat access, whose order it does not
    // know, and until it has landed waits for everything in flight instead of for the event's probe alone)
    if (pro_norm && col < klen)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(uniform_ptr(gain)), 0, (int)(2u * K), 0x00020000),
                                               (lds_ptr_t)(gl + wave * 512u), 16, (int)(2u * (k0 + col)), 0, 0, 0);
    // between the end of the row and the end of its last k-group the staged inputs are zeros, and
    // so must the gains be: whatever an earlier workgroup left there may read as NaN, and
    // 0 x NaN is NaN
    if (pro_norm)
      for (uint32_t i = klen + threadIdx.x; i < ((klen + 127u) & ~127u); i += kThreads) gl[i] = 0;
  };
  // Staging: the nb rows of a chunk, 256 inputs (1 KB) per instruction, a row's instructions dealt to the wavefronts,
  // with agent-coherent loads straight into LDS.  What lies between the end of a row and the end of its last
  // k-group is zeroed.  A rolled loop on purpose: unrolled, the addresses, LDS addresses and lane masks of all
  // sixteen copies are worked out ahead of the chunk loop, at the start of every task, and kept in spilled registers.
  // With one packing a kernel and no divisions 295 -> 243 spilled scalar registers; us a step: 8B layers at batch 8
  // 1072 -> 1044, serving burst 9357 -> 8800, odd sizes at batch 5 546 -> 508, mixture of experts at batch 1 961 -> 895.
  float rowsum = 0.f;   // lane b: this wavefront's sum of squares of staged row b
  auto stage = [&](uint32_t c) {
    const uint32_t k0 = c * Kc, klen = min(Kc, K - k0), kpad = (klen + 127u) & ~127u;
    if (c) request_gains(c);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(uniform_ptr(t.in)), 0, (int)kRange, 0x00020000);
#pragma unroll 1
    for (uint32_t b = 0; b < nb; ++b) {
      const uint32_t row = row_bytes(b) + 4u * k0;
#pragma unroll
      for (uint32_t h = 0; h < Kc / 2048u; ++h) {
        const uint32_t seg = wave + 8u * h;
        if (seg * 256u + 4u * (uint32_t)lane < klen)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(xs + (size_t)b * xstride + seg * 256u), 16, 16 * lane, (int)(row + 1024u * seg), 0, 16);
      }
    }
    if (kpad != klen)
      for (uint32_t i = threadIdx.x; i < nb * (kpad - klen); i += kThreads) xs[(size_t)(i / (kpad - klen)) * xstride + klen + i % (kpad - klen)] = 0.f;
  };
  u32x4 wA[4 * FR], wB[4 * FR];
  const bool preload = !(a.flags & kNoPreloadBit);   // off: the ablation of Section 6.5, Fig. 10
  // Both rounds (16 KB per wavefront) are requested before the event.  A wavefront sees its loads
  // complete in the order it issued them, so whatever is requested now stands between the event
  // and the staged input: more than this measured slower.
  const auto probe = probe_fn();
  request_gains(0u);
  request_round(wA, 0u, 0u, preload);   // (not wanted: loads past the range, see ld_stream16_ranged)
  asm volatile("; first round requested" ::: "memory");
  request_round(wB, 0u, 1u, preload);
  asm volatile("; second round requested" ::: "memory");
  {
    const uint32_t w = wait_fn(probe);
    if (w != kLinDone) return w;   // aborted or pre-empted: the requested weights are dropped
  }
  trace_mark(a, t, 1);
  if (!preload) {
    request_round(wA, 0u, 0u);
    asm volatile("; first round requested after the event" ::: "memory");
  }
  // sums of squares of the staged rows (before the gains), needed only by the epilogue: taken
  // behind the chunk's multiplies by wavefronts 0..3 (rows w, w + 4, ...), which are through their
  // share well before the upper four are (they win the arbitration on their SIMDs), so the pass is
  // off the path from the event to the first multiply and costs nothing at the end either
  auto row_squares = [&](uint32_t c) {
    const uint32_t klen = min(Kc, K - c * Kc);
    for (uint32_t r = wave; r < nb && wave < 4u; r += 4u) {
      float sq = 0.f;
      for (uint32_t col = 4u * (uint32_t)lane; col < klen; col += 256u) {
        const float4 v = *(const float4*)(xs + (size_t)r * xstride + col);
        sq = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, sq))));
      }
      sq = wave_sum_dpp(sq);
      if ((uint32_t)lane == r) rowsum += sq;
    }
  };
  // this lane's staged row, and its inputs of a k-group (operand U: input block 2 j + U)
  const uint32_t xrow = min(PACK == 1 ? frow : (PACK == 2 ? (frow & 7u) : (frow & 3u)), nb - 1u);
  const uint32_t xat = 2u * fk + mfma_split_at(PACK, frow);
  const float* xl = xs + (size_t)xrow * xstride + xat;
  const uint16_t* gx = gl + xat;
  f32x4 acc[4], acc_lo[4];   // (acc_lo: the lo term's products when PACK == 2)
  // one round slot: multiplies what buf holds for slot (c, i) -- fragment u of every slot group
  // against the three terms of that fragment's inputs, converted once per k-group -- and then
  // requests slot (c2, i2), two ahead, into the same registers
  auto step = [&](u32x4* buf, uint32_t c, uint32_t i, uint32_t c2, uint32_t i2) {
    const uint32_t kg0 = run_lo(c) + i * kgpr, hi = run_hi(c);
    if (kg0 < hi) {
#pragma unroll
      for (int q = 0; q < 4; ++q) pair_to_operands(buf[FR * q], buf[FR * q + 1]);
      MfmaOperands<PACK> op;
      static_for<0, 4>([&](auto Qc) {
        constexpr uint32_t Q = (uint32_t)decltype(Qc)::value;
        const uint32_t kg = kg0 + (Q >> sh);
        const bool rowok = kgpr == 1u ? Q < nrtw : true;
        if (kg < hi && rowok) {
          if (Q == 0u || (Q >> sh) != ((Q - 1u) >> sh)) op.load(xl + kg * KG, gx + kg * KG, pro_norm);   // first slot group of its k-group
#pragma unroll
          for (uint32_t U = 0; U < FR; ++U) {
            const bf16x8 av = __builtin_bit_cast(bf16x8, buf[FR * Q + U]);
            acc[Q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, op.first[U]), acc[Q], 0, 0, 0);
            if (PACK == 2) acc_lo[Q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, op.second[U]), acc_lo[Q], 0, 0, 0);
            if (PACK == 1) {
              acc[Q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, op.second[U]), acc[Q], 0, 0, 0);
              acc[Q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, op.third[U]), acc[Q], 0, 0, 0);
            }
          }
        }
      });
    }
    request_round(buf, c2, i2);
  };
  for (uint32_t c = 0; c < nchunk; ++c) {
    if (c) lds_barrier();   // everybody has finished with the previous chunk
    stage(c);
    drain_vmem();   // this wavefront's copies have landed
    lds_barrier();
    if (c == 0 && !preload) request_round(wB, 0u, 1u);
    if (c == 0) {
      trace_mark(a, t, 2);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = acc_lo[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const uint32_t ns = slots(c);
    for (uint32_t i = 0; i < ns; i += 2u) {
      const bool wrap = i + 2u >= ns;   // the slots two ahead are the first two of the next chunk
      const uint32_t c2 = wrap ? c + 1u : c, i2 = wrap ? 0u : i + 2u;
      step(wA, c, i, c2, i2);
      step(wB, c, i + 1u, c2, i2 + 1u);
    }
    if (pro_norm) row_squares(c);   // (the chunk is still staged: the next barrier is ahead)
  }
  trace_mark(a, t, 8);
  drain_vmem();   // (nothing but loads past the range)
  // ---- the column groups of a packed multiply added up: afterwards column b < nb holds the sum
  if (PACK == 3) {
    // An infinite weight or input gives what vector arithmetic gives, and that is in the hi columns alone: the lower
    // terms of a product with an infinity are NaN or of the other sign.
    float all[4] = {0.f, 0.f, 0.f, 0.f};   // not finite if one of the sums is not
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) all[i] += acc[j][i];
    if (__builtin_expect(__any(!(fabsf((all[0] + all[1]) + (all[2] + all[3])) < INFINITY)), 0)) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (frow >= 4u && !(fabsf(acc[j][i]) < INFINITY)) acc[j][i] = 0.f;
    }
  }
  if (PACK != 1) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // (a lane's column is its index in its row of 16 lanes: the value 8 / 4 columns up comes
        // by a DPP row shift; columns that get nothing are not results)
        const float v = acc[j][i];
        auto up = [](float x, auto ctrl) {
          return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, true));
        };
        if (PACK == 2) acc[j][i] = v + up(v, std::integral_constant<int, 0x108>{}) + acc_lo[j][i];        // hi + mid (8 columns up) + lo
        else acc[j][i] = v + up(v, std::integral_constant<int, 0x104>{}) + up(v, std::integral_constant<int, 0x108>{});   // hi + mid + lo, 4 columns apart
      }
  }
  lds_barrier();   // nobody reads the staged input any more: its space takes the partial tiles
  // ---- partial tiles -> LDS.  part[wave][slot group][row 0..15][col 0..15]
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) part[((wave * 4 + j) * 16 + (lane >> 4) * 4 + i) * 16 + (lane & 15)] = acc[j][i];
  if (pro_norm && lane < 16) ssq[wave * 16 + lane] = rowsum;
  lds_barrier();
  return kLinDone;
}

// NB: the largest number of staged rows there can be (an expert has at most as many tokens as the batch).
template <int NB, class RowOff, class RowBytes, class Probe, class Wait>
__device__ __forceinline__ uint32_t mfma_job(const StepArgs& a, const TaskDesc& t, float* lds, float* ssq, const MfmaGeom& G,
                                             const uint16_t* wbase, RowOff row_off, RowBytes row_bytes, bool pro_norm,
                                             const uint16_t* gain, Probe probe_fn, Wait wait_fn) {
  if (NB <= 4 || G.nb <= 4u) return mfma_job_packed<3>(a, t, lds, ssq, G, wbase, row_off, row_bytes, pro_norm, gain, probe_fn, wait_fn);
  if constexpr (NB > 4) {
    if (NB <= 8 || G.nb <= 8u) return mfma_job_packed<2>(a, t, lds, ssq, G, wbase, row_off, row_bytes, pro_norm, gain, probe_fn, wait_fn);
  }
  if constexpr (NB > 8) return mfma_job_packed<1>(a, t, lds, ssq, G, wbase, row_off, row_bytes, pro_norm, gain, probe_fn, wait_fn);
  return kLinAbort;
}

// Dot product of weight row r (16-row tile r / 16) with batch column bb from the partial tiles a
// job left in LDS: the row tile's slot groups of slice 0, then those of slice 1, ... added in
// that order.  Up to 32 partials, read eight at a time (one after the other they were a chain of LDS
// round trips: 1.3 us of the 3 us between the last multiply and the notification).
__device__ __forceinline__ float mfma_dot(const float* part, const MfmaGeom& G, uint32_t r, uint32_t bb) {
  const uint32_t rt = r >> 4, row = r & 15u;
  const uint32_t g = rt & (G.rg - 1u), j = rt >> G.rgsh;
  const uint32_t n = mfma_group_tiles(G.nrt, G.rgsh, g);   // row tiles of the wavefronts of group g
  const uint32_t psh = n >= 3u ? 0u : (n == 2u ? 1u : 2u);   // 1 << psh slot groups per slice, 4 >> psh apart
  const uint32_t np = G.ks << psh;
  const float* p0 = part + ((g * 4u + (n >= 2u ? j : 0u)) * 16u + row) * 16u + bb;
  float v = 0.f;
  for (uint32_t k0 = 0; k0 < np; k0 += 8u) {
    float p[8];
#pragma unroll
    for (uint32_t k = 0; k < 8u; ++k) {
      const uint32_t kk = k0 + k, s = kk >> psh, q = (kk & ((1u << psh) - 1u)) * (4u >> psh);
      p[k] = kk < np ? p0[((s << G.rgsh) * 4u + q) * 256u] : 0.f;
    }
#pragma unroll
    for (uint32_t k = 0; k < 8u; ++k) v += p[k];   // (absent ones add zero)
  }
  return v;
}
// 1 / rms of staged row bb from the wavefronts' sums of squares (every thread for itself: eight reads in flight, no barrier)
__device__ __forceinline__ float mfma_inv_rms(const float* ssq, uint32_t bb, uint32_t K, float eps) {
  float ss = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) ss += ssq[w * 16 + bb];
  return 1.0f / sqrtf(ss / (float)K + eps);
}

// LDS of a linear task (from the task area): job buffers (mfma_x_floats) | ssq [8][16] f32 | arrival flag.  A job takes up to 512 weight rows; a task of more (batch 3 and 4:
// an output head of more than 512 rows a worker, few tiles given) is worked off in several, the input staged
// again for each.
// PACK: the packing of the input terms, that of the graph's batch class: 3 up to 4 rows, 2 up to 8, 1 up to 16 (run_linear).
template <int PACK, bool MEGA, class Svc = NoJit>
__device__ __forceinline__ uint32_t linear_task_mfma(const TaskDesc& t, const StepArgs& a, float* lds, int32_t wait_ev,
                                                     uint32_t* s_flag, const Svc& svc = Svc{}) {
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t K = t.K, nb = t.b1 - t.b0, ncols = t.c1 - t.c0;
  const uint32_t gateup = (t.flags & TF_GATEUP) ? 1u : 0u;
  const uint32_t R = ncols << gateup;            // weight rows of the task ("ring rows")
  float* part = lds;
  float* ssq = lds + mfma_x_floats(nb);          // [8][16]
  // split-K task (TF_SPLITK): rows [row0, row0 + ncols) of the matrix, inputs of ONE part; the
  // weight pointer is already advanced to the part, rows are ldw apart
  const bool splitk = t.flags & TF_SPLITK;
  const uint32_t parts = splitk ? (t.p3 & 0xFFu) : 1u, my_part = splitk ? (t.p3 >> 8) : 0u;
  const uint32_t Hs = t.ld_out / parts;              // columns of the real output
  const uint32_t row0 = t.c0 - my_part * Hs, ldw = splitk ? t.p1 : K;
  const uint16_t* W = (const uint16_t*)t.w + (size_t)row0 * ldw;   // the task's first row (gate/up: of the gate rows)
  auto row_bytes = [&](uint32_t b) { return 4u * (t.b0 + b) * t.ld_in; };   // (at most 16 rows)
  const bool pro_norm = t.flags & TF_PRO_NORM;
  for (uint32_t r0 = 0; r0 < R; r0 += kMfmaJobRows) {
    const uint32_t Rj = min(R - r0, kMfmaJobRows), cj = r0 >> gateup, nj = Rj >> gateup;   // the job's rows, columns
    const MfmaGeom G = mfma_geom(K, nb, (Rj + 15u) / 16u, wave);
    auto row_off = [&](uint32_t rt, uint32_t row) {       // row: this lane's row of the 16-row tile
      const uint32_t r = min(rt * 16u + row, Rj - 1u);    // rows past the end repeat the last one
      const uint32_t wrow = gateup ? ((r >> 1) + ((r & 1u) ? t.p0 : 0u)) : r;
      // bytes from the job's first row: below 4 GB also where one task holds all of a larger matrix (batch 3
      // and 4 take any vocabulary; the gate/up halves of inputs that fit the LDS lie well within 4 GB)
      return wrow * ldw * 2u;
    };
    auto probe_fn = [&]() { return linear_probe<Svc>(a, r0 == 0 ? wait_ev : -1, wave, lane); };
    // the residual slice of this tile goes out ahead of the input (tile-local, small), a thread loads that of its first output:
    // its round trip overlaps the staging
    const uint32_t bsh = nb <= 4u ? 2u : (nb <= 8u ? 3u : 4u);   // batch columns padded to 4, 8 or 16 lanes: no division
    const bool resid = (t.flags & TF_EPI_RESID) && !splitk;
    float resv = 0.f;
    auto load_resid = [&]() {
      const uint32_t cc = threadIdx.x >> bsh, bb = threadIdx.x & ((1u << bsh) - 1u);
      if (resid && bb < nb && cc < nj) resv = ld_act(t.in2 + (size_t)(t.b0 + bb) * t.ld_out + t.c0 + cj + cc);
    };
    auto wait_fn = [&](const EventProbe& probe) -> uint32_t {
      if (wait_ev >= 0 && r0 == 0) {
        const uint32_t w = linear_wait(a, wait_ev, s_flag, wave, lane, svc, probe);
        if (w != kLinDone) return w;
      }
      load_resid();
      return kLinDone;
    };
    {
      const uint32_t w = mfma_job_packed<PACK>(a, t, lds, ssq, G, W + (size_t)cj * ldw, row_off, row_bytes, pro_norm, (const uint16_t*)t.w2, probe_fn, wait_fn);
      if (w != kLinDone) return w;
    }
    trace_mark(a, t, 3);
    // ---- all wavefronts: add the K slices in order, epilogue, outputs; then the notification
    {
      float* outp = (t.flags & TF_OUT_LOGITS) ? a.logits : t.out;
      for (uint32_t i = threadIdx.x; i < nj << bsh; i += kThreads) {
        const uint32_t cc = i >> bsh, bb = i & ((1u << bsh) - 1u);
        if (bb >= nb) continue;
        const float inv = pro_norm ? mfma_inv_rms(ssq, bb, K, t.f0) : 1.0f;
        float v;
        if (gateup) {
          const float gte = mfma_dot(part, G, 2 * cc, bb) * inv, up = mfma_dot(part, G, 2 * cc + 1, bb) * inv;
          v = gte / (1.0f + expf(-gte)) * up;
        } else {
          v = mfma_dot(part, G, cc, bb) * inv;
        }
        if (resid) v = (i < kThreads ? resv : ld_act(t.in2 + (size_t)(t.b0 + bb) * t.ld_out + t.c0 + cj + cc)) + v;
        st_act(outp + (size_t)(t.b0 + bb) * t.ld_out + t.c0 + cj + cc, v);   // split-K: the partial sums of this part
      }
    }
    if (r0 + kMfmaJobRows < R) lds_barrier();   // the next job reuses the buffers
  }
  if (MEGA || splitk) {
    // every wavefront's coherent stores complete before anyone is told
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    drain_vmem();
    lds_barrier();
  }
  if (splitk) {
    // arrival at the row block's counter now that the partial sums are visible; the last of the
    // `parts` tasks adds the parts in order, and the residual, into the real output -- all
    // wavefronts, one output each, the loads of an output in flight together
    uint32_t* last_flag = (uint32_t*)(ssq + 9 * 16);
    if (threadIdx.x == 0) {
      const uint32_t old = __hip_atomic_fetch_add(as_global(a.g->grp_counters + t.p2), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *last_flag = ((old + 1u) % parts == 0u) ? 1u : 0u;   // every step adds exactly `parts` (also when a captured launch is replayed with its step number frozen)
    }
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(*last_flag)) {
      float* xout = (float*)t.aux0;
      for (uint32_t i = threadIdx.x; i < ncols * nb; i += kThreads) {
        const uint32_t cc = i / nb, bb = i % nb;
        float v = ld_act(t.in2 + (size_t)(t.b0 + bb) * Hs + row0 + cc);
        float pv[8];
#pragma unroll
        for (uint32_t pp = 0; pp < 8; ++pp) pv[pp] = pp < parts ? ld_act(t.out + (size_t)(t.b0 + bb) * t.ld_out + pp * Hs + row0 + cc) : 0.f;
#pragma unroll
        for (uint32_t pp = 0; pp < 8; ++pp) v += pv[pp];   // parts in ascending order (absent ones add zero)
        st_act(xout + (size_t)(t.b0 + bb) * Hs + row0 + cc, v);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      drain_vmem();
    }
    lds_barrier();
  }
  if (wave == 0) {
    if (MEGA && t.trig_event >= 0) signal_from_wave0(a, t, lane);
    trace_mark(a, t, 4);
  }
  lds_barrier();   // the partial buffer is reused by the next task
  return kLinDone;
}

// ------------------------------------------------------------------------------ mixture of experts
// Section 6.4: an MoE block is a chain of tasks in the same graph.  `route` turns the router's
// output into the meta-tensor (layout next to moe_meta_words); expert tasks are fixed at compile
// time and use the meta-tensor to split the active experts' weight rows evenly among themselves
// at run time; token rows are gathered while the input is staged (no separate gather step).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, off, 64));
  return v;
}

// What bounds this task and the combine below is latency, a chain of round trips and selection rounds in
// one workgroup.  Batch 1, 128 experts, top 8, 12 layers: 1065 -> 1018 us a step with the selection kept
// to the experts there are and the combine's loads of eight experts in flight together.
// One task.  Softmax over all experts in fp32, the top_k largest probabilities (ties: lower expert
// index), renormalised to sum one; ranks of a token's experts are in ascending expert index.
// PER_LANE: experts a lane looks after, at least E / 64 (a loop over the eight that the largest E needs costs
// its branches in every selection round).
// A token's choice is a bit mask over the experts, built in scalar registers by the wavefront that makes it; behind the one
// barrier a thread per expert counts bits in the tokens' masks, which gives everything the meta-tensor holds (its tokens, where
// its list starts, its place among the active, the pairs) without a scan.  us a step at batch 1, 12 layers: lists by LDS atomics and
// scans behind four barriers 793, masks 783 (batch 16, 6 layers: no difference).
// LOCAL: `meta` is an expert task's copy in LDS, of which it reads the words up to the end of the pair list and not [1].
template <int PER_LANE, bool LOCAL>
__device__ __forceinline__ void moe_route(const float* in, uint32_t ld_in, uint32_t E, uint32_t TK, uint32_t B, float* lds, uint32_t* meta) {
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t P = B * TK, B4 = (B + 3u) & ~3u;
  uint64_t* masks = (uint64_t*)lds;                       // [B4][PER_LANE] bit l of word i: expert l + 64 i (batch <= 16)
  uint32_t* lower_words = (uint32_t*)(masks + B4 * PER_LANE);   // [B4][PER_LANE] experts in the mask's lower words (PER_LANE > 2)
  uint32_t* sel = lower_words + B4 * PER_LANE;            // [P] expert of pair p
  float* wsel = (float*)(sel + P);                        // [P] weight of pair p
  uint32_t* wave_most = (uint32_t*)(wsel + P);            // [8] largest token count among a wavefront's experts
  constexpr int kPerLane = PER_LANE;
  const uint32_t nper = (E + 63u) / 64u;   // experts per lane actually present (uniform)
  auto put = [&](uint32_t at, uint32_t v) {
    if constexpr (LOCAL) meta[at] = v;
    else st_act_u32(meta + at, v);
  };
  for (uint32_t tok = wave; tok < B4; tok += kThreads / 64) {
    if (tok >= B) {   // (nobody's: the counts below go by fours)
      if (lane < kPerLane) {
        masks[tok * kPerLane + lane] = 0;
        if constexpr (PER_LANE > 2) lower_words[tok * kPerLane + lane] = 0;
      }
      continue;
    }
    float pr[kPerLane];
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      const uint32_t e = (uint32_t)lane + 64u * i;
      pr[i] = -INFINITY;
      if ((uint32_t)i < nper && e < E) pr[i] = ld_act(in + (size_t)tok * ld_in + e);
    }
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) m = fmaxf(m, pr[i]);
    m = wave_max_dpp(m);
    float l = 0.f;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      const uint32_t e = (uint32_t)lane + 64u * i;
      const float lg = pr[i];
      pr[i] = 0.f;
      if ((uint32_t)i < nper && e < E) pr[i] = expf(lg - m);
      asm("" : "+v"(pr[i]));   // (the same bits in every instance: an expert task and the routing task have to choose alike)
      l += pr[i];
    }
    l = wave_sum_dpp(l);
    // left: what may still be chosen, as a number that grows with the probability; 0: an expert that is not there, or whose
    // probability is not a number, or that has been chosen.  (Of whole numbers the largest is found without a float maximum's
    // quieting of its operands.)
    uint32_t left[kPerLane];
    uint64_t taken[kPerLane];
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      if ((uint32_t)i < nper) pr[i] = pr[i] / l;
      left[i] = (uint32_t)i < nper && (uint32_t)lane + 64u * i < E && pr[i] >= 0.f ? __float_as_uint(pr[i]) + 1u : 0u;
      taken[i] = 0;
    }
    for (uint32_t j = 0; j < TK; ++j) {
      uint32_t best = left[0];
#pragma unroll
      for (int i = 1; i < kPerLane; ++i) best = max(best, left[i]);
      best = wave_reduce_dpp(best, [](uint32_t x, uint32_t y) { return max(x, y); });
      if (best == 0u) break;   // (a token whose router output is not finite selects nothing)
      // ties: the lowest expert
      if constexpr (PER_LANE == 2) {
        bool found = false;
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
          const uint64_t at = found ? 0ull : __ballot(left[i] == best);
          if (at) {
            const int first = __builtin_ctzll(at);
            taken[i] |= 1ull << first;
            left[i] = lane == first ? 0u : left[i];
            found = true;
          }
        }
      } else {   // (no branches: eight of them a round made it 19.0 us a routing task at 512 experts and batch 16, now 16.7)
        uint64_t at = 0;
        int word = 0;
#pragma unroll
        for (int i = kPerLane - 1; i >= 0; --i) {
          const uint64_t here = __ballot(left[i] == best);
          at = here ? here : at;
          word = here ? i : word;
        }
        const uint64_t one = at & (0ull - at);
#pragma unroll
        for (int i = 0; i < kPerLane; ++i) {
          const uint64_t mine = i == word ? one : 0ull;
          taken[i] |= mine;
          left[i] = __builtin_amdgcn_inverse_ballot_w64(mine) ? 0u : left[i];
        }
      }
    }
    if constexpr (!LOCAL) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < kPerLane; ++i) s += ((taken[i] >> lane) & 1ull) ? pr[i] : 0.f;
      s = wave_sum_dpp(s);
      uint32_t before = 0;   // selected experts with a smaller index, so far
#pragma unroll
      for (int i = 0; i < kPerLane; ++i) {
        if ((taken[i] >> lane) & 1ull) {
          const uint32_t rank = before + (uint32_t)__popcll(taken[i] & ((1ull << lane) - 1ull));
          sel[tok * TK + rank] = (uint32_t)lane + 64u * i;
          wsel[tok * TK + rank] = pr[i] / s;
        }
        before += (uint32_t)__popcll(taken[i]);
      }
      if ((uint32_t)lane >= before && (uint32_t)lane < TK) {
        sel[tok * TK + lane] = 0xFFFFFFFFu;
        wsel[tok * TK + lane] = 0.f;
      }
    }
    uint32_t lower = 0;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      if (lane == 0) {
        masks[tok * kPerLane + i] = taken[i];
        if constexpr (PER_LANE > 2) lower_words[tok * kPerLane + i] = lower;
      }
      lower += (uint32_t)__popcll(taken[i]);
    }
  }
  lds_barrier();
  static_assert(kMoeMaxExperts <= kThreads, "a thread per expert");
  const uint32_t e = threadIdx.x;
  const uint32_t w = wave;   // the word of the masks that has the expert's bit
  uint32_t cnt = 0, act = 0;   // the expert's tokens, active lower experts
  // Eight words a token are too many for every thread to read (128 reads at batch 16): a wavefront reads its own word of each,
  // what lies below it was counted when the mask was made, and the lower words' active experts are counted by all lanes
  // together: a lane ors a word of two tokens, then the lanes of a word or theirs.  us a step of 4 layers with 512 experts at
  // batch 16: lists by LDS atomics and scans 1130, all words read by every thread 1141, this (and the selection above) 1101.
  if constexpr (PER_LANE > 2) {
    static_assert(PER_LANE == 8, "a lane per word of eight tokens");
    uint32_t part[2] = {0, 0};
#pragma unroll
    for (uint32_t b = 0; b < 16u; b += 8u)
      if (8u * b + (uint32_t)lane < 8u * B4) {
        const uint64_t m = masks[8u * b + (uint32_t)lane];
        part[0] |= (uint32_t)m;
        part[1] |= (uint32_t)(m >> 32);
      }
    uint32_t active = 0;   // lane i < 8: experts of word i
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t v = part[h];
      v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);   // the lane 8 further in its row of 16
      const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
      v = r[0] | r[1];
      const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
      active += (uint32_t)__popc(q[0] | q[1]);
    }
#pragma unroll
    for (int i = 0; i < 7; ++i) act += (uint32_t)i < w ? (uint32_t)__builtin_amdgcn_readlane((int)active, i) : 0u;
  }
  if (e < E) {
    const uint64_t bit = 1ull << lane, below = bit - 1ull;
    uint32_t off = 0, of = 0;   // all pairs of lower experts, bit b: token b is its
    uint64_t ranks = 0;                  // four bits a token: its rank there (below TK <= 16)
    auto token = [&](uint32_t b, uint64_t own, uint32_t lower) {   // own: the token's word w; lower: its experts in lower words
      lower += (uint32_t)__popcll(own & below);
      off += lower;
      if (own & bit) {
        of |= 1u << b;
        ranks |= (uint64_t)lower << (4u * b);
      }
    };
    // (the masks of four tokens in flight: one after the other they are a chain of LDS round trips, 4 us at batch 16)
    if constexpr (PER_LANE == 2) {
      uint64_t any[2] = {};
      for (uint32_t b0 = 0; b0 < B4; b0 += 4u) {
#pragma unroll
        for (uint32_t u = 0; u < 4u; ++u) {
          const uint64_t m0 = masks[2u * (b0 + u)], m1 = masks[2u * (b0 + u) + 1u];
          any[0] |= m0;
          any[1] |= m1;
          token(b0 + u, w ? m1 : m0, w ? (uint32_t)__popcll(m0) : 0u);
        }
      }
      act = (uint32_t)__popcll((w ? any[1] : any[0]) & below) + (w ? (uint32_t)__popcll(any[0]) : 0u);
    } else {
      uint64_t any = 0;
      for (uint32_t b0 = 0; b0 < B4; b0 += 4u) {
#pragma unroll
        for (uint32_t u = 0; u < 4u; ++u) {
          const uint64_t own = masks[8u * (b0 + u) + w];
          any |= own;
          token(b0 + u, own, lower_words[8u * (b0 + u) + w]);
        }
      }
      act += (uint32_t)__popcll(any & below);
    }
    cnt = (uint32_t)__popc(of);
    if (e == E - 1u) put(0u, act + (cnt ? 1u : 0u));
    put(2u + E + e, cnt);
    put(2u + 2u * E + e, off);
    if (cnt) put(2u + act, e);
    for (uint32_t o = off; of; of &= of - 1u) {   // ascending token = ascending pair
      const uint32_t b = (uint32_t)__ffs((int)of) - 1u;
      put(2u + 3u * E + o++, b * TK + (uint32_t)(ranks >> (4u * b) & 15u));
    }
  }
  if constexpr (!LOCAL) {
    const uint32_t most = wave_reduce_dpp(cnt, [](uint32_t x, uint32_t y) { return max(x, y); });
    if (lane == 0) wave_most[wave] = most;
    for (uint32_t p2 = threadIdx.x; p2 < P; p2 += kThreads) {
      put(2u + 3u * E + P + p2, __float_as_uint(wsel[p2]));
      put(2u + 3u * E + 2u * P + p2, sel[p2]);
    }
    lds_barrier();
    if (threadIdx.x == 0) {
      uint32_t mx = wave_most[0];
#pragma unroll
      for (int i = 1; i < (int)(kThreads / 64); ++i) mx = max(mx, wave_most[i]);
      put(1u, mx);
    }
  }
}

__device__ __forceinline__ void body_moe_route(const TaskDesc& t, float* lds) {
  if (t.p0 <= 128u) moe_route<2, false>(t.in, t.ld_in, t.p0, t.p1, t.p2, lds, (uint32_t*)t.out);
  else moe_route<(int)(kMoeMaxExperts / 64), false>(t.in, t.ld_in, t.p0, t.p1, t.p2, lds, (uint32_t*)t.out);
}

// `ntile` 16-row tiles of one expert's weight matrix, starting at tile `tile0`, times the `ne`
// token rows routed to that expert: a matrix-core job (mfma_job) whose input rows are gathered
// through the expert's pair list while they are staged.  All wavefronts take part; ntile <= 32,
// ne <= 16.
// wait_ev >= 0: the job's inputs exist only once that event is activated (the first job of a
// second-stage expert task, see run_moe_task): it is waited for behind the job's first weight
// requests.  Returns false when the step is being aborted.
template <int NB>
__device__ __forceinline__ bool moe_expert_job(const TaskDesc& t, const StepArgs& a, float* lds, const uint16_t* W,
                                               uint32_t tile0, uint32_t ntile, uint32_t ne, const uint32_t* plist,
                                               uint32_t TK, int32_t wait_ev, uint32_t* s_flag) {
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t K = t.K;
  const uint32_t gateup = (t.flags & TF_GATEUP) ? 1u : 0u;
  const bool pro_norm = t.flags & TF_PRO_NORM;
  const MfmaGeom G = mfma_geom(K, ne, ntile, wave);
  float* part = lds;
  float* ssq = lds + moe_x_floats(a.g->batch);   // [8][16]
  uint32_t* rowidx = (uint32_t*)(ssq + 8 * 16);  // [16] pair of each staged row (= output row)
  uint32_t* rowin = rowidx + 16;                 // [16] input row: gate/up reads the token's row, down the pair's
  if (threadIdx.x < ne) {
    const uint32_t pair = plist[threadIdx.x];   // (the task's copy of the meta-tensor in LDS)
    rowidx[threadIdx.x] = pair;
    rowin[threadIdx.x] = gateup ? pair / TK : pair;
  }
  lds_barrier();
  auto row_off = [&](uint32_t rt, uint32_t row) {   // row: this lane's row of the 16-row tile
    const uint32_t r = (tile0 + rt) * 16u + row;    // row of the expert's gate/up-interleaved (or plain) order
    const uint32_t wrow = gateup ? ((r >> 1) + ((r & 1u) ? t.p0 : 0u)) : r;
    return wrow * K * 2u;   // bytes from the expert's first row
  };
  // (a lane holds a row's index: read from LDS as they are needed, each read would wait for the copies under way into LDS)
  const uint32_t in_row = rowin[min((uint32_t)lane, ne - 1u)];
  auto row_bytes = [&](uint32_t b) { return 4u * (uint32_t)__builtin_amdgcn_readlane((int)in_row, (int)b) * t.ld_in; };   // (at most 256 pairs)
  auto probe_fn = [&]() { return linear_probe<NoJit>(a, wait_ev, wave, lane); };
  auto wait_fn = [&](const EventProbe& probe) -> uint32_t {
    if (wait_ev < 0) return kLinDone;
    const uint32_t w = linear_wait(a, wait_ev, s_flag, wave, lane, NoJit{}, probe);
    trace_mark(a, t, 1);
    return w;
  };
  if (mfma_job<NB>(a, t, lds, ssq, G, W, row_off, row_bytes, pro_norm, (const uint16_t*)t.w2, probe_fn, wait_fn) != kLinDone) return false;
  const uint32_t ncols = (ntile * 16u) >> gateup, col0 = (tile0 * 16u) >> gateup;
  const uint32_t sh = ne <= 1u ? 0u : (ne <= 2u ? 1u : (ne <= 4u ? 2u : (ne <= 8u ? 3u : 4u)));
  for (uint32_t i = threadIdx.x; i < ncols << sh; i += kThreads) {
    const uint32_t cc = i >> sh, bb = i & ((1u << sh) - 1u);
    if (bb >= ne) continue;
    const float inv = pro_norm ? mfma_inv_rms(ssq, bb, K, t.f0) : 1.0f;
    float v;
    if (gateup) {
      const float gte = mfma_dot(part, G, 2 * cc, bb) * inv, up = mfma_dot(part, G, 2 * cc + 1, bb) * inv;
      v = gte / (1.0f + expf(-gte)) * up;
    } else {
      v = mfma_dot(part, G, cc, bb);
    }
    st_act(t.out + (size_t)rowidx[bb] * t.ld_out + col0 + cc, v);
  }
  lds_barrier();   // the next job reuses the buffers
  return true;
}

// Expert task `c0` of `p1`: the active experts' 16-row weight tiles, laid end to end in ascending
// expert order, are dealt to the expert tasks in shares of equal cost (the run-time refinement of
// Section 6.4); a task's share is worked off in jobs of at most 32 tiles that stay inside one expert.
// wait_ev >= 0: the caller has NOT waited for the task's event yet (only for the routing task's,
// so the meta-tensor is this step's); the first job does, behind its first weight requests.
// own_route: there may be no meta-tensor yet: the routing is worked out here, from the router's output (kMoeOwnRouteExperts).
template <int NB>
__device__ __forceinline__ bool body_moe_expert(const TaskDesc& t, const StepArgs& a, float* lds, int32_t wait_ev, uint32_t* s_flag, bool own_route) {
  const uint32_t* meta = (const uint32_t*)t.in2;
  const uint32_t E = t.p3 & 0xFFFFu, TK = t.p3 >> 16, NT = t.p1, rows_per_expert = t.p2;
  const uint32_t tiles_per_expert = rows_per_expert / 16u;
  // The part of the meta-tensor an expert task reads -- header, active list, per-expert counts and
  // offsets, pair lists -- comes to LDS in one round trip; looked up in device memory, every job
  // cost three dependent trips (expert, its count and offset, its pairs) before its first weight
  // request could go out.
  const uint32_t P = a.g->batch * TK, MW = 2u + 3u * E + P;
  uint32_t* mlds = (uint32_t*)(lds + moe_x_floats(a.g->batch) + 8 * 16 + 32);   // behind the staged row lists
  if (own_route) moe_route<2, true>((const float*)t.aux0, E, E, TK, a.g->batch, lds, mlds);
  else
    for (uint32_t i = threadIdx.x; i < MW; i += kThreads) mlds[i] = ld_relaxed(meta + i);
  lds_barrier();
  const uint32_t n_active = min(__builtin_amdgcn_readfirstlane(mlds[0]), E);
  uint32_t u0, u1;   // this task's share of the tiles: equal in cost, see moe_task_share
  moe_task_share(n_active, tiles_per_expert, NT, t.c0, &u0, &u1);
  while (u0 < u1) {
    const uint32_t ai = u0 / tiles_per_expert, tile0 = u0 % tiles_per_expert;
    const uint32_t ntile = min(min(u1 - u0, tiles_per_expert - tile0), 32u);
    const uint32_t e = min(__builtin_amdgcn_readfirstlane(mlds[2 + ai]), E);   // (E: rejected below; the two reads stay inside the copy)
    const uint32_t ne = __builtin_amdgcn_readfirstlane(mlds[2 + E + min(e, E - 1u)]);
    const uint32_t po = __builtin_amdgcn_readfirstlane(mlds[2 + 2 * E + min(e, E - 1u)]);
    if (e >= E || ne == 0 || ne > (uint32_t)NB || po + ne > P) {   // never index with a damaged meta-tensor
      if (threadIdx.x == 0) report(a, DE_BAD_META, e, ne);
      break;
    }
    const uint16_t* W = (const uint16_t*)t.w + (size_t)e * rows_per_expert * t.K;
    if (!moe_expert_job<NB>(t, a, lds, W, tile0, ntile, ne, mlds + 2 + 3 * E + po, TK, wait_ev, s_flag)) return false;
    wait_ev = -1;
    u0 += ntile;
  }
  // (no job ran: the task still ends after its event, like every task)
  if (wait_ev >= 0 && !wait_event(a, wait_ev, s_flag)) return false;
  return true;
}

// out[b][c] = resid[b][c] + sum over the token's experts, in ascending expert index, of
// weight x expert output.
__device__ __forceinline__ void body_moe_combine(const TaskDesc& t, const StepArgs& a) {
  const uint32_t E = t.p0, TK = t.p1, P = a.g->batch * TK, H = t.ld_out;
  const uint32_t* meta = (const uint32_t*)t.aux0;
  for (uint32_t b = t.b0; b < t.b1; ++b) {
    for (uint32_t c = t.c0 + threadIdx.x; c < t.c1; c += kThreads) {
      const float resid = ld_act(t.in2 + (size_t)b * H + c);
      float acc = 0.f;
      for (uint32_t k0 = 0; k0 < TK; k0 += 8u) {   // eight experts' values and weights in one round trip
        float wk[8], xk[8];
#pragma unroll
        for (uint32_t u = 0; u < 8u; ++u) {
          const uint32_t p = b * TK + min(k0 + u, TK - 1u);
          wk[u] = __uint_as_float(ld_relaxed(meta + 2 + 3 * E + P + p));
          xk[u] = ld_act(t.in + (size_t)p * t.ld_in + c);
        }
#pragma unroll
        for (uint32_t u = 0; u < 8u; ++u)
          if (k0 + u < TK) acc = fmaf(wk[u], xk[u], acc);
      }
      st_act(t.out + (size_t)b * H + c, resid + acc);
    }
  }
}

// Sum over an aligned group of N adjacent lanes (N a power of two <= 64); every lane gets it.
template <int N>
__device__ __forceinline__ float lane_group_sum(float v) {
#pragma unroll
  for (int off = N / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// T3: rotate q and k heads by the sequence position (half-split pairing), copy v, and append the
// new k and v rows to the cache as bf16.  Angles are evaluated in double precision.
__device__ __forceinline__ void body_rope(const TaskDesc& t, const StepArgs& a) {
  const uint32_t d = a.g->head_dim, half = d / 2, nq = a.g->n_q, nkv = a.g->n_kv;
  const uint32_t s0 = t.c0 / d, s1 = t.c1 / d;
  for (uint32_t b = t.b0; b < t.b1; ++b) {
    int32_t pos = as_global(a.positions)[b] + (int32_t)a.step;
    if (pos < 0 || (uint32_t)pos >= a.g->max_seq) {
      if (threadIdx.x == 0) report(a, DE_BAD_POSITION, b, (uint32_t)pos);
      continue;
    }
    const float* src = t.in + (size_t)b * t.ld_in;
    float* dst = t.out + (size_t)b * t.ld_out;
    // each thread owns two adjacent rotation pairs (i, i+1) so that cache rows are written as
    // 4-byte (two bf16) coherent stores
    for (uint32_t idx = threadIdx.x; idx < (s1 - s0) * (half / 2); idx += kThreads) {
      uint32_t s = s0 + idx / (half / 2), i = 2 * (idx % (half / 2));
      float2 lo = ld_act2(src + s * d + i), hi = ld_act2(src + s * d + i + half);
      if ((t.flags & TF_QK_NORM) && s < nq + nkv) {
        // RMSNorm over the head first: its half/2 threads are one aligned group of lanes
        float ss = lo.x * lo.x + lo.y * lo.y + hi.x * hi.x + hi.y * hi.y;
        ss = (half / 2 == 32) ? lane_group_sum<32>(ss) : lane_group_sum<16>(ss);
        const float inv = 1.0f / sqrtf(ss / (float)d + t.f0);
        const uint16_t* gn = (const uint16_t*)(s < nq ? t.w : t.w2);
        const uint32_t g0 = *as_global((const uint32_t*)(gn + i)), g1 = *as_global((const uint32_t*)(gn + i + half));
        lo.x *= inv * bf16_lo(g0); lo.y *= inv * bf16_hi(g0);
        hi.x *= inv * bf16_lo(g1); hi.y *= inv * bf16_hi(g1);
      }
      float r[4];   // lo.x, lo.y, hi.x, hi.y after rotation
      if (s < nq + nkv) {
        float u0[2] = {lo.x, lo.y}, u1[2] = {hi.x, hi.y};
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          float c, sn;
          rope_cs(a, pos, i + e, &c, &sn);
          r[e] = u0[e] * c - u1[e] * sn;
          r[2 + e] = u1[e] * c + u0[e] * sn;
        }
      } else {
        r[0] = lo.x; r[1] = lo.y; r[2] = hi.x; r[3] = hi.y;
      }
      st_act(dst + s * d + i, r[0]);
      st_act(dst + s * d + i + 1, r[1]);
      st_act(dst + s * d + i + half, r[2]);
      st_act(dst + s * d + i + half + 1, r[3]);
      if (s >= nq) {
        bool is_k = s < nq + nkv;
        uint32_t g = is_k ? s - nq : s - nq - nkv;
        uint16_t* cache = (uint16_t*)(is_k ? t.aux0 : t.aux1);
        uint16_t* row = cache + (((size_t)b * nkv + g) * a.g->max_seq + (uint32_t)pos) * d;
        st_act_u32((uint32_t*)(row + i), (uint32_t)f32_to_bf16(r[0]) | ((uint32_t)f32_to_bf16(r[1]) << 16));
        st_act_u32((uint32_t*)(row + i + half), (uint32_t)f32_to_bf16(r[2]) | ((uint32_t)f32_to_bf16(r[3]) << 16));
      }
    }
  }
}

// Position of sequence b in this step.  positions[] is the host's and stays as written for the
// whole launch (tasks add the step number) -- except in a serving launch, where the serving task
// rewrites it at the start of every step: then it holds the step's own positions and is read with
// coherent loads, after the serving task's event.
template <bool PAGED>
__device__ __forceinline__ int32_t step_position(const StepArgs& a, uint32_t b) {
  if (PAGED && (a.flags & kServeBit)) return (int32_t)ld_relaxed((const uint32_t*)a.positions + b);
  return as_global(a.positions)[b] + (int32_t)a.step;
}

// First row of chunk c of C of a sequence of len rows.  (A 64-bit division is a hundred instructions;
// up to kSmallSeq positions the product of a length and a task count (at most 16 x 64) fits 32 bits.)
constexpr uint32_t kSmallSeq = 1u << 21;
__device__ __forceinline__ uint32_t chunk_begin(const StepArgs& a, uint32_t c, uint32_t len, uint32_t C) {
  return a.g->max_seq <= kSmallSeq ? c * len / C : (uint32_t)((uint64_t)c * len / C);
}

// TF_ATTN_BALANCE: the batch x C chunk tasks of a KV head, numbered v = row x C + chunk, are dealt
// to the sequences in proportion to their lengths, every sequence at least one: sequence b gets
// 1 + floor((batch x C - batch) x len_b / total) tasks, and what is left over (fewer than batch)
// goes, one at a time, to the sequence whose chunks are longest at that moment (lowest index on
// ties).  A pure function of the positions, worked out by every wavefront for itself (lane b <
// batch holds sequence b; batch <= 16).  Returns the sequence of task v, the task's chunk number
// there, the sequence's chunk count, its first task and its position.
template <bool PAGED>
__device__ __forceinline__ void attn_deal(const StepArgs& a, uint32_t C, uint32_t v, uint32_t* seq, uint32_t* chunk,
                                          uint32_t* chunks, uint32_t* first, int32_t* position) {
  const uint32_t B = a.g->batch, li = threadIdx.x & 15u;
  uint32_t w = 0;
  int32_t pos = 0;
  if (li < B) {
    pos = step_position<PAGED>(a, li);
    w = (pos >= 0 && (uint32_t)pos < a.g->max_seq) ? (uint32_t)pos + 1u : 1u;   // (a bad position is reported by its tasks)
  }
  // within a row of 16 lanes by DPP moves (a lane shuffle is an LDS round trip, and the loop below is a
  // chain of them: at batch 16 the deal took 2.5 us ahead of the first row request)
  auto dpp = [](uint32_t x, auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xF, 0xF, true); };
  auto row_all = [&](uint32_t x, auto op) {   // op over the 16 lanes of the row, in every lane
    x = op(x, dpp(x, std::integral_constant<int, 0xB1>{}));    // lane ^ 1
    x = op(x, dpp(x, std::integral_constant<int, 0x4E>{}));    // lane ^ 2
    x = op(x, dpp(x, std::integral_constant<int, 0x141>{}));   // mirror in 8
    return op(x, dpp(x, std::integral_constant<int, 0x140>{}));   // mirror in 16
  };
  auto add = [](uint32_t x, uint32_t y) { return x + y; };
  const uint32_t total = row_all(w, add);
  uint32_t cnt = 0;
  if (li < B) cnt = 1u + (a.g->max_seq <= kSmallSeq ? (B * C - B) * w / total : (uint32_t)((uint64_t)(B * C - B) * w / total));
  const uint32_t left = B * C - row_all(cnt, add);   // uniform, < B
  for (uint32_t r = 0; r < left; ++r) {
    const float len = li < B ? (float)w / (float)cnt : 0.f;   // current chunk length of the sequence (at least 1 / cnt)
    const float mx = __uint_as_float(row_all(__float_as_uint(len), [](uint32_t x, uint32_t y) { return max(x, y); }));   // (no negative lengths)
    const uint32_t who = (uint32_t)__ballot(len == mx) & 0xFFFFu;   // (the wavefront's first 16 lanes)
    if (li == (uint32_t)__builtin_ctz(who)) ++cnt;
  }
  uint32_t end = cnt;   // inclusive prefix sum: first task after the sequence
  end += dpp(end, std::integral_constant<int, 0x111>{});   // row_shr 1, 2, 4, 8 (nothing comes in from the left)
  end += dpp(end, std::integral_constant<int, 0x112>{});
  end += dpp(end, std::integral_constant<int, 0x114>{});
  end += dpp(end, std::integral_constant<int, 0x118>{});
  const uint32_t start = end - cnt;
  const uint32_t mask = (uint32_t)__ballot(li < B && start <= v) & 0xFFFFu;
  const uint32_t bsel = 31u - (uint32_t)__builtin_clz(mask);                  // start of sequence 0 is 0 <= v
  *seq = bsel;
  *first = (uint32_t)__builtin_amdgcn_readlane((int)start, bsel);
  *chunks = (uint32_t)__builtin_amdgcn_readlane((int)cnt, bsel);
  *chunk = v - *first;
  *position = __builtin_amdgcn_readlane(pos, bsel);
}

// ------------------------------------------------------------------------------ attention on the matrix cores
// T4: split-KV decode attention for one (sequence, KV head, chunk).  Chunk c of C covers cache
// rows [c*len/C, (c+1)*len/C) with len = position + 1, so the last chunk holds the new row.
// Output per query head of the group, with the scores s times log2(e): sum_t 2^(s_t - m) V_t (D
// floats), m, l = sum_t 2^(s_t - m).
//
// Work: a wavefront takes blocks of 32 cache rows (wavefront w: blocks w, w + 8, ...), independent
// of the others until the partial results meet in LDS.  Per block
//   scores  S[32 rows][16 columns] = K[32][D] x Q[D][16]       two 16-row tiles, D / 32 multiplies each
//   p       = 2^(S - m), fp32, lane = (column, 4 rows of each tile)
//   output  O[16 rows][D] += P[16][32] x V[32][D]               D / 16 multiplies
// with v_mfma_f32_16x16x32_bf16.  Cache rows are bf16 as stored; queries and probabilities are
// fp32 and enter as the exact sum of three bf16 terms (split_hi_mid_lo), so every product is exact.
// The 16 columns (rows of P) hold the terms side by side: up to 4 query heads per KV head
// hi | mid | lo | 0 in four groups of four (fewer heads repeat), one multiply; 8 heads hi | mid in two groups of eight and a second
// multiply with lo | 0 into the same accumulators.  Adding the column groups (one or two DPP row
// rotations) leaves every lane with the whole score of its head.
//
// Why: on the vector ALUs a row costs about 135 instructions per wavefront and 4 rows (16 lanes a
// row, scores reduced over lanes, one exp per head and 16 lanes), 9 us of arithmetic alone for the
// 660-row chunks of the 8B shape at batch 8; here 32 rows cost 16 (8 heads: 32) multiplies and
// about 150 vector instructions, and the task streams.
//
// Operand layouts come without a shuffle through LDS:
//   K (A operand, lane = row + 16 x input group): loaded as 8 rows x 128 bytes per instruction and put
//     into operand order by one DPP move per register, see mfma_job_packed
//   P (A operand, lane = (head, term) + 16 x row group): the lane that holds the scores of tile rows
//     4 j .. 4 j + 3 of both tiles holds exactly 8 of the 32 inputs of the multiply; V follows that order
//   V (B operand, lane = column + 16 x row group): a lane loads its 8 rows at D / 16 consecutive
//     elements (whole rows per instruction) and transposes the 8 x (D / 16) block in its registers
//     (v_perm_b32); tile t then covers output elements (D / 16) column + t
//
// Rounding: what is left is the fp32 sums.  A score's D products go through D / 32 multiplies with
// accumulators of their own, added pairwise: chained through one accumulator every multiply rounds at the
// size the sum has reached, and an error of a score is a relative error of its weight (logits
// against 64 bits, root mean square over inputs with scores up to some tens: D = 128 with 8 query heads per KV
// head 1.53e-6 chained, 0.88e-6 pairwise, 0.99e-6 in vector arithmetic of runs of eight inputs).
//
// K and V rows of a block are requested ahead: the first block's before the task's event, the next
// K as soon as K has been multiplied, the next V likewise -- 8 to 16 KB in flight per wavefront
// (D = 128).  The requests of a round carry no branch (rows past the chunk repeat its last row), the
// loop's last round is peeled and requests nothing.
//
// Infinities: a cached element may be infinite as long as it only gives scores of -infinity (weight 0), and in
// vector arithmetic does no harm then.  Split into terms it does: infinity times the lower terms is NaN or of
// the other sign.  A NaN among the scores never leaves the sum of the weights, so a wavefront looks at that
// once, at the end, and where it is not finite does its rows again without the split.
//
// The running maximum m is only raised when a score exceeds it by more than 2^16 (lazy rescaling:
// sums and outputs are relative to m, so any m within the fp32 range gives the same digits).
//
// The row appended this step is not in the cache when rows are requested: the task of the last
// chunk has it in registers (fused RoPE), keeps the stored (bf16) values in LDS and adds it as a
// partial result of its own: m = its score, l = 1, output = the value row.
constexpr float kLazyMax = 16.f;   // in powers of two

template <int N>
__device__ __forceinline__ float row_ror(float v) {   // value of the lane N further in its row of 16
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xF, 0xF, true));
}

// Partial results of a task's sequence -> attention output, by the chunk task that arrives last:
// log-sum-exp over the C partials ([grp][d + 2]: output, max, sum each).  They are in the slots of C
// consecutive chunk tasks: rows of Cs slots, ld floats apart, from slot `slot` of the row at `row` on.
// A thread owns two adjacent output elements; all loads of up to 16 partials are in flight together
// (the loads are what this costs: 3.3 us for 16 partials when they went out 8 at a time, 2 dwords
// a partial, with an exp chain between).  They must go out without a wait between them: where the compiler finds a flat
// access nearby or a branch around each load it waits for everything, the task's own stores included.  Merge at batch 1,
// from own partial to output, 8 partials 4.4 -> 2.4 us, 16 partials of head size 64 3.0 -> 2.0; us a step: 1B class 629 -> 617, 8B 2730
// -> 2680, 2B class at batch 2, four tokens 2087 -> 2045, tiny model 36.0 -> 34.9.
// MARKED: the partials of the others say for themselves whether they are there, and the calling task's own, the
// last of the C, is in LDS (`own`: outputs [grp][d], `own_ml`: maximum and sum [grp][2]).
template <int D, int GRP, bool MARKED = false>
__device__ __forceinline__ void attn_merge_partials(uint32_t C, const float* row, uint32_t slot, uint32_t Cs, uint32_t ld, float* o,
                                                    const StepArgs& a, const TaskDesc& t, const float* own = nullptr, const float* own_ml = nullptr) {
  constexpr uint32_t per = GRP * (D + 2);
  constexpr int kAtOnce = 16;
  for (uint32_t i = threadIdx.x; i < (uint32_t)(GRP * D / 2); i += kThreads) {
    const uint32_t j = i / (D / 2), e = 2u * (i % (D / 2));
    float M = -INFINITY, L = 0.f, ax = 0.f, ay = 0.f;
    const float* part = row + (size_t)slot * per;
    uint32_t sl = slot;
    const uint32_t Cm = MARKED ? C - 1u : C;   // partials in memory
    float2 oml = make_float2(0.f, 0.f), oov = oml;
    if (MARKED) {
      oml = *(const float2*)(own_ml + 2 * j);
      oov = *(const float2*)(own + j * D + e);
    }
    if (MARKED && C == 1u) {   // (what the general case comes to)
      L = oml.y;
      ax = oov.x;
      ay = oov.y;
    } else
    for (uint32_t c0 = 0; c0 < C; c0 += kAtOnce) {
      float2 ml[kAtOnce], ov[kAtOnce];
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        ml[k] = make_float2(-INFINITY, 0.f);
        ov[k] = make_float2(0.f, 0.f);
      }
      const float* part1;
      uint32_t sl1;
      MarkWait mw;
      bool unset;
      do {
        part1 = part;
        sl1 = sl;
        unset = false;
        auto load = [&](auto kc) {
          constexpr int k = decltype(kc)::value;
          const float* pp = part1 + j * (D + 2);
          ml[k] = ld_act2(pp + D);
          ov[k] = ld_act2(pp + e);
          part1 += per;
          if (++sl1 == Cs) { sl1 = 0; part1 += ld - (size_t)Cs * per; }
        };
        // n partials in ascending entries, eight, four, two and one at a time: a branch around each of them made the compiler
        // wait for everything in flight between them (1.4 us to send off 7)
        const uint32_t n = min(Cm - min(c0, Cm), (uint32_t)kAtOnce), r = n >= 8u ? n - 8u : n;
        if (n >= 8u) static_for<0, 8>(load);
        if (r >= 4u) static_for<8, 12>(load);
        if (r & 10u) static_for<12, 14>(load);
        if (r & 9u) static_for<14, 15>(load);
        if (r & 8u) static_for<15, 16>(load);
        if (MARKED) {   // (kUnsetWord is the largest word there is)
          uint32_t top = 0;
#pragma unroll
          for (int k = 0; k < kAtOnce; ++k) top = max(top, max(mark_top(ml[k]), mark_top(ov[k])));
          asm("" : "+v"(top));   // (a vector register, also where every word is the same in all lanes)
          unset = top == kUnsetWord;
        }
      } while (MARKED && mark_wait(a, unset, mw));
      part = part1;
      sl = sl1;
      float Mn = M;
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) Mn = fmaxf(Mn, ml[k].x);
      const bool with_own = MARKED && c0 + kAtOnce >= C;   // (the last: in the order they have where all are in memory)
      if (with_own) Mn = fmaxf(Mn, oml.x);
      if (Mn == -INFINITY) continue;   // empty chunks only so far
      const float s0 = __builtin_amdgcn_exp2f(M - Mn);
      L *= s0; ax *= s0; ay *= s0;
#pragma unroll
      for (int k = 0; k < kAtOnce; ++k) {
        const float w = __builtin_amdgcn_exp2f(ml[k].x - Mn);   // 2^(-inf) = 0: empty
        L = fmaf(w, ml[k].y, L);
        ax = fmaf(w, ov[k].x, ax);
        ay = fmaf(w, ov[k].y, ay);
      }
      if (with_own) {
        const float w = __builtin_amdgcn_exp2f(oml.x - Mn);
        L = fmaf(w, oml.y, L);
        ax = fmaf(w, oov.x, ax);
        ay = fmaf(w, oov.y, ay);
      }
      M = Mn;
    }
    if (MARKED) {
      st_act2(o + 2u * i, mark_clean(ax / L), mark_clean(ay / L));
      mark_reset2(o + 2u * i, t.twin);
    } else {
      st_act2(o + 2u * i, ax / L, ay / L);
    }
  }
}

// The rows of one wavefront's blocks in vector arithmetic, into its partial results: for rows with elements that
// are not finite, see above.  Eight lanes a row, eight rows at a time, one head after the other; a row whose
// score is -infinity has weight 0 whatever its maximum.
template <int D, int GRP, uint32_t NTERM, class RowOff>
__device__ __forceinline__ void attn_rows_unsplit(const float* qs, const uint16_t* Kb, const uint16_t* Vb, RowOff row_off, uint32_t n_old,
                                                  uint32_t wave, uint32_t nblk, float scale, float* part, float* ml) {
  constexpr uint32_t EPL = D / 8, WS = D + 4;   // elements per lane
  const uint32_t lane = threadIdx.x & 63, e0 = EPL * (lane & 7u);
  auto unpack = [](const u32x4& w, float* f) {
#pragma unroll
    for (int k = 0; k < 4; ++k) { f[2 * k] = bf16_lo(w[k]); f[2 * k + 1] = bf16_hi(w[k]); }
  };
#pragma unroll 1
  for (uint32_t j = 0; j < (uint32_t)GRP; ++j) {
    float q[EPL], acc[EPL], m = -INFINITY, l = 0.f, odd = 0.f;
#pragma unroll
    for (uint32_t e = 0; e < EPL; ++e) {
      q[e] = qs[j * D + e0 + e];
      odd = fmaf(q[e], 0.f, odd);
      acc[e] = 0.f;
    }
    if (__any(odd != 0.f)) {   // a query that is not finite: no score is, and the result is NaN whatever the rows hold
      l = acc[0] = __builtin_nanf("");
#pragma unroll
      for (uint32_t e = 1; e < EPL; ++e) acc[e] = l;
    } else {
#pragma unroll 1
      for (uint32_t n = 0; wave + (n >> 2) * (kThreads / 64u) < nblk; ++n) {   // quarter n % 4 of the wavefront's block n / 4
        const uint32_t i = (wave + (n >> 2) * (kThreads / 64u)) * 32u + (n & 3u) * 8u + (lane >> 3);
        const size_t off = row_off(min(i, n_old - 1u)) + e0;
        u32x4 kw[EPL / 8], vw[EPL / 8];
#pragma unroll
        for (uint32_t h = 0; h < EPL / 8; ++h) {   // (agent-scope loads are right for every kind of launch)
          kw[h] = ld_row16_coherent(Kb + off + 8 * h);
          vw[h] = ld_row16_coherent(Vb + off + 8 * h);
        }
        float x[EPL], s = 0.f;
#pragma unroll
        for (uint32_t h = 0; h < EPL / 8; ++h) unpack(kw[h], x + 8 * h);
#pragma unroll
        for (uint32_t e = 0; e < EPL; ++e) s = fmaf(x[e], q[e], s);
        s += __shfl_xor(s, 1, 64);
        s += __shfl_xor(s, 2, 64);
        s += __shfl_xor(s, 4, 64);
        if (i < n_old && s != -INFINITY) {
          const float mn = fmaxf(m, s * scale), f = __builtin_amdgcn_exp2f(m - mn), p = __builtin_amdgcn_exp2f(fmaf(s, scale, -mn));
          m = mn;
          l = fmaf(l, f, p);
#pragma unroll
          for (uint32_t h = 0; h < EPL / 8; ++h) unpack(vw[h], x + 8 * h);
#pragma unroll
          for (uint32_t e = 0; e < EPL; ++e) acc[e] = fmaf(acc[e], f, p * x[e]);
        }
      }
      float M = m;
      for (int o = 8; o < 64; o <<= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
      const float f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
      m = M;
      l *= f;
#pragma unroll
      for (uint32_t e = 0; e < EPL; ++e) acc[e] *= f;
      for (int o = 8; o < 64; o <<= 1) {
        l += __shfl_xor(l, o, 64);
#pragma unroll
        for (uint32_t e = 0; e < EPL; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
      }
    }
    if (lane < 8u) {
#pragma unroll
      for (uint32_t e = 0; e < EPL; ++e) {
        part[j * WS + e0 + e] = acc[e];
#pragma unroll
        for (uint32_t term = 1; term < NTERM; ++term) part[(term * GRP + j) * WS + e0 + e] = 0.f;
      }
      if (lane == 0) {
        ml[2 * j] = m;
        ml[2 * j + 1] = l;
      }
    }
  }
}

// Cache rows of earlier steps are immutable during a step, so the task requests its first
// blocks of K and V rows BEFORE it waits for its dependent event; only the query (and the row
// appended this step) arrive later.
// These early reads are plain non-temporal loads.  In a multi-token launch they include the row
// another workgroup appended in the PREVIOUS step of the same launch; that is safe because (1) the
// row was written with coherent stores that completed before its task notified, and this worker
// has since waited for an event downstream of that notification (a step's first tasks wait for
// the previous step's terminal event), and (2) no cache can hold an older copy of the row's
// lines: a row fills whole 128-byte lines of its own and is never read before it is written (the
// row at the current position is excluded from the early reads and fetched coherently).
// The caller in turn must not change rows below a sequence's position while a launch runs.
// PAGED (TF_KV_PAGED; paper Section 6.1, paged attention): the cache is a pool of pages
// [kv_pages][n_kv][page][D] per layer and row r of sequence b is row r % page of page
// page_table[b][r / page].  The table (and, in a serving launch, positions[]) belong to THIS step
// only once the serving task has run, so the task first waits for that task's event -- activated
// at the very start of the step, long before the task's own event -- and only then deals the chunk
// tasks, looks up its pages and requests its rows.  Table entries are read with coherent loads
// (one per page of the chunk, all in flight together).  An entry
// outside the pool is reported and replaced by page 0: no address ever leaves the pool.
template <int D, int GRP, bool PAGED, bool MARKED>
__device__ __forceinline__ bool body_attn_mfma(const TaskDesc& t, const StepArgs& a, float* lds, int32_t wait_ev, uint32_t* s_flag) {
  constexpr uint32_t d = D, grp = GRP, NW = kThreads / 64, per = grp * (d + 2);
  constexpr bool TWO = GRP == 8;                       // the lo terms take a second multiply
  constexpr uint32_t HG = TWO ? 8u : 4u;               // columns per term group
  constexpr uint32_t NTERM = attn_term_groups(GRP);    // partial outputs per wavefront and head
  constexpr int KG = D / 64, NT = D / 16;              // 64-input groups of a score, output tiles
  constexpr uint32_t BLK = 32, WS = d + 4;
  using VVec = std::conditional_t<D == 128, u32x4, u32x2>;   // D / 16 elements of a value row
  constexpr int VW = D / 32;                                 // ... in words
  const uint32_t nq = a.g->n_q, nkv = a.g->n_kv, Cs = t.p1;
  const uint32_t bs = t.b0, u = t.c0 / per, g = u / Cs;   // the task's own row: where its partial result goes
  if (PAGED && (wait_ev >= 0 || MARKED) && a.g->serve_event >= 0 && !wait_event(a, a.g->serve_event, s_flag)) return false;
  // sequence, chunk and chunk count the task works on, first task of that sequence
  uint32_t b = bs, c = u % Cs, C = Cs, v0 = bs * Cs;
  int32_t pos;   // written by the host before the launch (or by the serving task)
  if (t.flags & TF_ATTN_BALANCE) attn_deal<PAGED>(a, Cs, bs * Cs + c, &b, &c, &C, &v0, &pos);
  else pos = (int32_t)uniform_u32((uint32_t)step_position<PAGED>(a, b));
  // a probability is 2^(s * kScale - m): one fused multiply-add and one v_exp_f32.  (The factor folded into
  // the query rounds every query element once more.)
  constexpr float kScale = (float)(1.4426950408889634074 / (D == 128 ? 11.313708498984760390 : 8.0));   // log2(e) / sqrt(d)
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* qs = lds;                                   // [grp][d]
  float* wpart = qs + grp * d;                       // [NW][NTERM][grp][WS]: partial outputs
  float* ml = wpart + NW * NTERM * grp * WS;         // [NW][grp][2]: running maximum and sum
  float* knew = ml + NW * grp * 2;                   // [d], [d]: the appended rows as stored; [8] their scores
  float* vnew = knew + d;
  float* snew = vnew + d;
  uint32_t* flag = (uint32_t*)(snew + 8);
  static_assert(grp * d + NW * NTERM * grp * WS + NW * grp * 2 + 2 * d + 8 + 16 == attn_lds_floats(D, GRP), "the host reserves this layout");
  uint32_t* pgs = flag + 16;                         // paged: the chunk's page numbers
  float* outp = t.out + (size_t)bs * t.ld_out + t.c0;
  const bool bad_pos = pos < 0 || (uint32_t)pos >= a.g->max_seq;
  const uint32_t len = bad_pos ? 0u : (uint32_t)pos + 1;
  const uint32_t t0 = chunk_begin(a, c, len, C), t1 = chunk_begin(a, c + 1u, len, C);
  const bool has_new = !bad_pos && c == C - 1;       // the chunk ends with the row appended this step
  const bool merger = MARKED && c == C - 1;      // (the latest of the sequence's tasks in every worker's order)
  const uint32_t n_old = __builtin_amdgcn_readfirstlane(t1 - t0 - (has_new ? 1u : 0u));   // rows of earlier steps
  const uint32_t nblk = (n_old + BLK - 1u) / BLK;
  // contiguous cache: the chunk's first row; paged: the layer's pools
  const uint16_t* Kb = (const uint16_t*)t.aux0 + (PAGED ? (size_t)0 : (((size_t)b * nkv + g) * a.g->max_seq + t0) * d);
  const uint16_t* Vb = (const uint16_t*)t.aux1 + (PAGED ? (size_t)0 : (((size_t)b * nkv + g) * a.g->max_seq + t0) * d);
  const uint32_t pshift = PAGED ? a.g->page_shift : 0u;
  const uint32_t pg0 = t0 >> pshift;
  bool bad_page = false;
  if constexpr (PAGED) {   // one coherent load per page, all in flight together: a row's address is then an LDS read
    const uint32_t* ptab = (const uint32_t*)a.g->page_table + (size_t)b * (a.g->max_seq >> pshift);
    const uint32_t npg = t1 > t0 ? ((t1 - 1u) >> pshift) - pg0 + 1u : 0u;
    for (uint32_t i = threadIdx.x; i < npg; i += kThreads) {
      uint32_t pg = ld_relaxed(ptab + pg0 + i);
      if (pg >= a.g->kv_pages) { bad_page = true; pg = 0; }
      pgs[i] = pg;
    }
    __syncthreads();
  }
  // element offset of row i of the chunk (row t0 + i of the sequence) from Kb / Vb
  auto row_off = [&](uint32_t i) {
    if constexpr (PAGED) {
      const uint32_t r = t0 + i;
      return ((((size_t)pgs[(r >> pshift) - pg0] * nkv + g) << pshift) + (r & ((1u << pshift) - 1u))) * d;
    } else {
      return (size_t)i * d;
    }
  };
  const uint32_t col = lane & 15u, jg = (uint32_t)lane >> 4;   // column / row of an operand, its input group
  u32x4 kreg[2][KG][2];   // [tile][64-input group][rows 0..7 / 8..15]
  VVec vreg[8];           // [row slot]
  // `coherent`: a paged cache in a launch of several steps is read with agent-scope loads (a page may
  // have changed owners within the launch) -- a compile-time choice, made once per task by the callers
  auto request_k = [&](auto coherent, uint32_t blk) {
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t i = min(blk * BLK + 16u * T + 8u * h + (lane & 7u), n_old - 1u);
        const uint16_t* p = Kb + row_off(i) + 8u * ((uint32_t)lane >> 3);
#pragma unroll
        for (int q = 0; q < KG; ++q) kreg[T][q][h] = decltype(coherent)::value ? ld_row16_coherent(p + 64 * q) : ld_stream16(p + 64 * q);
      }
  };
  auto request_v = [&](auto coherent, uint32_t blk) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const uint32_t i = min(blk * BLK + 16u * (s >> 2) + 4u * jg + (s & 3), n_old - 1u);
      const uint16_t* p = Vb + row_off(i) + (uint32_t)NT * col;
      if constexpr (D == 128) {
        vreg[s] = decltype(coherent)::value ? ld_row16_coherent(p) : ld_stream16(p);
      } else {
        if (decltype(coherent)::value) {
          const uint64_t w = __hip_atomic_load(as_global((const uint64_t*)p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          vreg[s] = u32x2{(uint32_t)w, (uint32_t)(w >> 32)};
        } else {
          vreg[s] = __builtin_nontemporal_load(as_global((const u32x2*)p));
        }
      }
    }
  };
  const bool coherent_rows = PAGED && !(a.flags & kOneStepBit);
  const bool mine = wave < nblk;   // (uniform) this wavefront has blocks
  auto first_rows = [&]() {
    if (!mine) return;
    if (coherent_rows) { request_k(std::true_type{}, wave); request_v(std::true_type{}, wave); }
    else { request_k(std::false_type{}, wave); request_v(std::false_type{}, wave); }
  };
  const bool preload = !(a.flags & kNoPreloadBit);
  // A wavefront's loads complete in the order they were issued: a poll behind the row requests
  // returns behind the rows.  So the first look at the event goes out ahead of them.
  EventProbe probe{};
  if (wait_ev >= 0 && wave == 0) probe = probe_event(a, wait_ev, lane);
  if (preload) {
    first_rows();
    asm volatile("; cache rows requested" ::: "memory");
  }
  if (wait_ev >= 0 && !wait_event(a, wait_ev, s_flag, probe)) return false;
  trace_mark(a, t, 1);
  if (!preload) {
    first_rows();
    asm volatile("; cache rows requested after the event" ::: "memory");
  }
  if (bad_pos) {
    if (threadIdx.x == 0) report(a, DE_BAD_POSITION, b, (uint32_t)pos);
    for (uint32_t i = threadIdx.x; i < per; i += kThreads) {
      if (!merger) st_act(outp + i, ((i % (d + 2)) == d) ? -INFINITY : 0.f);
      if (MARKED) mark_reset(outp + i, t.twin);
    }
    if (merger) {
      float* o = const_cast<float*>(t.in2) + (size_t)b * nq * d + (size_t)g * grp * d;
      for (uint32_t i = threadIdx.x; i < grp * d; i += kThreads) {
        st_act(o + i, 0.f);
        mark_reset(o + i, t.twin);
      }
    }
    return true;
  }
  const float* qsrc = t.in + (size_t)b * t.ld_in + (size_t)g * grp * d;
  uint16_t *krow = nullptr, *vrow = nullptr;   // the appended row in the cache
  if (has_new) {
    if constexpr (PAGED) {
      const size_t off = row_off((uint32_t)pos - t0);
      krow = const_cast<uint16_t*>(Kb) + off;
      vrow = const_cast<uint16_t*>(Vb) + off;
    } else {
      krow = (uint16_t*)t.aux0 + (((size_t)b * nkv + g) * a.g->max_seq + (uint32_t)pos) * d;
      vrow = (uint16_t*)t.aux1 + (((size_t)b * nkv + g) * a.g->max_seq + (uint32_t)pos) * d;
    }
  }
  if (t.flags & TF_ROPE_FUSED) {
    // the input is the raw QKV projection: rotate the group's query heads here; the task of the
    // last chunk also rotates this step's key, and appends key and value to the cache
    constexpr uint32_t half = d / 2;
    const float* angles = a.g->rope_tab + ((size_t)(a.epoch & 1u) * a.g->batch + b) * d;   // of this step, from the embedding tasks
    const bool qk_norm = t.flags & TF_QK_NORM;
    // a thread loads a rotation pair of the queries and, from the top of the workgroup, one of the appended
    // rows' shares -- two adjacent rotation pairs of the key or two adjacent value elements: one round trip
    static_assert(grp * half <= kThreads && half / 2 + half <= kThreads, "a thread has one pair of each");
    const uint32_t iq = threadIdx.x, in = kThreads - 1 - threadIdx.x;
    const bool has_q = iq < grp * half, has_k = has_new && in < half / 2, has_v = has_new && !has_k && in < half / 2 + half;
    const uint32_t jq = iq / half, eq = iq % half, ek = 2 * in, ev = 2 * (in - half / 2);
    const float* kvsrc = t.in + (size_t)b * t.ld_in + (has_k ? (size_t)(nq + g) * d + ek : (size_t)(nq + nkv + g) * d + ev);
    float u0 = 0.f, u1 = 0.f;
    float2 lo = make_float2(0.f, 0.f), hi = lo, rq = lo, r0 = lo, r1 = lo;
    MarkWait mw;
    uint32_t top;
    do {
      if (has_q) {
        u0 = ld_act(qsrc + jq * d + eq);
        u1 = ld_act(qsrc + jq * d + eq + half);
        rq = ld_act2(angles + 2u * eq);   // (cos, sin)
      }
      if (has_k || has_v) lo = ld_act2(kvsrc);
      if (has_k) {
        hi = ld_act2(kvsrc + half);
        r0 = ld_act2(angles + 2u * ek);
        r1 = ld_act2(angles + 2u * ek + 2u);
      }
      top = max(max(max(mark_top(u0), mark_top(u1)), max(mark_top(lo), mark_top(hi))), max(mark_top(rq), max(mark_top(r0), mark_top(r1))));
      asm("" : "+v"(top));
    } while (MARKED && mark_wait(a, top == kUnsetWord, mw));
    if (has_q) {
      if (qk_norm) {   // RMSNorm over the head: its `half` threads are one aligned group of lanes
        // (spelt out like the rotation below: left to the compiler, which square is rounded first depends on the code around it)
        const float inv = 1.0f / sqrtf(lane_group_sum<(int)half>(fmaf(u0, u0, u1 * u1)) / (float)d + t.f0);
        const uint16_t* gq = (const uint16_t*)t.w;
        u0 *= inv * bf16_to_f32(as_global(gq)[eq]);
        u1 *= inv * bf16_to_f32(as_global(gq)[eq + half]);
      }
      qs[jq * d + eq] = fmaf(u0, rq.x, -(u1 * rq.y));   // (spelt out: the same rounding in every instance)
      qs[jq * d + eq + half] = fmaf(u1, rq.x, u0 * rq.y);
    }
    if (has_k) {
      if (qk_norm) {   // the key's half/2 threads: one aligned group of lanes at the top of the workgroup
        const float ss = lane_group_sum<(int)(half / 2)>(fmaf(hi.y, hi.y, fmaf(hi.x, hi.x, fmaf(lo.x, lo.x, lo.y * lo.y))));
        const float inv = 1.0f / sqrtf(ss / (float)d + t.f0);
        const uint16_t* gk = (const uint16_t*)t.w2;
        const uint32_t g0 = *as_global((const uint32_t*)(gk + ek)), g1 = *as_global((const uint32_t*)(gk + ek + half));
        lo.x *= inv * bf16_lo(g0); lo.y *= inv * bf16_hi(g0);
        hi.x *= inv * bf16_lo(g1); hi.y *= inv * bf16_hi(g1);
      }
      const uint32_t w0 = (uint32_t)f32_to_bf16(fmaf(lo.x, r0.x, -(hi.x * r0.y))) | ((uint32_t)f32_to_bf16(fmaf(lo.y, r1.x, -(hi.y * r1.y))) << 16);
      const uint32_t w1 = (uint32_t)f32_to_bf16(fmaf(hi.x, r0.x, lo.x * r0.y)) | ((uint32_t)f32_to_bf16(fmaf(hi.y, r1.x, lo.y * r1.y)) << 16);
      st_act_u32((uint32_t*)(krow + ek), w0);
      st_act_u32((uint32_t*)(krow + ek + half), w1);
      *(float2*)(knew + ek) = make_float2(bf16_lo(w0), bf16_hi(w0));   // as stored
      *(float2*)(knew + ek + half) = make_float2(bf16_lo(w1), bf16_hi(w1));
    }
    if (has_v) {
      const uint32_t w = (uint32_t)f32_to_bf16(lo.x) | ((uint32_t)f32_to_bf16(lo.y) << 16);
      st_act_u32((uint32_t*)(vrow + ev), w);
      *(float2*)(vnew + ev) = make_float2(bf16_lo(w), bf16_hi(w));
    }
  } else {
    for (uint32_t i = threadIdx.x; i < grp * d; i += kThreads) qs[i] = ld_act(qsrc + i);
    if (has_new && threadIdx.x < d) {   // appended by the RoPE operator's task: coherent loads, two elements a thread
      const uint16_t* row = threadIdx.x < d / 2 ? krow : vrow;
      const uint32_t e = 2u * (threadIdx.x % (d / 2)), w = ld_relaxed((const uint32_t*)(row + e));
      *(float2*)((threadIdx.x < d / 2 ? knew : vnew) + e) = make_float2(bf16_lo(w), bf16_hi(w));
    }
  }
  lds_barrier();   // (published is LDS: nobody waits for the appended rows' stores here)
  trace_mark(a, t, 2);
  if (has_new && wave < grp) {   // score of the appended row for head `wave`
    float s = 0.f;
#pragma unroll
    for (uint32_t e = lane; e < d; e += 64) s = fmaf(qs[wave * d + e], knew[e], s);
    s = wave_sum_dpp(s);
    if (lane == 0) snew[wave] = s;
  }
  if (mine) {
    // ---- query operand: lane = column (term group, head) + 16 x input group, see above
    const uint32_t tg = col / HG, hd = (col % HG) % grp;
    u32x4 qop[KG][2], qlo[TWO ? KG : 1][2];   // (qlo: the second multiply of 8 heads)
#pragma unroll
    for (int q = 0; q < KG; ++q)
#pragma unroll
      for (int U = 0; U < 2; ++U) {
        const float* src = qs + hd * d + 64 * q + 8u * (2u * jg + U);
        u32x4 h, m, l;
        const u32x4 zero = {0u, 0u, 0u, 0u};
        split8(*(const float4*)src, *(const float4*)(src + 4), &h, &m, &l);
        if constexpr (TWO) {
          qop[q][U] = select4(tg == 0u, h, m);
          qlo[q][U] = select4(tg == 0u, l, zero);
        } else {
          qop[q][U] = select4(tg == 0u, h, select4(tg == 1u, m, select4(tg == 2u, l, zero)));
        }
      }
    float m = -INFINITY, lsum = 0.f;   // of head hd (the same in every lane of the head; lsum: this lane's rows)
    f32x4 O[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) O[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto block = [&](auto coherent, auto more, uint32_t blk) {
      // ---- scores: 32 inputs at a time, added up pairwise (see above)
      f32x4 S[2];
#pragma unroll
      for (int T = 0; T < 2; ++T) {
        f32x4 part[KG];
#pragma unroll
        for (int q = 0; q < KG; ++q) {
          pair_to_operands(kreg[T][q][0], kreg[T][q][1]);
          auto mul = [&](int U) {
            const bf16x8 kv = __builtin_bit_cast(bf16x8, kreg[T][q][U]);
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if constexpr (TWO) v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kv, __builtin_bit_cast(bf16x8, qlo[q][U]), v, 0, 0, 0);
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(kv, __builtin_bit_cast(bf16x8, qop[q][U]), v, 0, 0, 0);
          };
          part[q] = mul(0) + mul(1);
        }
        S[T] = KG == 2 ? part[0] + part[KG - 1] : part[0];
        __builtin_amdgcn_sched_barrier(0);   // (both tiles' sums at once take five more registers, which the callers' long-lived values lose)
      }
      if (decltype(more)::value) request_k(coherent, blk + NW);
      float s[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        float v = S[k >> 2][k & 3];
        v += row_ror<8>(v);
        if constexpr (!TWO) v += row_ror<4>(v);
        s[k] = v;
      }
      if ((blk + 1u) * BLK > n_old) {   // (uniform) the chunk's last, partial block
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (blk * BLK + 16u * (k >> 2) + 4u * jg + (k & 3) >= n_old) s[k] = -INFINITY;
      }
      float mx = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
      mx *= kScale;
      if (__any(mx > m + kLazyMax)) {   // a new maximum: the first block, and seldom after it
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float mn = fmaxf(m, mx);
        const float sc = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - mn);   // 2^(-inf) = 0 on the first block
        m = mn;
        lsum *= sc;
        // output row 4 jg + r belongs to head (4 jg + r) % HG: its factor sits in lane (head)
        float so[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float f0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), r));
          const float f1 = TWO ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), 4 + r)) : f0;
          so[r] = (jg & 1u) ? f1 : f0;
        }
#pragma unroll
        for (int k = 0; k < NT; ++k)
#pragma unroll
          for (int r = 0; r < 4; ++r) O[k][r] *= so[r];
      }
      // ---- probabilities, as the A operand of the second product
      float p[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        p[k] = __builtin_amdgcn_exp2f(fmaf(s[k], kScale, -m));
        lsum += p[k];
      }
      u32x4 ph, pm, pl, pop, plo;
      const u32x4 zero = {0u, 0u, 0u, 0u};
      split8(make_float4(p[0], p[1], p[2], p[3]), make_float4(p[4], p[5], p[6], p[7]), &ph, &pm, &pl);
      if constexpr (TWO) {
        pop = select4(tg == 0u, ph, pm);
        plo = select4(tg == 0u, pl, zero);
      } else {
        pop = select4(tg == 0u, ph, select4(tg == 1u, pm, select4(tg == 2u, pl, zero)));
      }
      // ---- outputs: tile k = elements NT col + k of the value rows
#pragma unroll
      for (int w = 0; w < VW; ++w)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const uint32_t sel = hf ? 0x07060302u : 0x05040100u;   // upper / lower halves of two rows' words
          u32x4 vo;
#pragma unroll
          for (int k = 0; k < 4; ++k) vo[k] = __builtin_amdgcn_perm(vreg[2 * k + 1][w], vreg[2 * k][w], sel);
          const bf16x8 vv = __builtin_bit_cast(bf16x8, vo);
          O[2 * w + hf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pop), vv, O[2 * w + hf], 0, 0, 0);
          if constexpr (TWO) O[2 * w + hf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, plo), vv, O[2 * w + hf], 0, 0, 0);
        }
      if (decltype(more)::value) request_v(coherent, blk + NW);
    };
    auto blocks = [&](auto coherent) {
      uint32_t blk = wave;
      for (; blk + NW < nblk; blk += NW) block(coherent, std::true_type{}, blk);
      block(coherent, std::false_type{}, blk);
    };
    if (coherent_rows) blocks(std::true_type{});
    else blocks(std::false_type{});
    // ---- the wavefront's partial results to LDS
    lsum += __shfl_xor(lsum, 16, 64);
    lsum += __shfl_xor(lsum, 32, 64);
    const bool finite = !__any(!(lsum < INFINITY));
    if (__builtin_expect(!finite, 0))
      attn_rows_unsplit<D, GRP, NTERM>(qs, Kb, Vb, row_off, n_old, wave, nblk, kScale, wpart + (size_t)wave * NTERM * grp * WS, ml + wave * grp * 2);
    if (finite && (uint32_t)lane < grp) {
      ml[(wave * grp + lane) * 2] = m;
      ml[(wave * grp + lane) * 2 + 1] = lsum;
    }
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) {
      const uint32_t row = 4u * jg + r, term = row / HG, head = row % HG;
      if (finite && term < NTERM && head < grp) {
        float* wp = wpart + (((size_t)wave * NTERM + term) * grp + head) * WS + (uint32_t)NT * col;
#pragma unroll
        for (int k = 0; k < NT; k += 4) *(float4*)(wp + k) = make_float4(O[k][r], O[k + 1][r], O[k + 2][r], O[k + 3][r]);
      }
    }
  }
  if (PAGED && bad_page) report(a, DE_BAD_PAGE, b, t0);   // (the rows came from page 0 instead: wrong, but in bounds)
  lds_barrier();
  trace_mark(a, t, 10);
  // ---- the wavefronts' results and the appended row -> the task's partial result, two elements a thread
  const uint32_t nw = min(nblk, NW);
  float* own_ml = (float*)flag;   // (nobody needs the queries or the flag any more)
  // (the thread of a head's first elements leaves its maximum and sum as well: threads of their own for those were
  // a second round of a loop with 8 heads of 128 elements, 1.0 us a task against 0.8 .. 1.8)
  static_assert(grp * d / 2 <= kThreads, "a thread has two elements");
  if (threadIdx.x < grp * d / 2) {
    const uint32_t j = threadIdx.x / (d / 2), e = 2u * (threadIdx.x % (d / 2));
    float mw[NW], M = has_new ? snew[j] * kScale : -INFINITY;
#pragma unroll
    for (uint32_t w = 0; w < NW; ++w) {
      mw[w] = w < nw ? ml[(w * grp + j) * 2] : -INFINITY;
      M = fmaxf(M, mw[w]);
    }
    const float Mr = M == -INFINITY ? 0.f : M;   // (every score -infinity: all weights 0)
    float x = 0.f, y = 0.f;
    const float wn = has_new ? __builtin_amdgcn_exp2f(fmaf(snew[j], kScale, -Mr)) : 0.f;
    float l = wn;
    if (has_new) { x = wn * vnew[e]; y = wn * vnew[e + 1]; }
#pragma unroll
    for (uint32_t w = 0; w < NW; ++w) {
      if (w >= nw) continue;
      const float f = __builtin_amdgcn_exp2f(mw[w] - Mr);
      l = fmaf(ml[(w * grp + j) * 2 + 1], f, l);
      float ox = 0.f, oy = 0.f;
#pragma unroll
      for (uint32_t term = 0; term < NTERM; ++term) {
        const float2 v = *(const float2*)(wpart + (((size_t)w * NTERM + term) * grp + j) * WS + e);
        ox += v.x; oy += v.y;
      }
      x = fmaf(f, ox, x);
      y = fmaf(f, oy, y);
    }
    // (M is a power of two's exponent, like everything the merges do with it)
    if (merger) {   // (stays here: this task merges)
      *(float2*)(qs + j * d + e) = make_float2(mark_clean(x), mark_clean(y));
      if (e == 0) *(float2*)(own_ml + 2u * j) = make_float2(mark_clean(M), mark_clean(l));
    } else {
      st_act2(outp + j * (d + 2) + e, MARKED ? mark_clean(x) : x, MARKED ? mark_clean(y) : y);
      if (e == 0) st_act2(outp + j * (d + 2) + d, MARKED ? mark_clean(M) : M, MARKED ? mark_clean(l) : l);
    }
  }
  trace_mark(a, t, 11);
  if constexpr (MARKED) {
    // No arrival counter: the sequence's last task in linearized order merges, and loads the others' partials
    // until they are there.  (Every worker runs its tasks in that order, so they never wait for this one.)
    if (merger) {
      lds_barrier();
      attn_merge_partials<D, GRP, true>(C, t.out + (size_t)(v0 / Cs) * t.ld_out + (size_t)g * Cs * per, v0 % Cs, Cs, t.ld_out,
                                        const_cast<float*>(t.in2) + (size_t)b * nq * d + (size_t)g * grp * d, a, t, qs, own_ml);
    }
    // (behind the merge: its loads would come back behind the acknowledgement of these stores)
    for (uint32_t i = threadIdx.x; i < per / 2; i += kThreads) mark_reset2(outp + 2u * i, t.twin);
  } else if (t.flags & TF_ATTN_MERGE) {
    // Arrival counter of (layer, sequence, KV head): the chunk task that arrives last sees all C
    // partials complete and merges them into the attention output.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    drain_vmem();
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t* cnt = a.g->grp_counters + t.p2 + b * nkv + g;
      uint32_t old = __hip_atomic_fetch_add(as_global(cnt), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (t.flags & TF_ATTN_BALANCE) {
        // the count changes with the lengths from step to step: the last arrival puts the counter
        // back to zero (nobody else touches it before the next step's attention tasks)
        *flag = (old + 1u == C) ? 1u : 0u;
        if (old + 1u == C) st_act_u32(cnt, 0u);
      } else {
        *flag = ((old + 1u) % C == 0u) ? 1u : 0u;   // every step adds exactly C
      }
    }
    __syncthreads();
    if (*flag) {
      // chunk k of the sequence is the partial result of task v0 + k, in that task's own slot
      attn_merge_partials<D, GRP>(C, t.out + (size_t)(v0 / Cs) * t.ld_out + (size_t)g * Cs * per, v0 % Cs, Cs, t.ld_out, const_cast<float*>(t.in2) + (size_t)b * nq * d + (size_t)g * grp * d, a, t);
    }
  }
  if constexpr (MARKED) {
    lds_barrier();
    if (mark_aborted()) { mark_report((uint32_t)t.dep_event); return false; }
  }
  return true;
}

// T5: merge the chunk partials of each query head with the log-sum-exp rule.
__device__ __forceinline__ void body_attn_merge(const TaskDesc& t, const StepArgs& a) {
  const uint32_t d = a.g->head_dim, grp = a.g->n_q / a.g->n_kv, C = t.p1;
  const uint32_t h0 = t.c0 / d, h1 = t.c1 / d;
  for (uint32_t b = t.b0; b < t.b1; ++b) {
    const float* part = t.in + (size_t)b * t.ld_in;
    float* out = t.out + (size_t)b * t.ld_out;
    for (uint32_t idx = threadIdx.x; idx < (h1 - h0) * d; idx += kThreads) {
      uint32_t h = h0 + idx / d, dim = idx % d, g = h / grp, j = h % grp;
      float M = -INFINITY;
      for (uint32_t c = 0; c < C; ++c) M = fmaxf(M, ld_act(part + ((size_t)(g * C + c) * grp + j) * (d + 2) + d));
      float L = 0.f, o = 0.f;
      for (uint32_t c = 0; c < C; ++c) {
        const float* p = part + ((size_t)(g * C + c) * grp + j) * (d + 2);
        float wgt = __builtin_amdgcn_exp2f(ld_act(p + d) - M);   // maxima are powers of two; 2^(-inf) = 0 for empty chunks
        L = fmaf(wgt, ld_act(p + d + 1), L);
        o = fmaf(wgt, ld_act(p + dim), o);
      }
      st_act(out + h * d + dim, o / L);
    }
  }
}

__device__ __forceinline__ void body_add(const TaskDesc& t) {
  const uint32_t nc = t.c1 - t.c0;
  for (uint32_t b = t.b0; b < t.b1; ++b)
    for (uint32_t i = threadIdx.x; i < nc; i += kThreads) {
      size_t o = (size_t)b * t.ld_out + t.c0 + i;
      st_act(t.out + o, ld_act(t.in + o) + ld_act(t.in2 + o));
    }
}

__device__ __forceinline__ void body_swiglu(const TaskDesc& t) {
  const uint32_t nc = t.c1 - t.c0, F = t.p0;
  for (uint32_t b = t.b0; b < t.b1; ++b)
    for (uint32_t i = threadIdx.x; i < nc; i += kThreads) {
      const float* gu = t.in + (size_t)b * t.ld_in;
      float gte = ld_act(gu + t.c0 + i), up = ld_act(gu + F + t.c0 + i);
      st_act(t.out + (size_t)b * t.ld_out + t.c0 + i, gte / (1.0f + expf(-gte)) * up);
    }
}

// Greedy sampling: the index of the largest logit of a sequence, lowest index on ties.  T tasks
// per sequence (t.p1): task j scans logits [V j / T, V (j+1) / T) -- it depends only on the LM-head
// tasks that produce them -- and leaves (largest value, its index) in its pair of the output row;
// the task of a sequence that arrives last (arrival counter t.p2 + sequence, T arrivals per step)
// picks the token from the T pairs.  The token goes to token_ids[b] for the next step's embedding
// task (and to tokens_out); the last step of a launch also advances positions[b].  Optionally
// keeps a copy of the logits.
__device__ __forceinline__ void body_argmax(const TaskDesc& t, const StepArgs& a, float* lds) {
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t V = t.K, B = a.g->batch, T = t.p1, j = t.c0 / 2u;
  const uint32_t q = V / T, r = V % T;
  const uint32_t v0 = j * q + min(j, r), v1 = (j + 1u) * q + min(j + 1u, r);   // the even split of V into T shares
  float* vmax = lds;                          // [8]
  uint32_t* imax = (uint32_t*)(lds + 8);      // [8]
  for (uint32_t b = t.b0; b < t.b1; ++b) {
    const float* row = a.logits + (size_t)b * V;
    float* const logits_all = a.g->logits_all;
    int32_t* const tokens_out = a.g->tokens_out;
    float* copy = logits_all ? logits_all + ((size_t)a.step * B + b) * V : nullptr;
    float best = -INFINITY;
    uint32_t best_i = 0xFFFFFFFFu;
    // One workgroup reads its share with coherent loads: what counts is how many of them are in
    // flight (one at a time, the row of a 152k vocabulary took about 150 us -- 5 % of a batch-1
    // step of the 8B shape).  32 per thread are requested before the first is looked at.
    constexpr int kInFlight = 32;
    for (uint32_t i0 = v0 + threadIdx.x; i0 < v1; i0 += kThreads * kInFlight) {   // ascending per thread: keeps the first maximum
      float v[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const uint32_t i = i0 + (uint32_t)u * kThreads;
        v[u] = i < v1 ? ld_act(row + i) : 0.f;
      }
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const uint32_t i = i0 + (uint32_t)u * kThreads;
        if (i < v1) {
          if (copy) as_global(copy)[i] = v[u];
          if (v[u] > best || best_i == 0xFFFFFFFFu) { best = v[u]; best_i = i; }
        }
      }
    }
    const float wbest = wave_max(best);
    const uint32_t wi = wave_min_u32(best == wbest ? best_i : 0xFFFFFFFFu);
    if (lane == 0) { vmax[wave] = wbest; imax[wave] = wi; }
    lds_barrier();
    if (threadIdx.x == 0) {
      float m = vmax[0];
      uint32_t mi = imax[0];
      for (uint32_t w = 1; w < kThreads / 64; ++w)
        if (vmax[w] > m || (vmax[w] == m && imax[w] < mi)) { m = vmax[w]; mi = imax[w]; }
      bool pick = true;
      if (T > 1u) {
        float* pairs = t.out + (size_t)b * t.ld_out;
        st_act(pairs + 2u * j, m);
        st_act_u32((uint32_t*)pairs + 2u * j + 1u, mi);
        drain_vmem();   // the pair is in place before the arrival counts
        uint32_t* cnt = a.g->grp_counters + t.p2 + b;
        const uint32_t old = __hip_atomic_fetch_add(as_global(cnt), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        pick = (old + 1u) % T == 0u;   // every step adds exactly T
        if (pick) {
          float pm[32];
          uint32_t pi[32];
#pragma unroll
          for (uint32_t k = 0; k < 32u; ++k) {
            if (k < T) { pm[k] = ld_act(pairs + 2u * k); pi[k] = ld_relaxed((const uint32_t*)pairs + 2u * k + 1u); }
          }
          m = pm[0];
          mi = pi[0];
#pragma unroll
          for (uint32_t k = 1; k < 32u; ++k)
            if (k < T && pm[k] > m) { m = pm[k]; mi = pi[k]; }   // shares ascend with k: the first maximum stays
        }
      }
      if (pick) {
        if (mi >= V) mi = 0;   // logits that are not numbers: keep the token in range
        st_act_u32((uint32_t*)const_cast<int32_t*>(a.token_ids) + b, mi);
        if (tokens_out) st_act_u32((uint32_t*)tokens_out + (size_t)a.step * B + b, mi);
        if ((uint32_t)a.step + 1u == a.n_steps && !(a.flags & kServeBit))   // (a serving launch: the serving task keeps the positions)
          st_act_u32((uint32_t*)const_cast<int32_t*>(a.positions) + b, (uint32_t)(as_global(a.positions)[b] + (int32_t)a.n_steps));
      }
    }
    lds_barrier();
  }
}

// The task on the start event of a serving graph (paper Section 6.1: the scheduler prepares a new
// decoding iteration by (1) removing completed requests, (2) admitting newly arrived requests and
// (3) updating the per-request KV-cache metadata; "this logic executes as a single task").  The
// paper fixes no policy; this one is the library's contract (mpk_serve_* in the public header):
//   (1) a slot whose request still has prompt tokens is fed the next one (the sampled token is
//       ignored: prompts go through the decode path a token per iteration); otherwise the sampled
//       token is the request's next output, and the request is finished on the end-of-sequence
//       token or with max_new tokens.  Finished slots, in ascending order, push their pages onto
//       the free stack in page-table order.
//   (2) idle slots, in ascending order, take the queued requests in arrival order, each only if
//       the pages it can ever need, ceil((prompt + max_new - 1) / page), are free and not promised
//       to running requests; the first request that does not fit ends admission (no overtaking).
//   (3) a running slot whose position is at a page boundary pops a page (ascending slot order);
//       an idle slot computes on token 0 at position 0 in its own page (page number = slot).
// One wavefront, lane b = slot b (batch <= 16): every slot's state is loaded and stored once, the
// sequential decisions (stack positions, admission) are prefix counts over lanes, so the task is
// a handful of memory round trips however many slots change.  All state is read and written with
// agent-scope accesses: attention tasks on other compute units read the tables in the same step.
__device__ __forceinline__ void body_serve(const StepArgs& a) {
  const ServeDev* Sp = a.g->serve;
  if (threadIdx.x >= 64 || Sp == nullptr) return;
  const ServeDev sv = *Sp;
  const uint32_t lane = threadIdx.x, B = a.g->batch, n_pages = a.g->kv_pages;
  const uint32_t shift = sv.page_shift, ps_mask = (1u << shift) - 1u;
  const bool mine = lane < B;
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t* tok_io = (uint32_t*)const_cast<int32_t*>(a.token_ids);
  uint32_t* pos_io = (uint32_t*)const_cast<int32_t*>(a.positions);
  int32_t req = mine ? (int32_t)ld_relaxed((const uint32_t*)sv.slot_req + lane) : -1;
  uint32_t pos = mine ? ld_relaxed((const uint32_t*)sv.slot_pos + lane) : 0u;
  uint32_t held = mine ? ld_relaxed((const uint32_t*)sv.slot_held + lane) : 0u;
  const uint32_t sampled = mine ? ld_relaxed(tok_io + lane) : 0u;
  uint32_t n_free = __builtin_amdgcn_readfirstlane(ld_relaxed(sv.scalars + kServeNFree));
  uint32_t promised = __builtin_amdgcn_readfirstlane(ld_relaxed(sv.scalars + kServePromised));
  uint32_t q_head = __builtin_amdgcn_readfirstlane(ld_relaxed(sv.scalars + kServeQHead));
  const uint32_t q_tail = __builtin_amdgcn_readfirstlane(ld_relaxed(sv.scalars + kServeQTail));
  auto pages_of = [&](uint32_t plen, uint32_t max_new) { return (plen + max_new - 1u + ps_mask) >> shift; };
  // ---- (1) completed requests leave
  uint32_t nxt = 0, need = 0;
  bool done = false, produced = false;
  if (req >= 0) {
    const uint32_t plen = ld_relaxed(sv.req_len + 2 * (size_t)req), max_new = ld_relaxed(sv.req_len + 2 * (size_t)req + 1);
    need = pages_of(plen, max_new);
    const uint32_t cached = pos + 1u;
    if (cached < plen) {
      nxt = ld_relaxed((const uint32_t*)sv.req_prompt + (size_t)req * sv.max_prompt + cached);
    } else {
      uint32_t n_out = ld_relaxed(sv.req_state + 2 * (size_t)req + 1);
      if (n_out < sv.max_new) st_act_u32((uint32_t*)sv.req_out + (size_t)req * sv.max_new + n_out, sampled);
      ++n_out;
      st_act_u32(sv.req_state + 2 * (size_t)req + 1, n_out);
      nxt = sampled;
      produced = true;
      done = (int32_t)sampled == sv.eos || n_out >= max_new;
    }
    pos = cached;
  }
  const uint32_t n_produced = (uint32_t)__builtin_popcountll(__ballot(produced));
  const uint32_t n_done = (uint32_t)__builtin_popcountll(__ballot(done));
  for (uint64_t retiring = __ballot(done); retiring; retiring &= retiring - 1ull) {
    const uint32_t b = (uint32_t)__builtin_ctzll(retiring);
    const uint32_t hb = (uint32_t)__builtin_amdgcn_readlane((int)held, (int)b);
    const uint32_t nb = (uint32_t)__builtin_amdgcn_readlane((int)need, (int)b);
    uint32_t* row = (uint32_t*)sv.table + (size_t)b * sv.max_blocks;
    for (uint32_t i = lane; i < hb && i < sv.max_blocks; i += 64u) {
      const uint32_t pg = ld_relaxed(row + i);
      if (n_free + i < n_pages) st_act_u32((uint32_t*)sv.free_stack + n_free + i, pg);
      st_act_u32(row + i, i == 0u ? b : 0xFFFFFFFFu);   // the idle slot's own page; the rest: none
    }
    n_free += hb;
    promised -= nb - hb;
  }
  if (done) {
    st_act_u32(sv.req_state + 2 * (size_t)req, 2u);
    req = -1;
    held = 0;
    pos = 0;
  }
  // ---- (1b) the running requests close ranks: in order, to the lowest slots (a slot is metadata
  // only, the rows stay in their pages), so that the graph of a smaller batch size can serve them
  {
    const uint64_t run_mask = __ballot(mine && req >= 0);
    const uint32_t n_run = (uint32_t)__builtin_popcountll(run_mask);
    if (run_mask != (1ull << n_run) - 1ull) {   // (uniform) there are gaps
      uint32_t my_src = lane, k = 0;
      for (uint64_t m = run_mask; m; m &= m - 1ull, ++k) {
        const uint32_t src = (uint32_t)__builtin_ctzll(m);
        if (lane == k) my_src = src;
        if (src == k) continue;
        // page-table row src -> row k (k < src; rows below k are final, rows above src untouched so far)
        const uint32_t hb = (uint32_t)__builtin_amdgcn_readlane((int)held, (int)src);
        uint32_t* from = (uint32_t*)sv.table + (size_t)src * sv.max_blocks;
        uint32_t* to = (uint32_t*)sv.table + (size_t)k * sv.max_blocks;
        for (uint32_t i = lane; i < sv.max_blocks; i += 64u) {
          const uint32_t v = i < hb ? ld_relaxed(from + i) : 0xFFFFFFFFu;
          st_act_u32(to + i, v);
          st_act_u32(from + i, i == 0u ? src : 0xFFFFFFFFu);   // vacated (a later move may fill it again)
        }
        drain_vmem();   // the next move may read what this one wrote
      }
      const int src_lane = (int)my_src;
      const int32_t req_m = __shfl(req, src_lane, 64);
      const uint32_t pos_m = (uint32_t)__shfl((int)pos, src_lane, 64), held_m = (uint32_t)__shfl((int)held, src_lane, 64);
      const uint32_t nxt_m = (uint32_t)__shfl((int)nxt, src_lane, 64);
      const bool keep = lane < n_run;
      req = keep ? req_m : -1;
      pos = keep ? pos_m : 0u;
      held = keep ? held_m : 0u;
      nxt = keep ? nxt_m : 0u;
    }
  }
  // the pages pushed above may be popped below, by other lanes: the stores must have completed
  drain_vmem();
  // ---- (2) arrivals enter, in order, while their pages are there
  const bool idle = mine && req < 0;
  const uint64_t idle_mask = __ballot(idle);
  const uint32_t n_idle = (uint32_t)__builtin_popcountll(idle_mask);
  uint32_t c_plen = 0, c_new = 0;   // lane i < 16: the request that is i-th in the queue
  if (lane < 16u && q_head + lane < q_tail && q_head + lane < sv.max_requests) {
    c_plen = ld_relaxed(sv.req_len + 2 * (size_t)(q_head + lane));
    c_new = ld_relaxed(sv.req_len + 2 * (size_t)(q_head + lane) + 1);
  }
  const uint32_t c_need = pages_of(c_plen, c_new);
  uint32_t n_admit = 0;
  for (uint32_t k = 0; k < n_idle; ++k) {
    if (q_head + k >= q_tail || q_head + k >= sv.max_requests) break;
    const uint32_t nd = (uint32_t)__builtin_amdgcn_readlane((int)c_need, (int)k);
    if (n_free - promised < nd) break;
    promised += nd;
    ++n_admit;
  }
  const uint32_t my_rank = (uint32_t)__builtin_popcountll(idle_mask & below) & 15u;
  const uint32_t got_need = (uint32_t)__shfl((int)c_need, (int)my_rank, 64);   // (all lanes take part)
  if (idle && my_rank < n_admit) {
    req = (int32_t)(q_head + my_rank);
    pos = 0;
    held = 0;
    need = got_need;
    nxt = ld_relaxed((const uint32_t*)sv.req_prompt + (size_t)req * sv.max_prompt);
    st_act_u32(sv.req_state + 2 * (size_t)req, 1u);
  }
  q_head += n_admit;
  // ---- (3) the iteration's metadata
  const bool act = mine && req >= 0;
  const bool drained = __ballot(act) == 0ull && q_head >= q_tail;   // nothing running, nothing queued
  const bool wants = act && (pos & ps_mask) == 0u;
  const uint64_t want_mask = __ballot(wants);
  if (wants) {
    const uint32_t idx = n_free - 1u - (uint32_t)__builtin_popcountll(want_mask & below);
    uint32_t pg = lane;   // (never taken: the admission rule keeps promised <= n_free)
    if (idx < n_pages) pg = ld_relaxed((const uint32_t*)sv.free_stack + idx);
    else report(a, DE_BAD_META, 0xFFFFFFFFu, idx);
    const uint32_t blk = pos >> shift;
    if (blk < sv.max_blocks) st_act_u32((uint32_t*)sv.table + (size_t)lane * sv.max_blocks + blk, pg);
    ++held;
  }
  const uint32_t n_popped = (uint32_t)__builtin_popcountll(want_mask);
  n_free -= n_popped;
  promised -= n_popped;
  if (mine) {
    st_act_u32((uint32_t*)sv.slot_req + lane, (uint32_t)req);
    st_act_u32((uint32_t*)sv.slot_pos + lane, act ? pos : 0u);
    st_act_u32((uint32_t*)sv.slot_held + lane, held);
    st_act_u32(tok_io + lane, act ? nxt : 0u);
    st_act_u32(pos_io + lane, act ? pos : 0u);
  }
  if (lane == 0) {
    st_act_u32(sv.scalars + kServeNFree, n_free);
    st_act_u32(sv.scalars + kServePromised, promised);
    st_act_u32(sv.scalars + kServeQHead, q_head);
    st_act_u32(sv.scalars + kServeIterations, ld_relaxed(sv.scalars + kServeIterations) + 1u);
    st_act_u32(sv.scalars + kServeTokens, ld_relaxed(sv.scalars + kServeTokens) + n_produced);
    st_act_u32(sv.scalars + kServeDone, ld_relaxed(sv.scalars + kServeDone) + n_done);
    // nothing running and nothing queued: this iteration is the launch's last (the step number
    // names the decision, so that no stale one is ever taken for it)
    if (drained) st_act_u32(sv.scalars + kServeStop, a.epoch);
  }
}

// NB, the batch class, pins the linear body of a kernel: a kernel that carries a single one keeps its
// register allocation (nearly) free of spills, one that decides between them at run time does not.
//   1: one row, vector body; 9: one row, large tasks: three weight buffers; 2: two rows, vector body;
//   11, 12: one and two rows, vector body, short weight rows packed (see LinGeom);
//   4, 8, 16: up to that many rows, matrix cores -- a kernel for each packing of the input terms (in one kernel
//   for all the three bodies had 398 to 431 spilled scalar registers)
template <int NB, bool MEGA, class Svc = NoJit>
__device__ __forceinline__ uint32_t run_linear(const TaskDesc& t, const StepArgs& a, float* lds, int32_t wait_ev,
                                           uint32_t* s_flag, const Svc& svc = Svc{}, uint32_t next_ti = 0) {
  if constexpr (NB == 4 || NB == 8 || NB == 16) return linear_task_mfma<NB == 4 ? 3 : NB == 8 ? 2 : 1, MEGA, Svc>(t, a, lds, wait_ev, s_flag, svc);
  else if constexpr (NB == 9) return linear_task<1, MEGA, Svc, true>(t, a, lds, wait_ev, s_flag, svc, next_ti);
  else if constexpr (NB == 11 || NB == 12) return linear_task<NB - 10, MEGA, Svc, false, true>(t, a, lds, wait_ev, s_flag, svc, next_ti);
  else return linear_task<NB, MEGA, Svc>(t, a, lds, wait_ev, s_flag, svc, next_ti);
}

// Runs one task that is neither a linear nor an attention nor an expert task.  wait_ev >= 0: the task must first
// wait for that event (persistent kernel).
// (Kernels for dense models are built without the mixture-of-experts bodies.)
template <bool MOE>
__device__ __forceinline__ bool run_task(const TaskDesc& t, const StepArgs& a, float* lds, int32_t wait_ev, uint32_t* s_flag) {
  if (wait_ev >= 0 && !wait_event(a, wait_ev, s_flag)) return false;
  trace_mark(a, t, 1);
  switch (t.kind) {
    case TK_EMBED: body_embed(t, a); break;
    case TK_RMSNORM: body_rmsnorm(t, lds); break;
    case TK_ROPE: body_rope(t, a); break;
    case TK_ATTN_MERGE: body_attn_merge(t, a); break;
    case TK_ADD: body_add(t); break;
    case TK_SWIGLU: body_swiglu(t); break;
    case TK_ARGMAX: body_argmax(t, a, lds); break;
    case TK_SERVE: body_serve(a); break;
    case TK_MOE_ROUTE: if (MOE) body_moe_route(t, lds); break;
    case TK_MOE_COMBINE: if (MOE) body_moe_combine(t, a); break;
    default: break;   // TK_DUMMY: no computation (normalization, Section 4.1)
  }
  return true;
}

// ------------------------------------------------------------------------------ runtime

// Has event e been activated for this step?  The whole wavefront calls it; the answer is uniform.
// Simple events: one counter, compared with epoch * required by lane 0.  Sharded events (all
// producers ahead-of-time): one counter per producer group (worker index mod kShards), each on its
// own 256-byte line; lanes 0 .. kShards-1 read one group's counter each -- a single load instruction
// -- and compare it with epoch * (that group's producers).  An arrival is then ONE atomic add that
// nobody waits for, and the producers spread over kShards lines (see kHierMinRequired).
__device__ __forceinline__ EventProbe probe_event(const StepArgs& a, int32_t e, int lane) {
  const MPK_CONST EventDesc& ev = *(const MPK_CONST EventDesc*)(a.events + e);
  EventProbe p;
  p.seen = p.need = 0;   // lanes without a counter agree
  if (ev.flags & EV_HIER) {
    if (lane < (int)kShards) {
      p.need = a.epoch * ((const MPK_CONST EventDesc*)(a.events + e))->sub_required[lane];
      p.seen = ld_relaxed(a.hier + (size_t)ev.hier_slot * kHierWordsPerEvent + (1 + lane) * kHierStrideWords);
    }
  } else if (lane == 0) {
    p.need = a.epoch * ev.required;
    p.seen = ld_relaxed(a.counters + e);
  }
  return p;
}
__device__ __forceinline__ bool probe_reached(const EventProbe& p) {
  return __builtin_amdgcn_readfirstlane((int)(__ballot((int32_t)(p.seen - p.need) >= 0) == ~0ull)) != 0;
}
__device__ __forceinline__ bool event_reached(const StepArgs& a, int32_t e, int lane) {
  return probe_reached(probe_event(a, e, lane));
}

// The first wavefront polls until event e is activated; *s_flag = 1, or 0 when the step is being
// aborted (watchdog or a peer's failure).  Called by all 64 lanes of the wavefront.
__device__ __forceinline__ void poll_event_wave0(const StepArgs& a, int32_t e, uint32_t* s_flag, int lane) {
  uint32_t ok = 1;
  if (!event_reached(a, e, lane)) {
    const uint64_t t_start = wall_clock64();
    uint32_t it = 0;
    while (!event_reached(a, e, lane)) {
      if ((++it & 255u) == 0) {
        uint32_t dead = 0;
        if (lane == 0) {
          if (ld_relaxed(a.g->err + 1) != 0) dead = 1;
          else if (wall_clock64() - t_start > a.g->timeout_ticks) {
            report(a, DE_TIMEOUT, (uint32_t)e, blockIdx.x);
            __hip_atomic_store(as_global(a.g->err + 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            dead = 1;
          }
        }
        if (__builtin_amdgcn_readfirstlane(dead)) { ok = 0; break; }
      }
    }
  }
  if (lane == 0) *s_flag = ok;
}

// Returns false when the step is being aborted (watchdog or a peer's failure).
__device__ __forceinline__ bool wait_event(const StepArgs& a, int32_t e, uint32_t* s_flag) {
  if (threadIdx.x < 64) poll_event_wave0(a, e, s_flag, (int)threadIdx.x);
  __syncthreads();   // later agent-scope loads cannot move above this barrier
  return __builtin_amdgcn_readfirstlane(*s_flag) != 0;
}

// The same behind an earlier look at the event (taken by all lanes of the first wavefront).
__device__ __forceinline__ bool wait_event(const StepArgs& a, int32_t e, uint32_t* s_flag, const EventProbe& probe) {
  if (threadIdx.x < 64) {
    if (!probe_reached(probe)) poll_event_wave0(a, e, s_flag, (int)threadIdx.x);
    else if (threadIdx.x == 0) *s_flag = 1;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(*s_flag) != 0;
}

// One lane: add this task's notification to event e (Section 5: "notify the triggering event").
// The arrival that activates an event whose range holds just-in-time tasks hands the event to
// its scheduler's queue.
__device__ __forceinline__ void notify_event(const StepArgs& a, int32_t e) {
  if ((a.flags & kLoseNotifyBit) && blockIdx.x == 0) return;   // MPK_DEBUG_LOSE_NOTIFY: the waiters' watchdog has to end the step
  const MPK_CONST EventDesc& ev = *(const MPK_CONST EventDesc*)(a.events + e);
  const uint32_t flags = ev.flags;
  bool activated = false;
  if (flags & EV_HIER) {
    uint32_t* blk = a.hier + (size_t)ev.hier_slot * kHierWordsPerEvent;
    const uint32_t grp = blockIdx.x % kShards;
    if ((flags & EV_JIT) && a.n_sched) {
      // a scheduler has to be told by the arrival that completes the event: the last arrival of a
      // producer group adds to the top counter, the last of those hands the event over
      uint32_t old = __hip_atomic_fetch_add(as_global(blk + (1 + grp) * kHierStrideWords), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (old + 1u == a.epoch * ev.sub_required[grp]) {
        old = __hip_atomic_fetch_add(as_global(blk), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        activated = old + 1u == a.epoch * ev.n_groups;
      }
    } else {
      __hip_atomic_fetch_add(as_global(blk + (1 + grp) * kHierStrideWords), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  } else if ((flags & EV_JIT) && a.n_sched) {
    const uint32_t old = __hip_atomic_fetch_add(as_global(a.counters + e), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    activated = old + 1u == a.epoch * ev.required;
  } else {
    __hip_atomic_fetch_add(as_global(a.counters + e), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (activated && (flags & EV_JIT) && a.n_sched) {
    const uint32_t sc = (uint32_t)e % a.n_sched;
    const uint32_t slot = __hip_atomic_fetch_add(as_global(a.g->evq_tail + sc * 64u), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(as_global(a.g->evq_buf + (size_t)sc * a.g->evq_cap + (slot & (a.g->evq_cap - 1u))),
                       ((uint64_t)(slot + 1u) << 32) | (uint32_t)e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// One lane: a task's notification.  Where the descriptor names the counter (a task with a worker of its own, no scheduler
// to tell), the event's record is not looked at: two dependent scalar reads less between the stores'
// acknowledgement and the notification.
__device__ __forceinline__ void notify_task(const StepArgs& a, const TaskDesc& t) {
  if (t.twin > 0 && !(t.flags & TF_OUT_MARKED)) {
    if ((a.flags & kLoseNotifyBit) && blockIdx.x == 0) return;
    __hip_atomic_fetch_add(as_global(a.hier + (uint32_t)t.twin - 1u), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    notify_event(a, t.trig_event);
  }
}

__device__ __forceinline__ void signal_event(const StepArgs& a, const TaskDesc& t) {
  // every wavefront waits until its own agent-scope stores have completed at the coherence point
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  drain_vmem();
  trace_mark(a, t, 6);
  __syncthreads();
  trace_mark(a, t, 7);
  if (threadIdx.x == 0) notify_task(a, t);
}

// Wavefront 0 only: like poll_event_wave0, but also watches the worker's just-in-time queue.
// s_flag[0] = 1 event activated, 0 abort, 2 a just-in-time task (index in s_flag[1]) is queued.
__device__ __forceinline__ void poll_event_or_jit_wave0(const StepArgs& a, int32_t e, uint32_t* s_flag, int lane, uint32_t jit_head) {
  const uint64_t* slot = a.g->wq_buf + (size_t)blockIdx.x * a.g->wq_cap + (jit_head & (a.g->wq_cap - 1u));
  const uint64_t t_start = wall_clock64();
  uint32_t ok, it = 0;
  while (true) {
    if (event_reached(a, e, lane)) { ok = 1; break; }
    uint32_t got = 0, dead = 0;
    if (lane == 0) {
      const uint64_t v = ld_relaxed64(slot);
      if ((uint32_t)(v >> 32) == jit_head + 1u) { s_flag[1] = (uint32_t)v; got = 1; }
      else if ((++it & 127u) == 0) {
        if (ld_relaxed(a.g->err + 1) != 0) dead = 1;
        else if (wall_clock64() - t_start > a.g->timeout_ticks) {
          report(a, DE_TIMEOUT, (uint32_t)e, blockIdx.x);
          __hip_atomic_store(as_global(a.g->err + 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          dead = 1;
        }
      }
    }
    if (__builtin_amdgcn_readfirstlane(got)) { ok = 2; break; }
    if (__builtin_amdgcn_readfirstlane(dead)) { ok = 0; break; }
  }
  if (lane == 0) s_flag[0] = ok;
}

// Wavefront 0 only, after a workgroup barrier: wait for this wavefront's own coherent stores,
// then notify the event.
__device__ __forceinline__ void signal_from_wave0(const StepArgs& a, const TaskDesc& t, int lane) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  drain_vmem();
  trace_mark(a, t, 7);
  if (lane == 0) notify_task(a, t);
}

// The first 192 bytes of the dynamic LDS are control words ([0] = result of the last event wait;
// from word 16: the kernel's arguments); task bodies use the rest.
// The arguments are kept there for the task functions that are real calls: a struct passed by
// value to such a function travels through private memory -- every one of the 512 lanes stores
// and re-loads its own 80-byte copy, 10 MB per call over the chip and a memory round trip before
// the task can start, and every call site gets a private copy of its own that crowds the weight
// buffers out of the registers (vector body: 55 spilled registers by value, none this way).
constexpr uint32_t kLdsArgsAt = 16;
static_assert(kLdsArgsAt * 4 + sizeof(StepArgs) <= kLdsCtrlFloats * 4, "control words too small for the arguments");
// Thread 0 leaves the arguments in LDS; the callers' next barrier publishes them.
__device__ __forceinline__ void publish_args(const StepArgs& a) {
  extern __shared__ __align__(16) float dyn_lds[];
  if (threadIdx.x == 0) {
    *(StepArgs*)(dyn_lds + kLdsArgsAt) = a;
    ((uint32_t*)dyn_lds)[kLdsAbortAt] = 0u;
  }
}
__device__ __forceinline__ StepArgs published_args() {
  extern __shared__ __align__(16) float dyn_lds[];
  return uniform_args(*(const StepArgs*)(dyn_lds + kLdsArgsAt));
}

// An expert task.  Inlined into the all-ahead-of-time walk from batch 3 on, which has nothing live across it: as a
// real function it saves 89 registers a lane on entry and restores them on exit, 0.2 MB a worker and call (a quarter
// of the expert stages' traffic at batch 16; us a step of the mixture-of-experts layers: batch 16 1525 -> 1430,
// 8 1115 -> 1047, 4 825 -> 769).  The other kernels call it (run_expert_task), as do the sets of one and two rows, whose
// vector body would spill 28 to 40 registers beside it; called directly and not from within run_other_task, with one
// packing and one call site, batch 1 899 -> 843.
template <int NB, bool MEGA>
__device__ __forceinline__ bool expert_task(const StepArgs& a, const TaskDesc& t, uint32_t task_index, bool skip_wait, float* lds, uint32_t* s_flag) {
  int32_t wait_ev = -1;
  bool own_route = false;
  if (MEGA) {
    debug_jitter(a, task_index);
    wait_ev = (!skip_wait && t.dep_event >= 0 && ((const MPK_CONST EventDesc*)(a.events + t.dep_event))->required != 0) ? t.dep_event : -1;
    trace_mark(a, t, 0);
    if ((a.flags & kTraceBit) && threadIdx.x == 0) as_global(a.g->trace)[(size_t)task_index * kTraceSlots + 5] = blockIdx.x;
    // Cross-task pre-loading (Section 5.3) for the experts' second stage: which experts are active
    // is known since the routing task, long before the first stage has produced this task's
    // inputs.  Such a task (the compiler leaves the routing task's event number + 1 in aux1)
    // waits for that event -- activated early in the first stage, so this returns at
    // once and only orders the reads of the meta-tensor -- finds its first job and requests that
    // job's first weights, and only then waits for its own event.
    // A first-stage task with a number in aux1 (the event that the routing task waits for, + 1) waits for that one instead of its
    // own and works the routing out by itself: see kMoeOwnRouteExperts.
    const bool early = wait_ev >= 0 && t.aux1 != nullptr, first = t.flags & TF_GATEUP;
    if (early && !wait_event(a, (int32_t)(uintptr_t)t.aux1 - 1, s_flag)) return false;
    own_route = early && first;
    if (own_route) wait_ev = -1;
    if (wait_ev >= 0 && !(early && !(a.flags & kNoPreloadBit))) {
      if (!wait_event(a, wait_ev, s_flag)) return false;
      wait_ev = -1;
    }
    if (wait_ev < 0) trace_mark(a, t, 1);
  }
  if (!body_moe_expert<NB>(t, a, lds, wait_ev, s_flag, own_route)) return false;
  if (MEGA) {
    trace_mark(a, t, 3);
    if (t.trig_event >= 0) signal_event(a, t);
    else __syncthreads();
    trace_mark(a, t, 4);
  }
  return true;
}

template <int NB, bool MEGA>
__device__ __noinline__ bool run_expert_task(uint32_t task_index, bool skip_wait) {
  const StepArgs a = published_args();
  task_index = uniform_u32(task_index);
  extern __shared__ __align__(16) float dyn_lds[];
  return expert_task<NB, MEGA>(a, ld_task(a, task_index), task_index, uniform_u32(skip_wait) != 0, dyn_lds + kLdsCtrlFloats, (uint32_t*)dyn_lds);
}

// Everything that is not a linear task runs in a function of its own (a real call): its
// thread-index arithmetic and temporaries then get their own register allocation instead of being
// hoisted to the top of the persistent loop, where they would crowd out the weight ring and
// force spills of registers that have loads in flight.
// Returns false when the step is being aborted.
template <bool MEGA, bool MOE>
__device__ __noinline__ bool run_other_task(uint32_t task_index, bool skip_wait) {
  const StepArgs a = published_args();
  task_index = uniform_u32(task_index);
  skip_wait = uniform_u32(skip_wait) != 0;
  extern __shared__ __align__(16) float dyn_lds[];
  float* lds = dyn_lds + kLdsCtrlFloats;
  uint32_t* s_flag = (uint32_t*)dyn_lds;
  const TaskDesc t = ld_task(a, task_index);
  int32_t wait_ev = -1;
  if (MEGA) {
    debug_jitter(a, task_index);
    wait_ev = (!skip_wait && t.dep_event >= 0 && ((const MPK_CONST EventDesc*)(a.events + t.dep_event))->required != 0) ? t.dep_event : -1;
    trace_mark(a, t, 0);
    if ((a.flags & kTraceBit) && threadIdx.x == 0) as_global(a.g->trace)[(size_t)task_index * kTraceSlots + 5] = blockIdx.x;
  }
  if (!run_task<MOE>(t, a, lds, wait_ev, s_flag)) return false;
  if (MEGA) {
    trace_mark(a, t, 3);
    if (t.trig_event >= 0) signal_event(a, t);
    else __syncthreads();
    trace_mark(a, t, 4);
  }
  return true;
}

// An attention task, one real function per (head_dim, query heads per KV head, kind of cache): the
// matrix-core body wants its own register allocation, and every batch class gets every shape this
// way (with the shapes pinned per kernel, a model without a kernel set of its own ran on a fallback
// that decided everything at run time and spilled 350 registers: head size 64 at batch 1, every
// model at batch 2 to 4).  skip_wait: the event is known to be active; signal: notify the
// triggering event (persistent kernel).
template <int D, int GRP, bool PAGED, bool MARKED>
__device__ __noinline__ bool run_attn_task(uint32_t task_index, bool skip_wait, bool signal) {
  const StepArgs a = published_args();
  task_index = uniform_u32(task_index);
  skip_wait = uniform_u32(skip_wait) != 0;
  signal = uniform_u32(signal) != 0;
  extern __shared__ __align__(16) float dyn_lds[];
  float* lds = dyn_lds + kLdsCtrlFloats;
  uint32_t* s_flag = (uint32_t*)dyn_lds;
  const TaskDesc t = ld_task(a, task_index);
  int32_t wait_ev = -1;
  if (signal) {
    debug_jitter(a, task_index);
    wait_ev = (!MARKED && !skip_wait && t.dep_event >= 0 && ((const MPK_CONST EventDesc*)(a.events + t.dep_event))->required != 0) ? t.dep_event : -1;
    trace_mark(a, t, 0);
    if ((a.flags & kTraceBit) && threadIdx.x == 0) as_global(a.g->trace)[(size_t)task_index * kTraceSlots + 5] = blockIdx.x;
  }
  if (!body_attn_mfma<D, GRP, PAGED, MARKED>(t, a, lds, wait_ev, s_flag)) return false;
  if (signal) {
    trace_mark(a, t, 3);
    if (t.trig_event >= 0) signal_event(a, t);
    else lds_barrier();
    trace_mark(a, t, 4);
  }
  return true;
}
// Runs a task that is not a linear task.  (A callee's result comes back in a vector register: it is
// made scalar again, or the whole task loop, and every descriptor load in it, turns into per-lane code.)
template <bool MARKED>
__device__ __forceinline__ bool call_attn_task(const StepArgs& a, uint32_t task_index, bool skip_wait, bool signal) {
  switch (a.g->attn_shape) {   // see attn_shape_index
#define MPK_ATTN_CASE(D, LG)                                                                                                   \
    case attn_shape_index(D, 1u << LG, 0): return run_attn_task<D, (1 << LG), false, MARKED>(task_index, skip_wait, signal); \
    case attn_shape_index(D, 1u << LG, 1): return run_attn_task<D, (1 << LG), true, MARKED>(task_index, skip_wait, signal);
    MPK_ATTN_CASE(64, 0) MPK_ATTN_CASE(64, 1) MPK_ATTN_CASE(64, 2) MPK_ATTN_CASE(64, 3)
    MPK_ATTN_CASE(128, 0) MPK_ATTN_CASE(128, 1) MPK_ATTN_CASE(128, 2) MPK_ATTN_CASE(128, 3)
#undef MPK_ATTN_CASE
    default: return false;   // (the host admits no other shape)
  }
}
// MARKS: the kernel runs marked descriptors (an attention task has both its input and its output marked, or neither).
template <int NB, bool MEGA, bool MOE, bool MARKS = false>
__device__ __forceinline__ bool call_task(const StepArgs& a, uint16_t kind, uint16_t flags, uint32_t task_index, bool skip_wait) {
  bool ok;
  if (MOE && kind == TK_MOE_EXPERT) ok = run_expert_task<NB == 9 ? 1 : NB, MEGA>(task_index, skip_wait);
  else if (kind != TK_ATTN_PARTIAL) ok = run_other_task<MEGA, MOE>(task_index, skip_wait);
  else if (MARKS && (flags & TF_IN_MARKED)) ok = call_attn_task<true>(a, task_index, skip_wait, MEGA);
  else ok = call_attn_task<false>(a, task_index, skip_wait, MEGA);
  return __builtin_amdgcn_readfirstlane((int)ok) != 0;
}

__device__ __forceinline__ bool event_active(const StepArgs& a, int32_t e) {
  const MPK_CONST EventDesc& ev = *(const MPK_CONST EventDesc*)(a.events + e);
  if (ev.required == 0) return true;
  if (ev.flags & EV_HIER) {   // (one lane: the group counters one after the other, all in flight together)
    const uint32_t* blk = a.hier + (size_t)ev.hier_slot * kHierWordsPerEvent;
    uint32_t v[kShards];
#pragma unroll
    for (uint32_t k = 0; k < kShards; ++k) v[k] = ld_relaxed(blk + (1 + k) * kHierStrideWords);
    bool ok = true;
#pragma unroll
    for (uint32_t k = 0; k < kShards; ++k) ok = ok && (int32_t)(v[k] - a.epoch * ev.sub_required[k]) >= 0;
    return ok;
  }
  return (int32_t)(ld_relaxed(a.counters + e) - a.epoch * ev.required) >= 0;
}


// One scheduler wavefront (Section 5.1): takes activated events from its own queue and hands the
// just-in-time tasks of each event's range to the workers' queues, round-robin from a cursor of
// its own -- local state only, no coordination with other schedulers (Section 6.1).
__device__ __forceinline__ void scheduler_wave(const StepArgs& a, uint32_t sc) {
  const int lane = threadIdx.x & 63;
  const uint32_t W = a.g->n_workers;
  uint32_t head = ld_relaxed(a.g->sched_state + sc * 64u), cursor = ld_relaxed(a.g->sched_state + sc * 64u + 1u);
  uint32_t todo = ld_u32c(a.g->sched_nev + sc);
  // schedulers that hand out the same number of tasks per layer move their cursors in lock-step:
  // start them evenly spread over the workers, or they would all pile onto the same few
  const uint32_t spread = sc * (W / a.n_sched);
  // the start event has no notifications: its owner dispatches it unprompted
  const MPK_CONST EventDesc& sev = *(const MPK_CONST EventDesc*)(a.events + a.g->start_event);
  bool pending_start = (sev.flags & EV_JIT) && a.g->start_event % a.n_sched == sc;
  while (todo > 0 || pending_start) {
    uint32_t e;
    if (pending_start) {
      e = a.g->start_event;
      pending_start = false;
    } else {
      const uint64_t* slot = a.g->evq_buf + (size_t)sc * a.g->evq_cap + (head & (a.g->evq_cap - 1u));
      uint64_t v = ld_relaxed64(slot);
      if ((uint32_t)(v >> 32) != head + 1u) {
        const uint64_t t_start = wall_clock64();
        uint32_t it = 0;
        bool dead = false;
        while ((uint32_t)((v = ld_relaxed64(slot)) >> 32) != head + 1u) {
          if ((++it & 255u) == 0) {
            if (ld_relaxed(a.g->err + 1) != 0) { dead = true; break; }
            if (wall_clock64() - t_start > a.g->timeout_ticks) {
              if (lane == 0) {
                report(a, DE_TIMEOUT, 0x80000000u | sc, blockIdx.x);
                __hip_atomic_store(as_global(a.g->err + 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              }
              dead = true;
              break;
            }
          }
        }
        if (dead) break;
      }
      e = (uint32_t)v;
      ++head;
      --todo;
    }
    const MPK_CONST EventDesc& ev = *(const MPK_CONST EventDesc*)(a.events + e);
    const uint32_t first = ev.first, n = ev.last - ev.first;
    for (uint32_t i = lane; i < n; i += 64) {
      const uint32_t ti = first + i;
      const MPK_CONST TaskDesc& td = *(const MPK_CONST TaskDesc*)(a.tasks + ti);
      if (td.flags & TF_JIT) {
        const uint32_t w = (cursor + spread + i) % W;
        const uint32_t s = __hip_atomic_fetch_add(as_global(a.g->wq_tail + w * 64u), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(as_global(a.g->wq_buf + (size_t)w * a.g->wq_cap + (s & (a.g->wq_cap - 1u))),
                           ((uint64_t)(s + 1u) << 32) | ti, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    cursor += n;
  }
  if (lane == 0) {
    __hip_atomic_store(as_global(a.g->sched_state + sc * 64u), head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(as_global(a.g->sched_state + sc * 64u + 1u), cursor % W, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

constexpr uint32_t kPickExit = 0xFFFFFFFFu, kPickAbort = 0xFFFFFFFEu;

// Worker side of the hybrid launch (Section 5.2): just-in-time tasks first; when none is queued,
// the head of the ahead-of-time queue if its dependent event is activated (or, for a linear task,
// regardless: see linear_wait); exit once the
// ahead-of-time queue is exhausted and the terminal event has been activated.  One lane decides,
// the result goes through LDS.  Returns a task index (bit 31 set: it came from the JIT queue).
__device__ __forceinline__ uint32_t pick_task(const StepArgs& a, uint32_t* ctrl, uint32_t* jit_head, uint32_t* ai, uint32_t q1) {
  if (threadIdx.x == 0) {
    const uint32_t w = blockIdx.x;
    uint32_t pick;
    const uint64_t t_start = wall_clock64();
    uint32_t it = 0;
    while (true) {
      const uint64_t v = ld_relaxed64(a.g->wq_buf + (size_t)w * a.g->wq_cap + (*jit_head & (a.g->wq_cap - 1u)));
      if ((uint32_t)(v >> 32) == *jit_head + 1u) {
        pick = (uint32_t)v | 0x80000000u;
        ++*jit_head;
        break;
      }
      if (*ai < q1) {
        const uint32_t ti = ld_u32c(a.g->aot + *ai);
        const MPK_CONST TaskDesc* td = (const MPK_CONST TaskDesc*)(a.tasks + ti);
        const int32_t dep = td->dep_event;
        // a linear task may start before its event: it requests its weights, then waits for the
        // event itself while serving this worker's just-in-time queue (linear_wait)
        if (dep < 0 || td->kind == TK_LINEAR || event_active(a, dep)) {
          pick = ti;
          ++*ai;
          break;
        }
      } else if (event_active(a, (int32_t)a.g->terminal_event)) {
        pick = kPickExit;
        break;
      }
      if ((++it & 63u) == 0) {
        if (ld_relaxed(a.g->err + 1) != 0) { pick = kPickAbort; break; }
        if (wall_clock64() - t_start > a.g->timeout_ticks) {
          report(a, DE_TIMEOUT, 0x40000000u | (*ai < q1 ? ld_u32c(a.g->aot + *ai) : 0u), blockIdx.x);
          __hip_atomic_store(as_global(a.g->err + 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          pick = kPickAbort;
          break;
        }
      }
    }
    ctrl[1] = pick;
    ctrl[2] = *jit_head;
    ctrl[3] = *ai;
  }
  __syncthreads();
  *jit_head = __builtin_amdgcn_readfirstlane(ctrl[2]);
  *ai = __builtin_amdgcn_readfirstlane(ctrl[3]);
  const uint32_t pick = __builtin_amdgcn_readfirstlane(ctrl[1]);
  __syncthreads();   // ctrl may be rewritten only after everybody has read it
  return pick;
}

// Batch classes whose kernels run marked descriptors.
constexpr bool has_marks(int nb) { return nb == 1 || nb == 2 || nb == 9 || nb == 11 || nb == 12; }

// Every task ahead-of-time: the worker walks its pre-enqueued list, each task waits for its own
// event.  after_first_step: a task without producers (an embedding task) first waits for the
// previous step's terminal event, i.e. for that step's sampling tasks.  Returns false on abort.
template <int NB, bool MOE, bool MARKS, bool SINGLE>
__device__ __forceinline__ bool aot_pass(const StepArgs& a, uint32_t q0, uint32_t q1, float* lds, uint32_t* s_flag,
                                         bool after_first_step) {
  for (uint32_t qi = q0; qi < q1; ++qi) {
    const uint32_t ti = ld_u32c(a.g->aot + qi);
    const TaskDesc t = ld_task(a, ti);
    if (after_first_step && t.dep_event == (int32_t)a.g->start_event) {
      StepArgs prev = a;
      prev.epoch = a.epoch - 1u;
      if (!__builtin_amdgcn_readfirstlane((int)wait_event(prev, (int32_t)a.g->terminal_event, s_flag))) return false;
    }
    if (t.kind == TK_LINEAR) {
      debug_jitter(a, ti);
      const int32_t wait_ev = (!(MARKS && (t.flags & TF_IN_MARKED)) && t.dep_event >= 0 && ((const MPK_CONST EventDesc*)(a.events + t.dep_event))->required != 0) ? t.dep_event : -1;
      trace_mark(a, t, 0);
      if ((a.flags & kTraceBit) && threadIdx.x == 0) as_global(a.g->trace)[(size_t)t.index * kTraceSlots + 5] = blockIdx.x;
      // (the next task of this worker: a flagged task pre-loads its first half blocks into LDS pages)
      std::conditional_t<MARKS, NoJitMarks, NoJit> svc;
      svc.n_next = min(q1 - qi - 1u, 2u);
      if (svc.n_next > 0) svc.next[0] = ld_u32c(a.g->aot + qi + 1);
      if (svc.n_next > 1) svc.next[1] = ld_u32c(a.g->aot + qi + 2);
      if (!run_linear<NB, true>(t, a, lds, wait_ev, s_flag, svc, svc.next[0])) {
        if (MARKS && mark_aborted()) mark_report((uint32_t)t.dep_event);
        return false;
      }
    } else if (MOE && SINGLE && !has_marks(NB) && t.kind == TK_MOE_EXPERT) {
      if (!expert_task<NB == 9 ? 1 : NB, true>(a, t, ti, false, lds, s_flag)) return false;
    } else {
      if (!call_task<NB, true, MOE, MARKS>(a, t.kind, t.flags, ti, false)) return false;
    }
  }
  return true;
}

// Serving launches end when the server has drained (Section 5: the kernel runs until the workload
// is done).  The serving task that finds nothing running and nothing queued records its step
// number; steps after that one are not run, but they must still count for the events -- the host
// has advanced the step number for all of them, and events compare counters with step x producers
// -- so every worker adds the notifications of its own tasks, `steps` times each, and leaves.
__device__ __noinline__ void serve_skip_steps(StepArgs a_in, uint32_t q0, uint32_t q1, uint32_t steps) {
  const StepArgs a = uniform_args(a_in);
  q0 = uniform_u32(q0); q1 = uniform_u32(q1); steps = uniform_u32(steps);
  for (uint32_t qi = q0 + threadIdx.x; qi < q1; qi += kThreads) {
    const int32_t e = ((const MPK_CONST TaskDesc*)(a.tasks + ld_u32c(a.g->aot + qi)))->trig_event;
    if (e < 0) continue;
    const MPK_CONST EventDesc& ev = *(const MPK_CONST EventDesc*)(a.events + e);
    uint32_t* cnt = (ev.flags & EV_HIER) ? a.hier + (size_t)ev.hier_slot * kHierWordsPerEvent + (1u + blockIdx.x % kShards) * kHierStrideWords
                                         : a.counters + e;
    __hip_atomic_fetch_add(as_global(cnt), steps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
// Did an earlier step of this run (steps a.epoch - a.step .. a.epoch - 1) find the server drained?
__device__ __forceinline__ bool serve_drained(const StepArgs& a) {
  const uint32_t stop = __builtin_amdgcn_readfirstlane(ld_relaxed(a.g->serve->scalars + kServeStop));
  return stop - (a.epoch - (uint32_t)a.step) < (uint32_t)a.step;
}

// A launch that is one step of a run: true when an earlier step of the run left the server
// drained -- this step's share of the event counters has then been settled and the kernel leaves.
// (A real call, so that the kernel around it keeps the code it has without it.)
__device__ __noinline__ bool serve_step_gate(StepArgs a_in, uint32_t q0, uint32_t q1) {
  const StepArgs a = uniform_args(a_in);
  if (!(a.flags & kServeBit) || a.step == 0 || !serve_drained(a)) return false;
  serve_skip_steps(a, q0, q1, 1u);
  // The marked copy that the drained step wrote is put back to unset by the first step behind it, as that
  // step's tasks would have done; the other copy the drained step's tasks have put back.
  const uint32_t stop = __builtin_amdgcn_readfirstlane(ld_relaxed(a.g->serve->scalars + kServeStop));
  if (a.g->mark_words && a.epoch - stop == 1u) {
    float* copy = a.g->mark_base + (size_t)(stop & 1u) * a.g->mark_words;
    for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < a.g->mark_words; i += gridDim.x * kThreads) st_act_u32((uint32_t*)(copy + i), kUnsetWord);
    const uint32_t n = a.g->batch * a.g->head_dim;
    for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) st_act_u32((uint32_t*)(a.g->rope_tab + (stop & 1u) * n + i), kUnsetWord);
  }
  return true;
}

// Multi-token launch (graphs with the sampling operator, no schedulers): the task list is walked
// n_steps times, the epoch -- hence every counter target -- growing by one each time.  A kernel of
// its own: with the step loop in mpk_mega_kernel the single-step launch measured 2 to 4 % slower.
template <int NB, bool MOE>
__global__ void __launch_bounds__(kThreads) mpk_loop_kernel(StepArgs a) {
  extern __shared__ __align__(16) float dyn_lds[];
  float* lds = dyn_lds + kLdsCtrlFloats;
  uint32_t* s_flag = (uint32_t*)dyn_lds;
  const uint32_t w = blockIdx.x;
  const uint32_t q0 = ld_u32c(a.g->aot_off + w), q1 = ld_u32c(a.g->aot_off + w + 1);
  const uint32_t n_steps = a.n_steps;
  for (uint32_t step = 0; step < n_steps; ++step, ++a.epoch) {
    a.step = (uint16_t)step;
    if (step > 0 && (a.flags & kServeBit) && serve_drained(a)) {
      // The previous step's serving task found the server drained; every worker has since run a
      // task downstream of it, so all of them read the same decision here.  The counters move only
      // after that step has ended altogether (its terminal event), or one would pass the target
      // that one of its tasks is still waiting for.
      StepArgs prev = a;
      prev.epoch = a.epoch - 1u;
      if (!wait_event(prev, (int32_t)a.g->terminal_event, s_flag)) return;
      serve_skip_steps(a, q0, q1, n_steps - step);
      return;
    }
    __syncthreads();   // (nobody is inside a task function any more)
    publish_args(a);
    __syncthreads();
    if (!aot_pass<NB, MOE, false, false>(a, q0, q1, lds, s_flag, step > 0)) return;
  }
}

// HYBRID: the hybrid launch (scheduler workgroups); otherwise the all-ahead-of-time walk.  Two kernels:
// in one that holds both, the hybrid walk's spilled registers (two rows 164 against none, three buffers 175
// against 26) are the other's too, and a reload from scratch memory waits for every weight load in flight.
// RUN: the instance launched once per step for a run of several steps (vector linear bodies): it
// can find that an earlier step of the run left the server drained.  A kernel of its own, so that
// the single-step kernel stays exactly as it is (1.2 % slower with the check compiled in).
template <int NB, bool MOE, bool HYBRID, bool RUN = false>
__global__ void __launch_bounds__(kThreads) mpk_mega_kernel(StepArgs a) {
  extern __shared__ __align__(16) float dyn_lds[];
  float* lds = dyn_lds + kLdsCtrlFloats;
  uint32_t* s_flag = (uint32_t*)dyn_lds;
  const uint32_t w = blockIdx.x;
  publish_args(a);
  __syncthreads();
  if (HYBRID && w >= a.g->n_workers) {
    // scheduler workgroup: 4 scheduler wavefronts (Section 5.1, Table 2), the rest leave
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t sc = (w - a.g->n_workers) * 4u + wave;
    if (wave < 4u && sc < a.n_sched) scheduler_wave(a, sc);
    return;
  }
  const uint32_t q0 = ld_u32c(a.g->aot_off + w), q1 = ld_u32c(a.g->aot_off + w + 1);
  if constexpr (!HYBRID) {
    // (a run of serving iterations issued as one launch per step: the launches behind the one
    // that found the server drained only settle their share of the event counters)
    if (RUN && __builtin_amdgcn_readfirstlane((int)serve_step_gate(a, q0, q1))) return;
    aot_pass<NB, MOE, has_marks(NB), true>(a, q0, q1, lds, s_flag, false);
    return;
  }
  if constexpr (HYBRID) {
    uint32_t jit_head = ld_relaxed(a.g->wq_head + w), ai = q0;
    while (true) {
      const uint32_t pick = pick_task(a, (uint32_t*)dyn_lds, &jit_head, &ai, q1);
      if (pick == kPickExit || pick == kPickAbort) break;
      const uint32_t ti = pick & 0x7FFFFFFFu;
      const TaskDesc t = ld_task(a, ti);
      if (t.kind == TK_LINEAR) {
        debug_jitter(a, ti);
        trace_mark(a, t, 0);
        if ((a.flags & kTraceBit) && threadIdx.x == 0) as_global(a.g->trace)[(size_t)t.index * kTraceSlots + 5] = blockIdx.x;
        const int32_t wait_ev = (t.dep_event >= 0 && ((const MPK_CONST EventDesc*)(a.events + t.dep_event))->required != 0) ? t.dep_event : -1;
        uint32_t r;
        // started before its event is activated; a just-in-time task that arrives first pre-empts it
        while ((r = run_linear<NB, true>(t, a, lds, wait_ev, s_flag, JitWatch{jit_head})) == kLinPreempted) {
          const uint32_t tj = __builtin_amdgcn_readfirstlane(((uint32_t*)dyn_lds)[1]);
          lds_barrier();   // everybody has read the control word
          ++jit_head;
          // (a just-in-time task may itself be a linear task -- an operator whose tiles read only part
          // of a just-in-time operator's output is labelled just-in-time too, Section 5.2: its event
          // has been activated, so it runs without waiting and without watching the queue)
          const TaskDesc tjd = ld_task(a, tj);
          if (tjd.kind == TK_LINEAR) {
            debug_jitter(a, tj);
            if (run_linear<NB, true>(tjd, a, lds, -1, s_flag) != kLinDone) { r = kLinAbort; break; }
          } else if (!call_task<NB, true, MOE>(a, tjd.kind, tjd.flags, tj, true)) { r = kLinAbort; break; }
        }
        if (r == kLinAbort) break;
      } else {
        if (!call_task<NB, true, MOE>(a, t.kind, t.flags, ti, true)) break;
      }
    }
    if (threadIdx.x == 0) __hip_atomic_store(as_global(a.g->wq_head + w), jit_head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Kernel-per-operator baseline: the same task bodies, one launch per operator, dependencies
// enforced by stream order (what the paper's comparison systems do, Section 6.5).
template <int NB, bool MOE>
__global__ void __launch_bounds__(kThreads) mpk_op_kernel(StepArgs a, uint32_t first) {
  extern __shared__ __align__(16) float dyn_lds[];
  float* lds = dyn_lds + kLdsCtrlFloats;
  publish_args(a);
  __syncthreads();
  const uint32_t ti = ld_u32c(a.g->op_list + first + blockIdx.x);
  const TaskDesc t = ld_task(a, ti);
  if (t.kind == TK_LINEAR) {
    run_linear<NB, false>(t, a, lds, -1, nullptr);
  } else {
    call_task<NB, false, MOE>(a, t.kind, t.flags, ti, true);
  }
}


// One set of kernels per batch class (see run_linear) and per presence of the mixture-of-experts task
// kinds; every set takes every attention shape.
struct KernelVariant {
  int nb;
  bool moe;
  void (*mega)(StepArgs);     // all tasks ahead-of-time
  void (*op)(StepArgs, uint32_t);
  void (*loop)(StepArgs);
  void (*hybrid)(StepArgs);   // with scheduler workgroups
  void (*run_step)(StepArgs); // one step of a run of several, a launch per step
};
// index, batch class, mixture of experts, optimisation level, vector registers that a kernel may spill, that its hybrid walk may
// (build.py reads the last three).
//
// Level.  Kernel sets are compiled for size.  Two compute units share 64 KB of instructions, and a layer of a mixture of experts
// walks through more than that: its instruction cache misses 1300 times a layer at batch 1, 5400 at batch 16 (of some 3500 lines
// that a dense layer is made of and that stay), each a trip to the L2 for a whole workgroup.  us a step, -O3 / -Os: mixture of
// experts at batch 1 688 / 667, batch 16 1396 / 1378; dense sets, which fit, 0 to 2 % (tiny model 34.6 / 34.1, 8B 2690 / 2680, 8B
// layers at batch 8 1002 / 997, 2B class at batch 2, four tokens 2039 / 2027).  Not the set of one packed row (1B class 619 both,
// shorter rows +0.6 %).
//
// Spills.  What the sets have, the same at both levels; the build fails above it.  A reload from scratch memory waits for every weight
// load in flight, so the matrix-core bodies must have none; and a set of theirs that did (-Oz: 86 in the walk of batch 16 with
// experts) gave NaN for experts of more than 8 rows, for a reason that reading its code has not shown.
#define MPK_VARIANT_LIST(X) \
  X(0, 1, false, Os, 0, 0) X(1, 9, false, Os, 12, 40) X(2, 2, false, Os, 4, 34) \
  X(3, 4, false, Os, 0, 0) X(4, 8, false, Os, 0, 0) X(5, 16, false, Os, 0, 0) \
  X(6, 1, true, Os, 0, 0) X(7, 2, true, Os, 4, 34) \
  X(8, 4, true, Os, 0, 0) X(9, 8, true, Os, 0, 0) X(10, 16, true, Os, 0, 0) \
  X(11, 11, false, O3, 0, 0) X(12, 12, false, Os, 3, 34)
#define MPK_COUNT_VARIANT(...) + 1
constexpr int kNumVariants = 0 MPK_VARIANT_LIST(MPK_COUNT_VARIANT);
#undef MPK_COUNT_VARIANT
#define MPK_DECLARE_VARIANT(I, ...) const KernelVariant* kernel_variant_##I();
MPK_VARIANT_LIST(MPK_DECLARE_VARIANT)
#undef MPK_DECLARE_VARIANT

}  // namespace mpk

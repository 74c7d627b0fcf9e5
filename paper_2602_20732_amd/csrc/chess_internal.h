// Internal declarations shared by the HIP translation units of libchess (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/chess.h"
#include "../../include/chess_debug.h"

namespace chess {

constexpr int kHeadDim = 128;        // d
constexpr int kWave = 64;            // CDNA wavefront
constexpr int kMaxGroup = 16;        // q heads per KV head: one MFMA N-tile
constexpr int kTileTokens = 32;      // tokens per decode tile = K extent of one 16x16x32 MFMA

// Geometry every kernel needs, passed by value.
struct Geom {
    int32_t n_q_heads, n_kv_heads, group;
    int32_t page_size;               // B
    int32_t n_c, n_g;                // pages per chunk, chunks per grid
    int32_t max_pages, max_chunks, max_grids;   // row strides of block table / summary arrays
    int32_t max_sel;                 // row stride of page_ids
    uint32_t inv_nc, inv_ng;         // ceil(2^31 / n_c), ceil(2^31 / n_g): divisions by n_c / n_g as a multiply-high (div_by)
};

enum Schedule : int32_t { kLazy = 0, kMerged = 1, kEager = 2 };
enum ClusterMode : int { kSolo = 0, kCluster = 1, kEagerCluster = 2 };   // which code a selection kernel has (select_device.h)

struct SelectParams {
    int32_t plan, sink, window, budget_pages, budget_bp, over_chunk, over_grid, rho_g_bp, rho_c_bp, rho_p_bp;
    int32_t cap2, cap3;              // most candidate slots level 2 / level 3 can have (host bound)
    int32_t cap_keys, cap_kg, cap_kc;   // LDS capacities: keys of one level, kept grids, kept chunks
    int32_t probe;                   // CHESS_PROBE_*
    int32_t poll_limit;              // polls before a wait for published keys is given up
    int32_t general_cut;             // test hook: every level takes the general (LDS radix) cut
    int32_t local_grids;             // every member scores all grids itself (no exchange at the grid level)
    int32_t schedule;                // which units are scored together (select_device.h)
    uint32_t inv_members, inv_others;   // of the members of a cluster, of all but one of them (div_by; 0 for none)
    int32_t deciders;                // members that run the cuts; under the eager schedule the others only score
    int32_t keep_ties;               // the threshold rule: a level keeps every unit that ties with its k-th
    const int32_t* budget_per_seq;   // device [batch] or null: a value > 0 is that sequence's page budget
};

// A kernel argument as a register of its own.  Arguments arrive in groups of up to sixteen scalar registers, and a kernel
// that runs out of those saves and restores whole groups, sixteen lane reads for one value (step_kernel executed more of
// these than of anything else); a value that has been through here is saved and restored alone.
template <class V>
__device__ __forceinline__ V own_reg(V v)
{
    asm("" : "+s"(v));
    return v;
}
__device__ __forceinline__ Geom own_regs(const Geom& g)
{
    return Geom{own_reg(g.n_q_heads), own_reg(g.n_kv_heads), own_reg(g.group), own_reg(g.page_size), own_reg(g.n_c), own_reg(g.n_g),
                own_reg(g.max_pages), own_reg(g.max_chunks), own_reg(g.max_grids), own_reg(g.max_sel), own_reg(g.inv_nc), own_reg(g.inv_ng)};
}
__device__ __forceinline__ SelectParams own_regs(const SelectParams& p)
{
    SelectParams r;
    r.plan = own_reg(p.plan); r.sink = own_reg(p.sink); r.window = own_reg(p.window); r.budget_pages = own_reg(p.budget_pages);
    r.budget_bp = own_reg(p.budget_bp); r.over_chunk = own_reg(p.over_chunk); r.over_grid = own_reg(p.over_grid);
    r.rho_g_bp = own_reg(p.rho_g_bp); r.rho_c_bp = own_reg(p.rho_c_bp); r.rho_p_bp = own_reg(p.rho_p_bp);
    r.cap2 = own_reg(p.cap2); r.cap3 = own_reg(p.cap3); r.cap_keys = own_reg(p.cap_keys); r.cap_kg = own_reg(p.cap_kg);
    r.cap_kc = own_reg(p.cap_kc); r.probe = own_reg(p.probe); r.poll_limit = own_reg(p.poll_limit);
    r.general_cut = own_reg(p.general_cut); r.local_grids = own_reg(p.local_grids); r.schedule = own_reg(p.schedule);
    r.deciders = own_reg(p.deciders); r.inv_members = own_reg(p.inv_members); r.inv_others = own_reg(p.inv_others); r.keep_ties = own_reg(p.keep_ties); r.budget_per_seq = p.budget_per_seq;   // (a pointer would lose its address space)
    return r;
}

// The page budget the plan fixes for sequence b, or 0 when it is derived from the sequence's page count:
// budget_per_seq[b] when given and positive (clamped to what a page_ids row can hold), else budget_pages.
__device__ __forceinline__ int fixed_budget(const SelectParams& sp, const Geom& g, int b)
{
    const int per = sp.budget_per_seq != nullptr ? sp.budget_per_seq[b] : 0;
    const int room = g.max_sel - sp.sink - sp.window;
    return per > 0 ? (per < room ? per : (room > 1 ? room : 1)) : sp.budget_pages;
}

#ifndef CHESS_SEL_THREADS
#define CHESS_SEL_THREADS 256
#endif
constexpr int kSelThreads = CHESS_SEL_THREADS;   // workgroup of the selection kernels
constexpr int kSelMaxCluster = 32;   // most workgroups per (sequence, KV head)
// int32 from one arrival counter to the next.  Atomics on words of one 128-byte line are served one after the other, about 12 ns each:
// with its counter next to the others, the entropy of 16 rows of 32 splits took 11.6 us where it takes 6.7, 8 rows 8.1 (6.1); 32
// attention launches of 4 x 8 rows and the selection ahead of them 297 (281); 8 layers of 256 rows and the monitor 123.5 (119.9).
constexpr int kArrivalStride = 64;
constexpr int kSelMetaStride = kArrivalStride;   // int32 per (sequence, KV head): [0] members that are done with the published keys

// Select scratch in the caller's workspace (device pointers).
struct SelectWs {
    uint64_t* keys;                  // [rows][key_stride]  published candidate keys: grids | chunk slots | page slots;
    int64_t key_stride;              //   all zero between launches
    uint64_t* tail;                  // [rows][4] keys of the refreshed tail grid / chunk / page; zero between launches
    int32_t* meta;                   // [rows][kSelMetaStride], zero between launches
    int32_t* error;                  // one word of kErr* bits
#ifdef CHESS_PROF
    int32_t* prof;                   // [rows][Prof::kSlots] phase timestamps in 10 ns ticks (profiling builds only)
#endif
};
constexpr int kErrWait = 1;          // a wait for published keys was given up
constexpr int kErrOverflow = 2;      // the threshold rule kept more units than a list has room for (the list was cut short)

// Where in the argument segment of a kernel of this signature the first argument of type Arg lies: in order, each at the next multiple of
// its alignment.
template <class Arg, class... Args>
constexpr size_t kernarg_offset(void (*)(Args...))
{
    size_t at = 0, found = ~(size_t)0;
    const auto place = [&](size_t size, size_t align, bool it) {
        at = (at + align - 1) / align * align;
        found = it && found == ~(size_t)0 ? at : found;
        at += size;
    };
    (place(sizeof(Args), alignof(Args), std::is_same_v<Args, Arg>), ...);
    return found;
}

// The 64-byte lines of a kernel's arguments that hold bytes [kBegin, kEnd), asked for with the kernel's first instructions, so that the
// arguments are in the scalar cache when they are read: a first read takes 1.2 us, and the compiler puts it in front of its use.
template <size_t kBegin, size_t kEnd>
struct ArgLines {
    static_assert(kBegin < kEnd, "the kernel has no such parameter");
    static constexpr size_t kFirst = kBegin / 64, kLines = (kEnd - 1) / 64 - kFirst + 1;
    uint32_t w[kLines];
    __device__ __forceinline__ void ask()
    {
        typedef __attribute__((address_space(4))) const volatile uint32_t* kernarg;     // (volatile: not moved to where they are held)
        kernarg p = (kernarg)__builtin_amdgcn_kernarg_segment_ptr();
#pragma unroll
        for (size_t i = 0; i < kLines; ++i) w[i] = p[(kFirst + i) * 16];
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void hold() const
    {
#pragma unroll
        for (size_t i = 0; i < kLines; ++i) asm volatile("" : : "s"(w[i]) : "memory");
    }
};

// Those of the argument of type Arg of a kernel of signature Kernel (which whatever launches the kernel holds it to).
template <class Kernel, class Arg>
using ArgLinesOf = ArgLines<kernarg_offset<Arg>(Kernel(nullptr)), kernarg_offset<Arg>(Kernel(nullptr)) + sizeof(Arg)>;

// A pointer that travels as a number.
template <class V>
__device__ __forceinline__ V* device_pointer(uint64_t at)
{
    return (V*)(__attribute__((address_space(1))) V*)at;
}

// One word that every lane needs, as a vector load: the first of a kernel is back after 0.93 us, a scalar load after 1.25 (the lengths
// in the fused step, the phase marks of a profiling build).  The same value in every lane.
__device__ __forceinline__ int load_by_lane(const int32_t* p)
{
    int zero = 0;
    asm("" : "+v"(zero));
    return p[zero];
}

// Values that cross workgroups inside one launch travel as agent-scope atomics: on gfx950 these are loads and
// stores with the sc1 bit, which do not live in the per-XCD L2s as cached copies (a store is written through to
// the memory side that all eight XCDs share before it is acknowledged, a load is served from there), so they are
// coherent across the device without any cache maintenance.  Two kinds of message:
//  * a published word that IS the message (a key, polled until it is non-zero) needs no ordering against anything
//    else;
//  * data announced by something else (split partials by the arrival counter): the writer's waves wait until their
//    sc1 stores are acknowledged (s_waitcnt 0: by then they are at the shared memory side) before the workgroup's
//    barrier and the arrival, and the reader's sc1 loads, issued after it has seen the last arrival, are served from
//    that same place.  The language-level equivalent, a release fence before and an acquire fence after the arrival
//    at agent scope, was measured: it compiles to a write-back and an invalidate of the whole L2 (buffer_wbl2 sc1 /
//    buffer_inv sc1), which these accesses do not need, and costs 12 us per sparse-decode launch (14 -> 26 us).  So
//    the ordering rests on the hardware behaviour above, with relaxed atomics, not on the abstract memory model.
__device__ __forceinline__ void publish_u64(uint64_t* p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t observe_u64(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_f32(float* p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float observe_f32(const float* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by every thread of a workgroup after its publish_* stores.  Returns true (to every thread)
// in the workgroup that arrives last of `expected`; that workgroup also re-arms the counter for the
// next launch.  Nobody waits.  The counter must be 0 before the first launch.
__device__ __forceinline__ bool arrive_last(int32_t* counter, int expected, int* lds_flag)
{
    __builtin_amdgcn_s_waitcnt(0);                   // this wave's published stores are acknowledged, its loads have returned
    __syncthreads();
    if (threadIdx.x == 0) {
        const int old = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int last = old == expected - 1;
        if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *lds_flag = last;
    }
    __syncthreads();
    return *lds_flag != 0;
}

// The same where a row's workgroups are of two kinds: deciders (splits of the row's attention) and helpers (which only
// published keys).  One word counts both, deciders in its lower half.  Returns, to every thread, kLastDecider in the
// decider that arrives last of the deciders and kLastOfAll in whichever workgroup arrives last of all; that one re-arms
// the counter.
constexpr int kLastDecider = 1, kLastOfAll = 2;
__device__ __forceinline__ int arrive_of_two(int32_t* counter, bool decider, int n_deciders, int n_helpers, int* lds_flag)
{
    __builtin_amdgcn_s_waitcnt(0);                   // this wave's published stores are acknowledged, its loads have returned
    __syncthreads();
    if (threadIdx.x == 0) {
        const int old = __hip_atomic_fetch_add(counter, decider ? 1 : 0x10000, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int d = (old & 0xffff) + (decider ? 1 : 0), h = (old >> 16) + (decider ? 0 : 1);
        const bool all = d == n_deciders && h == n_helpers;
        if (all) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *lds_flag = (decider && d == n_deciders ? kLastDecider : 0) | (all ? kLastOfAll : 0);
    }
    __syncthreads();
    return *lds_flag;
}

}  // namespace chess

struct chess_ctx {
    chess_config cfg;
    chess::Geom geom;
    float sm_scale;
    int device;
    int n_cu;
    int lds_per_block;
    size_t page_off, chunk_off, grid_off, summary_bytes;   // bytes
    int max_splits;
    int force_splits, force_waves;                         // 0 = automatic
    size_t ws_acc_off, ws_ml_off, workspace_bytes;
    size_t ws_ent_off, ws_entcnt_off;                      // entropy partials, their arrival counters
    size_t ws_keys_off, ws_tail_off, ws_meta_off, ws_cnt_off, ws_err_off, ws_prof_off;   // select scratch, decode arrival counters, error word
    int64_t key_stride;
    int force_cluster;                                     // 0 = automatic
    int force_schedule;                                    // 0 = automatic, 1 + kLazy / kMerged / kEager
    int force_general_cut;                                 // 0 = automatic
    int poll_limit;                                        // 0 = the default
    int dense_blocks;                                      // workgroups of attention over every page per CU
    int occ_lds, occ_blocks;                               // cached occupancy query of the select kernel
    int step_occ_lds, step_occ_blocks;                     // ... and of the fused step kernel
    int shared_occ_lds, shared_occ_blocks;                 // ... and of the model-wide select kernel
    size_t ws_zero_off, ws_zero_bytes;                     // the part chess_workspace_init clears
    void* static_scratch;                                  // this device's copy of the library's own scratch array (or null)
};

namespace chess {

// Launch `kernel` on `stream` and report the launch status.
template <typename... KArgs, typename... Args>
inline hipError_t launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t stream, Args... args)
{
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, args...);
    return hipGetLastError();
}

// Launchers (each returns a hipError_t from the launch).
// (summary arrays travel as void*: fp32 or bf16 by the context's summary_dtype)
hipError_t launch_summarize(chess_ctx* ctx, const uint16_t* k_pool, const int32_t* block_table,
                            const int32_t* seq_lens, int batch, const int32_t* from_page, int recent,
                            void* pages, void* chunks, void* grids, hipStream_t stream);

hipError_t launch_select(chess_ctx* ctx, const uint16_t* q, const void* pages, const void* chunks,
                         const void* grids, const int32_t* seq_lens, int batch, int cluster, const SelectParams& sp,
                         const SelectWs& ws, size_t lds_bytes, int32_t* page_ids, int32_t* n_selected,
                         hipStream_t stream);
// Device pointers of one fused decode-step launch.
struct StepLaunch {
    const uint16_t* q;
    void* pages;             // the summary buffer: pages, chunks and grids behind one another
    const uint16_t* k_pool;
    const uint16_t* v_pool;
    const int32_t* block_table;
    const int32_t* seq_lens;
    int32_t* page_ids;
    int32_t* n_selected;
    float* out;
    float* ws_acc;
    float* ws_ml;
    int32_t* arrivals;       // [rows][kArrivalStride], as launch_decode's
    int32_t refresh_tail;
};
hipError_t launch_step(chess_ctx* ctx, const StepLaunch& sl, int batch, int cluster, const SelectParams& sp,
                       const SelectWs& ws, size_t lds_bytes, int union_off, hipStream_t stream);
size_t step_lds_bytes(const SelectParams& sp, int max_sel, int* union_off);
hipError_t step_occupancy(int page_size, bool bf16, int lds_bytes, int* blocks_per_cu);
hipError_t select_occupancy(bool bf16, int lds_bytes, int* blocks_per_cu);

// The model-wide scope: per-layer probes (fp32 [batch][H_kv][128]) and summary buffers, passed by value.
constexpr int kMaxLayers = CHESS_MAX_LAYERS;
constexpr int kSharedMaxCluster = 128;
struct SharedTable {
    const float* probes[kMaxLayers];
    const char* summaries[kMaxLayers];
    size_t page_off, chunk_off, grid_off;            // bytes into a summary buffer
    int n_layers;
};
struct AnchorTable {
    const char* summaries[kMaxLayers];
    float* anchors[kMaxLayers];
    size_t page_off;
};
hipError_t launch_anchor(chess_ctx* ctx, const AnchorTable& tab, int n_layers, const int32_t* seq_lens, int batch,
                         int window, hipStream_t stream);
hipError_t select_shared_occupancy(bool bf16, int lds_bytes, int* blocks_per_cu);
hipError_t launch_select_shared(chess_ctx* ctx, const SharedTable& tab, const int32_t* seq_lens, int batch, int cluster,
                                const SelectParams& sp, const SelectWs& ws, size_t lds_bytes, int32_t* page_ids,
                                int32_t* n_selected, hipStream_t stream);
size_t select_lds_bytes(const SelectParams& sp, int max_sel);
hipError_t dense_occupancy(int page_size, int group, int* blocks_per_cu);
hipError_t launch_append(chess_ctx* ctx, const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool, uint16_t* v_pool,
                         const int32_t* block_table, const int32_t* seq_lens, int batch, int32_t* page_ids,
                         int32_t* n_selected, hipStream_t stream);
// arrivals: as launch_decode's
hipError_t launch_reuse(chess_ctx* ctx, const uint16_t* q, const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool,
                        uint16_t* v_pool, const int32_t* block_table, const int32_t* seq_lens, int32_t* page_ids,
                        int32_t* n_selected, int batch, int n_splits, int waves, float* out, float* ws_acc, float* ws_ml,
                        int32_t* arrivals, hipStream_t stream);
hipError_t launch_extend(chess_ctx* ctx, const int32_t* seq_lens, int batch, int32_t* page_ids, int32_t* n_selected,
                         hipStream_t stream);
constexpr int kEntMaxSplits = 32;
// page_steps > 0: the thread that ends up with a sequence's entropy also does that sequence's trigger update.
// partials: [batch][splits][4]; arrivals: int32 [batch][kArrivalStride], as launch_decode's.
hipError_t launch_entropy(chess_ctx* ctx, const uint16_t* logits, int batch, int vocab, int64_t row_stride, int splits,
                          float* H, float* partials, int32_t* arrivals, int page_steps, double tau_h, double tau_v,
                          float* history, int32_t* count, int32_t* fire, double* stats, hipStream_t stream);
hipError_t launch_trigger(const float* H, int batch, int page_steps, double tau_h, double tau_v, float* history,
                          int32_t* count, int32_t* fire, double* stats, hipStream_t stream);
// p[0], p[stride], ...: n_words of them
hipError_t launch_zero(chess_ctx* ctx, int32_t* p, size_t n_words, int stride, hipStream_t stream);

// page_ids == nullptr: every page of the sequence.  n_splits >= 1; the last split of a (sequence,
// KV head) to finish merges the partials and writes `out`.  `arrivals`: int32 [rows][kArrivalStride], of which the first word of
// each row is used, zero before first use and left at zero.
hipError_t launch_decode(chess_ctx* ctx, const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool,
                         const int32_t* block_table, const int32_t* seq_lens, const int32_t* page_ids,
                         const int32_t* n_selected, int batch, int n_splits, int waves, int n_slots, float* out,
                         float* ws_acc, float* ws_ml, int32_t* arrivals, hipStream_t stream);

}  // namespace chess

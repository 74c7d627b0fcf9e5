// The whole decode step of one layer in one launch: coarse-to-fine page selection (Sec. 3.2, Alg. 1 stage 2)
// followed at once by block-sparse attention over the selected pages, read in place (Sec. 4.3, App. B).
//
// A cluster of C workgroups per (sequence, KV head) runs the three selection levels (select_device.h); the D of them
// that run the cuts (all, unless the schedule is eager) end up with the same page list in their LDS, so the list never
// travels through memory: member m goes straight on to decode tiles m, m + D, ... of it (decode_device.h) as split m of
// D, and the last of them to finish merges the D partials.  Compared with chess_select + chess_sparse_decode this saves a
// kernel boundary, the round trip of the list through HBM and the second kernel's start-up loads.
// Member 0 also writes the list to page_ids / n_selected when the caller wants it.
#include "decode_device.h"
#include "split_rule.h"
#include "select_device.h"

#include <type_traits>

namespace chess {

static_assert(kSelThreads % kWave == 0 && kSelThreads >= 256, "the fused step decodes with every wave of the workgroup");
constexpr int kStepWaves = kSelThreads / kWave;

struct StepArgs {
    const uint16_t* k_pool;
    const uint16_t* v_pool;
    int32_t* page_ids;       // may be null
    int32_t* n_selected;     // may be null
    float* out;
    float* ws_acc;
    float* ws_ml;
    int32_t* arrivals;
    float scale_log2;
    int32_t union_off;       // byte offset of the LDS region selection and decode share (after the page list)
    int32_t refresh_tail;    // recompute the summaries of the tail page, its chunk and its grid first
};

// The kernel's parameters (the table in step_kernel_of holds every instance to them).
using StepKernel = void (*)(uint64_t, uint64_t, uint64_t, uint64_t, int, int, int, int, int, int, StepArgs, Geom, SelectParams, SelectWs);

// A struct among the kernel's arguments, read where this stands and not when the kernel starts: what comes before does not wait for it,
// and what the compiler would keep in scalar registers meanwhile -- or, as there are too few, save and restore -- can be read again.
// With kAgain StepArgs are read again behind the selection (lane reads in the eager kernel's code: 930, so 440).  us, kept /
// read again: eager 1 x 4K 15.9 / 15.1, 32 layers of 1 x 32K 663 / 639; lean, reselection of 96 sequences, 116.1 / 109.0; but solo, 8
// layers of 32 x 16-32K, 259.8 / 262.8 and in clusters 8 x 128K 82.6 / 84.1: those two keep them.
template <class Arg>
__device__ __forceinline__ Arg late_arg()
{
    constexpr size_t at = kernarg_offset<Arg>(StepKernel(nullptr));
    static_assert(at != ~(size_t)0 && at % 4 == 0 && sizeof(Arg) % 4 == 0, "the kernel has no such parameter");
    typedef __attribute__((address_space(4))) const uint32_t* kernarg;
    kernarg p = (kernarg)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p) : : "memory");          // (nothing is moved across: not these loads, and not those before)
    struct Words { uint32_t w[sizeof(Arg) / 4]; } r;
#pragma unroll
    for (size_t i = 0; i < sizeof(Arg) / 4; ++i) r.w[i] = p[at / 4 + i];
    return __builtin_bit_cast(Arg, r);
}
// The structs' lines (see ArgLines; hold() goes where they are read).
using StepLines = ArgLines<kernarg_offset<StepArgs>(StepKernel(nullptr)), kernarg_offset<SelectWs>(StepKernel(nullptr)) + sizeof(SelectWs)>;
// (a pointer put together from words has no address space, and accesses through it would be flat ones)
template <class V>
__device__ __forceinline__ void in_device(V*& p) { p = device_pointer<V>((uint64_t)p); }
__device__ __forceinline__ StepArgs late_step_args()
{
    StepArgs a = late_arg<StepArgs>();
    in_device(a.k_pool); in_device(a.v_pool); in_device(a.page_ids); in_device(a.n_selected);
    in_device(a.out); in_device(a.ws_acc); in_device(a.ws_ml); in_device(a.arrivals);
    return a;
}
template <bool kAgain>
__device__ __forceinline__ StepArgs late_args(const StepArgs& a)
{
    if constexpr (kAgain) return late_step_args();
    else return a;
}

// The per-step refresh of the summaries (Sec. 3.1, Eq. 1-2) of the tail page, its chunk and its grid, done by one
// workgroup per (sequence, KV head) inside the step: thread c < 128 owns column c and adds in the same order as
// the summarize kernel (tokens, then the chunk's pages, then the grid's chunks, ascending, fp64, one rounding to
// the storage type per vector; a parent averages its children as they are stored), so the vectors are the ones
// chess_summarize_tail writes.  They go to the summaries and to `fresh` (LDS, [3][128]: page, chunk, grid); their
// scores against the probe are published as keys in tail_words[0..2] (grid, chunk, page) when `publish` is set (a
// cluster of one has nobody to tell) and kept in sh.tail_key.  In two steps, so that the rows' round trip hides behind
// the scoring of the grids: request, then finish.  Every thread of the workgroup must call both.
template <int B, class T>
struct TailUnits {
    static constexpr int kSib = 8;
    uint16_t kr[B];          // this thread's column of the page's key rows
    T sp[kSib], sc[kSib];    // ... of the first other pages of the chunk and the first other chunks of the grid
    // (rows past the last token repeat it, children past the tail unit -- the last of each -- repeat it: neither is added)
    __device__ __forceinline__ void request_siblings(const T* pages_row, const T* chunks_row, int P, const Geom& g)
    {
        const int c = threadIdx.x;
        if (c >= kHeadDim) return;
        const int tp = P - 1, tc = div_by(tp, g.inv_nc), tg = div_by(tc, g.inv_ng);
        const int p_lo = tc * g.n_c, c_lo = tg * g.n_g;
#pragma unroll
        for (int x = 0; x < kSib; ++x) {
            sp[x] = pages_row[(size_t)min(p_lo + x, tp) * kHeadDim + c];
            sc[x] = chunks_row[(size_t)min(c_lo + x, tc) * kHeadDim + c];
        }
    }
    __device__ __forceinline__ void request_rows(const uint16_t* __restrict__ k_pool, int64_t phys, int h, int H, int L, int P)
    {
        const int c = threadIdx.x;
        if (c >= kHeadDim) return;
        const int n_tok = L - (P - 1) * B;
        const uint16_t* rows = k_pool + ((phys * H + h) * B) * kHeadDim + c;
#pragma unroll
        for (int t = 0; t < B; ++t) kr[t] = rows[(size_t)min(t, n_tok - 1) * kHeadDim];
    }
    // all requested at once: one round trip for the usual hierarchy of 8 x 8
    __device__ __forceinline__ void request(const uint16_t* __restrict__ k_pool, int64_t phys, const T* pages_row,
                                            const T* chunks_row, int h, int H, int L, int P, const Geom& g)
    {
        request_rows(k_pool, phys, h, H, L, P);
        request_siblings(pages_row, chunks_row, P, g);
    }
    __device__ __forceinline__ void finish(T* pages_row, T* chunks_row, T* grids_row, int L, int P, const Geom& g,
                                           const double (&pr)[8], T* fresh, uint64_t* tail_words, bool publish, Shared& sh)
    {
        const int tid = threadIdx.x;
        const int tp = P - 1, tc = div_by(tp, g.inv_nc), tg = div_by(tc, g.inv_ng);
        const int n_tok = L - tp * B, p_lo = tc * g.n_c, c_lo = tg * g.n_g;
        if (tid < kHeadDim) {
            const int c = tid;
            // (a value is converted here and not as soon as it has arrived: converted early, the key rows were waited for before the
            // children's sums, and as doubles took so many registers that pages of 32 spilled.  us a layer, pages of 32, early / here:
            // 4 x 64K 28.9 / 25.8, with bf16 vectors 31.4 / 25.8, 1 x 32K 21.4 / 18.6, 32 x 16-32K with four KV heads 32.1 / 29.4)
            double acc_c = 0.0, acc_g = 0.0;
#pragma unroll
            for (int x = 0; x < kSib; ++x) {
                asm volatile("" : "+v"(sp[x]), "+v"(sc[x]));
                if (p_lo + x < tp) acc_c += loaded(sp[x]);
                if (c_lo + x < tc) acc_g += loaded(sc[x]);
            }
            // fan-outs beyond eight: the other children, eight at a time
            for (int j0 = p_lo + kSib; j0 < tp; j0 += kSib) {
#pragma unroll
                for (int x = 0; x < kSib; ++x) sp[x] = pages_row[(size_t)min(j0 + x, tp) * kHeadDim + c];
#pragma unroll
                for (int x = 0; x < kSib; ++x)
                    if (j0 + x < tp) acc_c += loaded(sp[x]);
            }
            for (int j0 = c_lo + kSib; j0 < tc; j0 += kSib) {
#pragma unroll
                for (int x = 0; x < kSib; ++x) sc[x] = chunks_row[(size_t)min(j0 + x, tc) * kHeadDim + c];
#pragma unroll
                for (int x = 0; x < kSib; ++x)
                    if (j0 + x < tc) acc_g += loaded(sc[x]);
            }
            double acc_p = 0.0;
#pragma unroll
            for (int t = 0; t < B; ++t) {
                asm volatile("" : "+v"(kr[t]));
                if (t < n_tok) acc_p += loaded(kr[t]);
            }
            const T vp = stored<T>(acc_p / (double)n_tok);
            const T vc = stored<T>((acc_c + loaded(vp)) / (double)(tp - tc * g.n_c + 1));
            const T vg = stored<T>((acc_g + loaded(vc)) / (double)(tc - tg * g.n_g + 1));
            pages_row[(size_t)tp * kHeadDim + c] = vp;
            chunks_row[(size_t)tc * kHeadDim + c] = vc;
            grids_row[(size_t)tg * kHeadDim + c] = vg;
            fresh[c] = vp;
            fresh[kHeadDim + c] = vc;
            fresh[2 * kHeadDim + c] = vg;
        }
        __syncthreads();
        // scores of the three vectors, one 16-lane group each, with the arithmetic of score_rows
        const int g16 = tid >> 4, ln = tid & 15;
        if (g16 < 3) {
            Vec<T> v;
            v.load(fresh + g16 * kHeadDim, ln);
            const double d = row16_sum(dot8<T>(pr, v));
            if (ln == 15) {
                const uint64_t key = order_key(d);
                const int level = 2 - g16;                            // fresh[0] is the page, fresh[2] the grid
                if (publish) publish_u64(tail_words + level, key);
                sh.tail_key[level] = key;
            }
        }
        __syncthreads();
    }
};

// What the first loads need beside pointers, in few registers: KV heads, the group, and how the first phase is shared (see
// choose_first_share): units a member takes, whether every member takes the same, whether the refreshing member (the last one under the
// eager schedule, else the first) takes none.
struct FirstLoads {
    static constexpr int kLocal = 1, kSpare = 2, kQueryProbe = 4, kGrids = 8, kChunks = 16, kFlagBits = 5, kPerBits = 11;
    int heads, share;        // n_kv_heads << 8 | group; per << kPerBits | members << kFlagBits | flags
};
static_assert(kSelMaxCluster < 1 << (FirstLoads::kPerBits - FirstLoads::kFlagBits), "members fit their bits");

// The eager schedule's last member, where the tail units are refreshed: it does that and nothing else.  Its keys are the last to be
// published, so its chain of loads (length, block table, key rows) waits for nothing of the others': with a share's vectors requested
// ahead of the block-table entry, the others waited 2 us more for its keys (32 layers of 1 x 32K 655 us).
template <int B, class T>
__device__ __forceinline__ void refresh_only(int L_lane, const int32_t* bt_row, T* pages_row, const VecBases& bases, ProbeRows<T>& probe, const uint16_t* q_rows, int G, int H,
                                             int h, size_t row, int C, int max_pages, const StepLines& lines, Shared& sh)
{
    __shared__ T fresh[3 * kHeadDim];
    const int L = min(max(__builtin_amdgcn_readfirstlane(L_lane), 0), max_pages * B), P = (L + B - 1) / B;
    if (P == 0) return;
    const int phys = load_by_lane(bt_row + P - 1);
    lines.hold();
    const StepArgs a = late_step_args();
    const Geom g = late_arg<Geom>();
    const SelectParams sp = late_arg<SelectParams>();
    SelectWs ws = late_arg<SelectWs>();
    in_device(ws.keys); in_device(ws.tail);
    T* chunks_row = pages_row + (int64_t)bases.chunks * kHeadDim;
    T* grids_row = pages_row + (int64_t)bases.grids * kHeadDim;
    TailUnits<B, T> tail;
    tail.request_siblings(pages_row, chunks_row, P, g);
    double pr[8];
    probe.sum(q_rows, G, pr);
    tail.request_rows(a.k_pool, __builtin_amdgcn_readfirstlane(phys), h, H, L, P);
    uint64_t* tail_words = ws.tail + row * 4;
    const bool compete = P > sp.sink + sp.window;     // (otherwise nobody reads the keys; the summaries are kept current)
    tail.finish(pages_row, chunks_row, grids_row, L, P, g, pr, fresh, tail_words, compete, sh);
    if (!compete) return;
    const int nc = div_by(P + g.n_c - 1, g.inv_nc), ng = div_by(nc + g.n_g - 1, g.inv_ng);
    if (arrive_of_two(a.arrivals + row * kArrivalStride, false, sp.deciders, C - sp.deciders, &sh.flag) & kLastOfAll)
        clear_published(pub_layout(ws.keys + row * ws.key_stride, g), CascadeResult{0, ng + nc, P - sp.window, false}, tail_words);
}

// grid = (C, H_kv, batch); T = storage type of the summaries (float or bf16 bits); kMode: see cascade_with; kLean: three
// workgroups on a compute unit instead of two (see launch_step)
// The pointers that the first loads need are numbers in the kernel's signature: a pointer among the arguments is looked up by the
// runtime at each launch, and in most processes the first launch with memory that it has not seen as an argument yet took longer there
// (first pass of a newly prepared reselection of 96 ragged sequences, two layers, states in turn in one process, pointers / numbers: 176 /
// 130 us in three processes of seven, 181 / 130 and 184 / 136 in two, equal in the others).
// The first loads need nothing but preloaded registers, and nothing waits for the other arguments before they are on their way: units of
// the first phase are counted in the configuration's (max_grids, then max_chunks, then max_pages), so that their vectors can be requested
// while the sequence's length is still on its way (0.93 us; 1.25 as a scalar load, which came back with the arguments).
// us a layer, with the vectors asked for behind the length and the arguments / as here: 1 x 4K 14.7 / 14.0, 32 layers of 1 x 32K 20.0 /
// 18.6, 8 of 32 x 16-32K 32.5 / 31.1, 2 of 8 x 128K 41.0 / 39.0, 8 of 1 x 256K with pages of 32 33.6 / 31.6.
template <int B, class T, int kMode, bool kLean>
__global__ __launch_bounds__(kSelThreads) __attribute__((amdgpu_waves_per_eu(kLean ? 3 : 2))) void step_kernel(uint64_t q_at, uint64_t seq_lens_at, uint64_t pages_at, uint64_t block_table_at,
                            int heads, int share, int max_pages, int max_chunks, int max_grids, int summary_rows, StepArgs, Geom, SelectParams, SelectWs)
{
    // (what the first loads need comes in registers, ahead of the structs: see build.py)
    const uint16_t* q = device_pointer<const uint16_t>(q_at);
    const int32_t* seq_lens = device_pointer<const int32_t>(seq_lens_at);
    __shared__ Shared sh;
    Prof prof;
    prof.mark(0);
    const int h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int H = heads >> 8, G = heads & 255, n_q_heads = H * G;
    const bool query_probe = (share & FirstLoads::kQueryProbe) != 0;
    StepLines lines;
    lines.ask();
    int L_raw = load_by_lane(seq_lens + b);                           // (scalar when it is used)
    const uint16_t* q_rows = q + ((size_t)b * n_q_heads + (size_t)h * G) * kHeadDim;
    double pr[8];
    ProbeRows<T> probe;
    probe.request(q_rows, 0, G);
    // ---- the first trip of the first phase's vectors
    const int m = kMode == kSolo ? 0 : blockIdx.x, C = kMode == kSolo ? 1 : (share >> FirstLoads::kFlagBits) & ((1 << (FirstLoads::kPerBits - FirstLoads::kFlagBits)) - 1);
    const size_t row = (size_t)b * H + h;
    T* pages_row = device_pointer<T>(pages_at) + row * max_pages * kHeadDim;
    const VecBases bases = bases_of(summary_rows, (int)row, max_pages, max_chunks, max_grids);
    const int32_t* bt_row = device_pointer<const int32_t>(block_table_at) + (size_t)b * max_pages;
    int tail_phys = 0;                                                // of the last page, where member 0 refreshes the tail units
    Vec<T> fly[kFlyOf<T, kLean>];
    const int n_static = (share & FirstLoads::kGrids ? max_grids : 0) + (share & FirstLoads::kChunks ? max_chunks : 0) + (kMode == kEagerCluster ? max_pages : 0);
    FirstShare first{n_static > 0, kMode == kSolo || (share & FirstLoads::kLocal) != 0, 0, n_static};
    {
        const int per = share >> FirstLoads::kPerBits, who = kMode == kEagerCluster ? C - 1 : 0;
        const bool spare = (share & FirstLoads::kSpare) != 0;
        if (!first.local) {
            first.lo = spare && m == who ? n_static : min(n_static, (spare && m > who ? m - 1 : m) * per);
            first.hi = min(n_static, first.lo + per);
        }
        const auto vec_of = [&](int slot) {
            if constexpr (kMode == kEagerCluster) return AllTarget{max_grids, max_grids + max_chunks, 0, 0, 0, 0, 0, bases}.vec(slot);
            else return GridPhaseTarget{max_grids, 0, 0, bases}.vec(slot);
        };
        if constexpr (kMode == kEagerCluster) {
            if (spare && m == who) {                                  // (what it asks for comes behind nothing)
                refresh_only<B, T>(L_raw, bt_row, pages_row, bases, probe, q_rows, G, H, h, row, C,
                                   max_pages, lines, sh);
                return;
            }
        }
        const auto ask = [&]() { ask_rows<T, kFlyOf<T, kLean>>(pages_row, first.lo, max(first.hi, 1), vec_of, tid >> 4, tid & 15, fly); };
        // The member that refreshes the tail units asks for the last block-table entry ahead of the vectors, or instead of them: the
        // key rows, which wait for it, are what its first cut waits for (loads return in order).
        const auto ask_last = [&]() { tail_phys = load_by_lane(bt_row + max((min(max(L_raw, 0), max_pages * B) + B - 1) / B - 1, 0)); };
        // (the length is waited for on either side of a branch: behind it, the wait would be for every load of the other side)
        if (kMode == kSolo || (kMode == kCluster && (!first.asked || (spare && m == 0)))) {
            L_raw = __builtin_amdgcn_readfirstlane(L_raw);
            if (m == 0) ask_last();
            probe.arrived();
            if (kMode == kSolo && first.asked) ask();
        } else {
            ask();                                                    // (of an empty share: some vector, which nobody looks at)
            L_raw = __builtin_amdgcn_readfirstlane(L_raw);
            if (kMode == kCluster && m == 0) ask_last();
        }
    }
    lines.hold();
    const StepArgs a = late_step_args();
    const Geom g_args = late_arg<Geom>();
    SelectParams sp_args = late_arg<SelectParams>();
    in_device(sp_args.budget_per_seq);
    SelectWs ws = late_arg<SelectWs>();
    in_device(ws.keys); in_device(ws.tail); in_device(ws.meta); in_device(ws.error);
    const Geom g = own_regs(g_args);
    const SelectParams sp = own_regs(sp_args);
    constexpr int PPT = 32 / B;
    extern __shared__ unsigned long long lds_raw[];
    int32_t* ids_l = reinterpret_cast<int32_t*>(lds_raw);                                  // [max_sel] the page list
    int32_t* phys_l = ids_l + g.max_sel;                                                   // [max_sel] their physical pages
    T* fresh = reinterpret_cast<T*>(reinterpret_cast<char*>(lds_raw) + a.union_off - 3 * kHeadDim * sizeof(float));   // [3][128]
    char* un = reinterpret_cast<char*>(lds_raw) + a.union_off;
    uint64_t* keys = reinterpret_cast<uint64_t*>(un);                                      // selection's view
    int32_t* kept_grids = reinterpret_cast<int32_t*>(keys + sp.cap_keys);
    int32_t* kept_chunks = kept_grids + sp.cap_kg;
    int32_t* phys_by_slot = kept_chunks + sp.cap_kc;                                       // [cap3]
    DecodeLds<kStepWaves> dl(reinterpret_cast<float*>(un));                                // decode's view
    // C members score; the first D of them go on to the cuts and the attention (all of them unless the schedule is eager)
    const int D = kMode == kEagerCluster ? sp.deciders : C;
    const int lane = tid & 63, wave = tid >> 6, m16 = lane & 15, grp = lane >> 4;
    const int k_fixed = fixed_budget(sp, g, b);
    init_shared(sh, sp.poll_limit);
    const int L = min(max(L_raw, 0), max_pages * B);
    const int P = (L + B - 1) / B;
    const int s = sp.sink, w = sp.window;
    if (P == 0) {                                                     // empty sequence: no pages, zero output
        if (m == 0) {
            if (a.page_ids) for (int i = tid; i < g.max_sel; i += kSelThreads) a.page_ids[row * g.max_sel + i] = -1;
            if (a.n_selected && tid == 0) a.n_selected[row] = 0;
            for (int i = tid; i < G * kHeadDim; i += kSelThreads) (a.out + ((size_t)b * n_q_heads + (size_t)h * G) * kHeadDim)[i] = 0.f;
        }
        return;
    }
    T* chunks_row = pages_row + (int64_t)bases.chunks * kHeadDim;
    T* grids_row = pages_row + (int64_t)bases.grids * kHeadDim;
    if (!query_probe) load_anchor<T>(pages_row, P, w, pr);
    // one member refreshes the tail units (eager: refresh_only's)
    const bool tail_on = a.refresh_tail != 0;
    const bool refreshes = kMode != kEagerCluster && tail_on && m == 0;
    uint64_t* tail_words = tail_on ? ws.tail + row * 4 : nullptr;
    TailUnits<B, T> tail;
    auto requested = [&]() {                                          // (the first vectors to score are on their way)
        if (query_probe) probe.sum(q_rows, G, pr);
        if (!kLean && refreshes) tail.request(a.k_pool, __builtin_amdgcn_readfirstlane(tail_phys), pages_row, chunks_row, h, H, L, P, g);
    };
    auto refresh_tail = [&]() {
        if (kLean) tail.request(a.k_pool, __builtin_amdgcn_readfirstlane(tail_phys), pages_row, chunks_row, h, H, L, P, g);   // (no registers for it before)
        tail.finish(pages_row, chunks_row, grids_row, L, P, g, pr, fresh, tail_words, C > 1 && P > s + w, sh);
    };
    __syncthreads();
    prof.mark(1);                                                     // prologue done

        // ---- the page list, in every member's LDS
    const PubLayout pubs = pub_layout(ws.keys + row * ws.key_stride, g);
    CascadeResult res;
    res.n_kp = 0; res.n_a = 0; res.n_p = 0; res.overflow = false;
    int n_sel;
    if (P <= s + w) {                                                 // safety pages cover the sequence
        if (refreshes) {                                              // nobody reads the keys; the summaries are kept current
            requested();
            refresh_tail();
        }
        if (m >= D) return;
        n_sel = min(P, g.max_sel);
        for (int i = tid; i < n_sel; i += kSelThreads) { ids_l[i] = i; phys_l[i] = bt_row[i]; }
    } else {
        // the block-table entries of the safety pages are requested now and used after the selection
        const bool safety_early = s + w <= kSelThreads;
        const int safety_lp = tid < s ? tid : P - w + (tid - s);
        int safety_phys = 0;
        if (safety_early && tid < s + w) safety_phys = bt_row[safety_lp];
        // kept pages and their physical pages go straight to their places in the list, behind the sinks
        const HeadScorer<T, kLean> scorer{pages_row, bases, pr, fly};
        const bool ok = cascade_with<kMode, true>(scorer, P, g, sp, pubs, m, C, m < D, keys, kept_grids,
                                         kept_chunks, ids_l + s, sh, &res, prof, tail_words, refreshes, requested, refresh_tail, k_fixed, first, bt_row,
                                         phys_by_slot, phys_l + s);
        if (!ok) {
            if (tid == 0) __hip_atomic_fetch_or(ws.error, kErrWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if (m >= D) {                                                 // a helper is done; normally long before the deciders are
            if (arrive_of_two(a.arrivals + row * kArrivalStride, false, D, C - D, &sh.flag) & kLastOfAll) clear_published(pubs, res, tail_words);
            return;
        }
        if (res.overflow && m == 0 && tid == 0) __hip_atomic_fetch_or(ws.error, kErrOverflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // union with the safety pages: sinks, kept pages, window -- already ascending
        const int n_kp = res.n_kp;
        n_sel = s + n_kp + w;
        if (safety_early) {
            if (tid < s + w) {
                const int at = tid < s ? tid : n_kp + tid;
                ids_l[at] = safety_lp;
                phys_l[at] = safety_phys;
            }
        } else {
            for (int i = tid; i < s + w; i += kSelThreads) {
                const int lp = i < s ? i : P - w + (i - s), at = i < s ? i : n_kp + i;
                ids_l[at] = lp;
                phys_l[at] = bt_row[lp];
            }
        }
    }
    __syncthreads();
    const StepArgs late = late_args<kMode == kEagerCluster || kLean>(a);
    float* late_out = late.out + ((size_t)b * n_q_heads + (size_t)h * G) * kHeadDim;
    if (m == 0) {
        if (late.page_ids) for (int i = tid; i < g.max_sel; i += kSelThreads) late.page_ids[row * g.max_sel + i] = i < n_sel ? ids_l[i] : -1;
        if (late.n_selected && tid == 0) late.n_selected[row] = n_sel;
    }
    prof.mark(14);                                                    // list built

    // ---- attention over this member's tiles of the list: split m of D
    const int n_tiles = (n_sel + PPT - 1) / PPT;
    const int stride = D * kStepWaves;
    const int t = m + D * wave;
    int raw_cur[PPT], raw_nxt[PPT];
    fetch_ids<B, true>(raw_cur, t, ids_l, max(n_sel, 1));
    fetch_ids<B, true>(raw_nxt, t + stride, ids_l, max(n_sel, 1));
    WaveAcc<B> acc;
    acc.init(q_rows, G, m16, grp);
    run_tiles<B, true, true, kLean>(acc, t, stride, n_tiles, n_sel, raw_cur, raw_nxt, ids_l, max(n_sel, 1), bt_row, phys_l, late.k_pool, late.v_pool, H, h, L, P,
                 late.scale_log2, m16, grp);
    prof.mark(15);                                                    // tiles done
    const bool split_up = combine_waves<kStepWaves>(acc.o, acc.m_run, acc.l_run, dl, G, D, m, row * D, late_out, late.ws_acc, late.ws_ml);
    prof.mark(16);                                                    // partial published (or, alone, the output written)
    // (profiling builds keep two timelines per row: member 0's and that of the member that merges)
    const int n_helpers = P <= s + w ? 0 : C - D;                     // (without a selection they have left)
    const int last = split_up || n_helpers > 0 ? arrive_of_two(late.arrivals + row * kArrivalStride, true, D, n_helpers, &sh.flag) : 0;
    prof.mark(17);
    // every member is done with the key words (the stores' way to memory hides behind the merge)
    if (last & kLastOfAll) clear_published(pubs, res, tail_words);
    if (split_up && (last & kLastDecider)) merge_splits<kStepWaves, kMode == kCluster ? kMergeCluster : kMergeStep>(G, D, row * D, late_out, late.ws_acc, late.ws_ml);
#ifdef CHESS_PROF
    prof.mark(18);
    if (tid == 0 && (!split_up || (last & kLastDecider))) prof.store(ws.prof + (row * 2 + 1) * Prof::kSlots);
    if (tid == 0 && m == 0) prof.store(ws.prof + (row * 2) * Prof::kSlots);
#endif
}

constexpr int kSoloLean = 3;                          // a cluster of one with three workgroups on a compute unit (see launch_step)
constexpr int kStepModes = 4;
static StepKernel step_kernel_of(int page_size, bool bf16, int mode)
{
    // [page size 16 / 32][fp32 / bf16][mode]
    static const StepKernel table[2][2][kStepModes] = {
        {{step_kernel<16, float, kSolo, false>, step_kernel<16, float, kCluster, false>, step_kernel<16, float, kEagerCluster, false>,
          step_kernel<16, float, kSolo, true>},
         {step_kernel<16, uint16_t, kSolo, false>, step_kernel<16, uint16_t, kCluster, false>, step_kernel<16, uint16_t, kEagerCluster, false>,
          step_kernel<16, uint16_t, kSolo, true>}},
        {{step_kernel<32, float, kSolo, false>, step_kernel<32, float, kCluster, false>, step_kernel<32, float, kEagerCluster, false>,
          step_kernel<32, float, kSolo, true>},
         {step_kernel<32, uint16_t, kSolo, false>, step_kernel<32, uint16_t, kCluster, false>, step_kernel<32, uint16_t, kEagerCluster, false>,
          step_kernel<32, uint16_t, kSolo, true>}}};
    return table[page_size == 16 ? 0 : 1][bf16 ? 1 : 0][mode];
}

// The region that the selection's levels and then the attention take.
static size_t step_level_bytes(const SelectParams& sp)
{
    const size_t sel = (size_t)sp.cap_keys * 8 + ((size_t)(sp.cap_kg + sp.cap_kc + sp.cap3) * 4 + 7) / 8 * 8;
    const size_t dec = (size_t)DecodeLds<kStepWaves>::kFloats * sizeof(float);
    return sel > dec ? sel : dec;
}

// Dynamic LDS of the fused kernel and where its shared region starts.
size_t step_lds_bytes(const SelectParams& sp, int max_sel, int* union_off)
{
    const size_t list = ((size_t)max_sel * 2 * 4 + 15) / 16 * 16 + 3 * kHeadDim * sizeof(float);   // page list, physical pages, refreshed tail vectors
    *union_off = (int)list;
    return list + step_level_bytes(sp);
}

// Workgroups that fit on a compute unit, of the kernels whose workgroups wait for each other.
hipError_t step_occupancy(int page_size, bool bf16, int lds_bytes, int* blocks_per_cu)
{
    int fit[2] = {0, 0};
    for (const int mode : {kCluster, kEagerCluster}) {
        const StepKernel kern = step_kernel_of(page_size, bf16, mode);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit[mode == kEagerCluster], kern, kSelThreads, lds_bytes);
        if (e != hipSuccess) return e;
    }
    *blocks_per_cu = fit[0] < fit[1] ? fit[0] : fit[1];
    return hipSuccess;
}

// Which of the first phase's vectors are requested before the lengths are known: units counted in the configuration's, dealt as
// the phase deals them; only where the first trip is all of them and, beside the eager schedule (whose bytes choose_eager bounds), they are
// few: of sequences much shorter than the configuration's most of them do not exist (8 MB take 1.3 us; us a layer with room for 4 to 32
// times the length, behind the length / as here: 1 x 4K 16.5 / 16.3 and 18.9 / 18.0, 8 x 8K 25.6 / 23.9,
// 32 x 4K 19.1 / 18.5; but 96 of 12 pages with room for 512 18.8 / 19.5, and where sink and window cover the sequence, which needs no vector
// at all, 8 of 5 pages 11.0 / 11.5).
static void choose_first_share(const Geom& g, const SelectParams& sp, int mode, int64_t rows, int cluster, bool bf16, int refresh_tail, FirstLoads* f)
{
    const bool solo = mode == kSolo || mode == kSoloLean, eager = mode == kEagerCluster;
    const int trip = kSelGroups * (bf16 ? 16 : 8) / (mode == kSoloLean ? 2 : 1);             // (HeadScorer::kTrip)
    int n = g.max_grids;
    if (sp.schedule == kMerged && !solo) n += g.max_chunks;
    if (eager) n += g.max_chunks + g.max_pages;
    const bool local = solo || (!eager && sp.schedule != kMerged && sp.local_grids != 0 && n <= kSelGroups * 8);
    const int without = cluster > 1 ? (n + cluster - 2) / (cluster - 1) : n;
    const bool spare = refresh_tail != 0 && !local && (eager || without <= trip);
    const int per = local ? n : spare ? without : (n + cluster - 1) / cluster;
    const int64_t bytes = rows * (local ? (int64_t)n * cluster : n) * kHeadDim * (bf16 ? 2 : 4);
    f->share |= cluster << FirstLoads::kFlagBits;
    if (!eager && (sp.cap_kg >= g.max_grids || per > trip || bytes > (8LL << 20))) return;      // (a grid level that keeps every grid is not scored)
    f->share |= per << FirstLoads::kPerBits | FirstLoads::kGrids | (n > g.max_grids ? FirstLoads::kChunks : 0) | (local ? FirstLoads::kLocal : 0) |
                (spare ? FirstLoads::kSpare : 0);
}

hipError_t launch_step(chess_ctx* ctx, const StepLaunch& sl, int batch, int cluster, const SelectParams& sp,
                       const SelectWs& ws, size_t lds_bytes, int union_off, hipStream_t stream)
{
    const Geom& g = ctx->geom;
    StepArgs a;
    a.k_pool = sl.k_pool; a.v_pool = sl.v_pool;
    a.page_ids = sl.page_ids; a.n_selected = sl.n_selected;
    a.out = sl.out; a.ws_acc = sl.ws_acc; a.ws_ml = sl.ws_ml; a.arrivals = sl.arrivals;
    a.scale_log2 = ctx->sm_scale * 1.4426950408889634f;
    a.union_off = union_off;
    a.refresh_tail = sl.refresh_tail;
    const dim3 grid(cluster, g.n_kv_heads, batch), block(kSelThreads);
    // Alone on their rows, more workgroups than two a compute unit would run in two rounds, the second nearly empty: from there on
    // the kernel that fits three times (half the vectors in flight, no tile ahead, the tail unit's rows requested when they are
    // needed: 142-154 registers instead of 198-212).  us a layer, two / three a compute unit: 576 rows of 8-16K 59.8 / 45.8,
    // 768 of 4-21K 73.2 / 58.2 (ratios and bf16 vectors 52.7 / 39.4), 1024 of 8K 61.8 / 57.3, 1536 of 4-8K 79.6 / 67.9, 2048 of 4K
    // 89.8 / 86.5.  Below, it depends: 512 of 8-16K 39.5 / 37.7, 512 of 16K with bf16 vectors 38.5 / 43.4, 256 of 16-32K 41.0 / 41.0.
    const bool lean = lean_step(ctx->n_cu, (int64_t)batch * g.n_kv_heads, step_level_bytes(sp) + sizeof(Shared));
    const int mode = cluster == 1 ? (lean ? kSoloLean : kSolo) : sp.schedule == kEager ? kEagerCluster : kCluster;
    const bool bf16 = ctx->cfg.summary_dtype == CHESS_SUMMARY_BF16;
    FirstLoads first{g.n_kv_heads << 8 | g.group, sp.probe == CHESS_PROBE_QUERY ? FirstLoads::kQueryProbe : 0};
    choose_first_share(g, sp, mode, (int64_t)batch * g.n_kv_heads, cluster, bf16, sl.refresh_tail, &first);
    const StepKernel kern = step_kernel_of(g.page_size, bf16, mode);
    if (lds_bytes > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
    }
    return launch(kern, grid, block, lds_bytes, stream, (uint64_t)sl.q, (uint64_t)sl.seq_lens, (uint64_t)sl.pages, (uint64_t)sl.block_table,
                  first.heads, first.share, g.max_pages, g.max_chunks, g.max_grids, ctx->cfg.max_batch * g.n_kv_heads, a, g, sp, ws);
}

}  // namespace chess

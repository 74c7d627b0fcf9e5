// The selection under the paper's own scope (Sec. 3.1, Eq. 1: a unit's vector is the concatenation, over all
// layers and heads, of the per-layer, per-head means) with the key anchor of Sec. 3.2, Eq. 3 as the probe:
// one score per unit, S(u) = sum over layers l and KV heads h of probe[l][h] . v[l][h][u] (Eq. 4 on the
// flattened vectors), one page set per sequence for the whole model.
//
// anchor_kernel: Eq. 3 for every (layer, sequence, KV head), as an output of its own.
// select_shared_kernel: a cluster of C workgroups per sequence runs the three levels of select_device.h; only the
// scoring differs.  A unit's vector is n_layers * H_kv rows of 512 bytes in as many arrays, so all 16 lane
// groups of a workgroup work on the same few slots: group j takes the rows r = j, j + 16, ... (row r = layer
// r / H_kv, head r % H_kv), up to eight slots and two rows or four slots and four rows at a time (sixteen vectors in flight per group), fp64
// partial sums; the groups' partials are added in group order through LDS.  The order of the additions is fixed, so a
// unit's score does not depend on the launch shape.
#include "select_device.h"

namespace chess {

// grid = (ceil(rows / 16), n_layers), 256 threads: a 16-lane group per (layer, sequence, KV head)
template <class T>
__global__ __launch_bounds__(256) void anchor_kernel(AnchorTable tab, const int32_t* __restrict__ seq_lens, int rows, Geom g,
                                                     int window)
{
    const int row = blockIdx.x * 16 + (threadIdx.x >> 4), ln = threadIdx.x & 15, l = blockIdx.y;
    if (row >= rows) return;
    const int b = row / g.n_kv_heads;
    const int L = min(max(seq_lens[b], 0), g.max_pages * g.page_size);
    const int P = (L + g.page_size - 1) / g.page_size;
    const T* pages = reinterpret_cast<const T*>(tab.summaries[l] + tab.page_off);
    double pr[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (P > 0) load_anchor<T>(pages + (size_t)row * g.max_pages * kHeadDim, P, window, pr);
    // the anchor is an fp32 vector [128] in dim order, whatever arrangement the lanes hold it in
    float* dst = tab.anchors[l] + (size_t)row * kHeadDim;
#pragma unroll
    for (int i = 0; i < 8; ++i) dst[Vec<T>::lane_dim(ln, i)] = (float)pr[i];
}

hipError_t launch_anchor(chess_ctx* ctx, const AnchorTable& tab, int n_layers, const int32_t* seq_lens, int batch,
                         int window, hipStream_t stream)
{
    const int rows = batch * ctx->geom.n_kv_heads;
    if (ctx->cfg.summary_dtype == CHESS_SUMMARY_BF16)
        return launch(anchor_kernel<uint16_t>, dim3((rows + 15) / 16, n_layers), dim3(256), 0, stream, tab, seq_lens, rows,
                      ctx->geom, window);
    return launch(anchor_kernel<float>, dim3((rows + 15) / 16, n_layers), dim3(256), 0, stream, tab, seq_lens, rows, ctx->geom,
                  window);
}

// Where the layers' probes and summaries are, in LDS.
struct SharedRows {
    uint64_t probes[kMaxLayers], summaries[kMaxLayers];
};

constexpr int kSharedSlots = 8;                      // slots a workgroup scores together

template <class T>
struct SharedScorer {
    static constexpr int kTrip = kSharedSlots;
    const SharedTable& tab;
    const SharedRows* rows;                          // LDS
    int b;
    const Geom& g;
    double* red;                                     // LDS [16 groups][kSharedSlots]
    VecBases at{0, 0};                               // (a slot's array and unit say where its rows are)

    // One pass: the N work slots s0 .. s0 + N - 1, all of one level (N is a template parameter so that exactly N
    // vectors per row are requested, all before the first is used: a run-time count would make the compiler wait
    // for each).
    template <int N, class Target>
    __device__ __forceinline__ void pass(int s0, Target target, bool local, uint64_t* keys, uint64_t* pub) const
    {
        const int tid = threadIdx.x, g16 = tid >> 4, ln = tid & 15;
        const int H = g.n_kv_heads, R = tab.n_layers * H;
        const int level = target(s0).array;          // (never the merged schedule: a pass stays inside one array)
        const size_t level_off = level == 0 ? tab.grid_off : level == 1 ? tab.chunk_off : tab.page_off;
        const size_t units = level == 0 ? g.max_grids : level == 1 ? g.max_chunks : g.max_pages;
        int unit[N];
        double part[N];
#pragma unroll
        for (int x = 0; x < N; ++x) {
            unit[x] = target(s0 + x).unit;
            part[x] = 0.0;
        }
        // Sixteen vectors in flight per group: four rows per trip where there are up to four slots, and two rows for what is left
        // then (up to 32 rows of all groups: four would be repeats; 16 rows a unit 21.5 us with two, 23.0 with four, 8 x 16K at 1 %).
        // A trip's last rows may not exist: it then reads the first row again and does not add it (an infinite component times a
        // zero probe would be a NaN).  The pointers come from LDS: loads from memory return in order, so a pointer fetched behind
        // vectors is waited for with them (four rows so: 83 us where two took 75).  Eight rows are slower.  (Why is not shown.  The
        // rows lie in as many buffers as there are layers, and a compute unit misses 95 address translations a launch, by counter,
        // where an attention launch misses 5; what these cost is not known.)  us, 32 layers of 8 KV heads at 1 %: two rows with
        // pointers from memory / from LDS / four rows / eight up to two slots: 4 sequences of 24-32K 75.8 / 72.1 / 67.8 / 71.6; one of
        // 32K 61.2 / 52.2 / 51.2 / 53.0; 16 of 8K 78.5 / 71.7 / 68.2 / 74.3
        const size_t head_bytes = units * (kHeadDim * sizeof(T));
        const size_t first_head = level_off + (size_t)b * H * head_bytes;
        const int step_l = kSelGroups / H, step_h = kSelGroups - step_l * H;
        int l = g16 / H, h = g16 - l * H, r = g16;
        const auto trip = [&](auto rows_a_trip) {
            constexpr int kRows = decltype(rows_a_trip)::value;
            if (r < R) {
                const float* from[kRows];
                const char* base[kRows];
#pragma unroll
                for (int y = 0; y < kRows; ++y) {
                    const bool have = r + y * kSelGroups < R;      // (r itself always is)
                    if (y > 0 && !have) {
                        from[y] = from[0];
                        base[y] = base[0];
                    } else {
                        from[y] = device_pointer<const float>(rows->probes[l]) + ((size_t)b * H + h) * kHeadDim;
                        base[y] = device_pointer<const char>(rows->summaries[l]) + first_head + (size_t)h * head_bytes;
                    }
                    h += step_h;
                    l += step_l + (h >= H ? 1 : 0);
                    h -= h >= H ? H : 0;
                    l = min(l, tab.n_layers - 1);                  // (past the last row: not read)
                }
                // the probes in the arrangement the vectors are held in (two runs of four consecutive dims)
                float4 pa[kRows], pb[kRows];
                Vec<T> v[kRows][N];
#pragma unroll
                for (int y = 0; y < kRows; ++y) {
                    pa[y] = *reinterpret_cast<const float4*>(from[y] + Vec<T>::lane_dim(ln, 0));
                    pb[y] = *reinterpret_cast<const float4*>(from[y] + Vec<T>::lane_dim(ln, 4));
#pragma unroll
                    for (int x = 0; x < N; ++x)       // always load (unit 0 when the slot has no unit): all stay in flight
                        v[y][x].load(reinterpret_cast<const T*>(base[y]) + (size_t)max(unit[x], 0) * kHeadDim, ln);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int y = 0; y < kRows; ++y) {
                    const bool have = r + y * kSelGroups < R;
                    const float pf[8] = {pa[y].x, pa[y].y, pa[y].z, pa[y].w, pb[y].x, pb[y].y, pb[y].z, pb[y].w};
                    double pr[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) pr[i] = (double)pf[i];
#pragma unroll
                    for (int x = 0; x < N; ++x) {
                        const double sum = dot8<T>(pr, v[y][x], part[x]);
                        part[x] = have ? sum : part[x];
                    }
                }
            }
            r += kRows * kSelGroups;
        };
        int left = R;                                          // rows of all groups
        if constexpr (N <= 4)
            for (; left > 2 * kSelGroups; left -= 4 * kSelGroups) trip(std::integral_constant<int, 4>{});
        for (; left > 0; left -= 2 * kSelGroups) trip(std::integral_constant<int, 2>{});
#pragma unroll
        for (int x = 0; x < N; ++x) {
            const double d = row16_sum(part[x]);
            if (ln == 15) red[g16 * kSharedSlots + x] = d;
        }
        __syncthreads();
        if (tid < N) {
            double d = 0.0;
#pragma unroll
            for (int j = 0; j < kSelGroups; ++j) d += red[j * kSharedSlots + tid];
            const SlotRef ref = target(s0 + tid);
            if (ref.dest >= 0) {
                if (local) keys[ref.dest] = ref.unit >= 0 ? order_key(d) : 0ull;
                else publish_u64(pub + ref.dest, ref.unit >= 0 ? order_key(d) : kAbsentKey);
            }
        }
        __syncthreads();                              // red is reused by the next pass
    }

    template <class Target, class Requested>
    __device__ __forceinline__ void operator()(int lo, int hi, Target target, bool local, uint64_t* keys, uint64_t* pub, Requested, bool) const
    {
        // the share in passes of equal size (the last may be shorter), at most kSharedSlots slots each
        const int n_pass = (hi - lo + kSharedSlots - 1) / kSharedSlots;
        const int per_pass = n_pass > 0 ? (hi - lo + n_pass - 1) / n_pass : 0;
        for (int s0 = lo; s0 < hi; s0 += per_pass) {
            switch (min(per_pass, hi - s0)) {             // uniform over the workgroup
            case 1: pass<1>(s0, target, local, keys, pub); break;
            case 2: pass<2>(s0, target, local, keys, pub); break;
            case 3: pass<3>(s0, target, local, keys, pub); break;
            case 4: pass<4>(s0, target, local, keys, pub); break;
            case 5: pass<5>(s0, target, local, keys, pub); break;
            case 6: pass<6>(s0, target, local, keys, pub); break;
            case 7: pass<7>(s0, target, local, keys, pub); break;
            default: pass<8>(s0, target, local, keys, pub); break;
            }
        }
    }
};
static_assert(kSharedSlots == 8, "the dispatch in SharedScorer lists the pass sizes");

// grid = (C, 1, batch); T = storage type of the summaries
template <class T, int kMode>
__global__ __launch_bounds__(kSelThreads) void select_shared_kernel(SharedTable tab, const int32_t* __restrict__ seq_lens,
                                                                    Geom g, SelectParams sp, SelectWs ws,
                                                                    int32_t* __restrict__ page_ids,
                                                                    int32_t* __restrict__ n_selected)
{
    extern __shared__ unsigned long long lds_raw[];
    uint64_t* keys = reinterpret_cast<uint64_t*>(lds_raw);                    // [cap_keys]
    int32_t* kept_grids = reinterpret_cast<int32_t*>(keys + sp.cap_keys);     // [cap_kg]
    int32_t* kept_chunks = kept_grids + sp.cap_kg;                            // [cap_kc]
    int32_t* sel_pages = kept_chunks + sp.cap_kc;                             // [max_sel]
    __shared__ Shared sh;
    __shared__ double red[kSelGroups * kSharedSlots];
    __shared__ SharedRows rows;

    const int m = blockIdx.x, C = gridDim.x, b = blockIdx.z, tid = threadIdx.x;
    const int H = g.n_kv_heads, B = g.page_size;
    Prof prof;
    init_shared(sh, sp.poll_limit);
    if (tid < tab.n_layers) {                        // (read after the barrier below)
        rows.probes[tid] = reinterpret_cast<uint64_t>(tab.probes[tid]);
        rows.summaries[tid] = reinterpret_cast<uint64_t>(tab.summaries[tid]);
    }
    const int L = min(max(seq_lens[b], 0), g.max_pages * B);
    const int k_fixed = fixed_budget(sp, g, b);
    const int P = (L + B - 1) / B;
    const int s = sp.sink, w = sp.window;
    // the list is the same for every KV head of the sequence: it is written H times, in the layout the
    // decode calls read
    if (P <= s + w) {                                                 // safety pages cover the sequence
        if (m == 0) {
            for (int i = tid; i < H * g.max_sel; i += kSelThreads) {
                const int at = i % g.max_sel;
                page_ids[(size_t)b * H * g.max_sel + i] = at < P ? at : -1;
            }
            if (tid < H) n_selected[b * H + tid] = min(P, g.max_sel);
        }
        return;
    }
    __syncthreads();

    const PubLayout pubs = pub_layout(ws.keys + (size_t)b * ws.key_stride, g);
    CascadeResult res;
    const SharedScorer<T> scorer{tab, &rows, b, g, red};
    const bool ok = cascade_with<kMode, false>(scorer, P, g, sp, pubs, m, C, m == 0, keys, kept_grids, kept_chunks, sel_pages, sh,
                                        &res, prof, nullptr, false, [] {}, [] {}, k_fixed, FirstShare{});
    if (!ok) {
        if (tid == 0) __hip_atomic_fetch_or(ws.error, kErrWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (C > 1) {
        // whoever is last to be done with the published words clears them for the next launch
        if (arrive_last(ws.meta + (size_t)b * kSelMetaStride, C, &sh.flag)) clear_published(pubs, res);
    }
    if (m != 0) return;
    if (res.overflow && tid == 0) __hip_atomic_fetch_or(ws.error, kErrOverflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    const int n_kp = res.n_kp, n_sel = s + n_kp + w;
    for (int i = tid; i < H * g.max_sel; i += kSelThreads) {
        const int at = i % g.max_sel;
        int v = -1;
        if (at < s) v = at;
        else if (at < s + n_kp) v = sel_pages[at - s];
        else if (at < n_sel) v = P - w + (at - s - n_kp);
        page_ids[(size_t)b * H * g.max_sel + i] = v;
    }
    if (tid < H) n_selected[b * H + tid] = n_sel;
}

using SharedKernel = void (*)(SharedTable, const int32_t*, Geom, SelectParams, SelectWs, int32_t*, int32_t*);
static SharedKernel shared_kernel_of(bool bf16, bool solo)
{
    if (bf16) return solo ? select_shared_kernel<uint16_t, kSolo> : select_shared_kernel<uint16_t, kCluster>;
    return solo ? select_shared_kernel<float, kSolo> : select_shared_kernel<float, kCluster>;
}

// (a cluster of one needs no co-residency: what counts is how many of the clusters' workgroups fit)
hipError_t select_shared_occupancy(bool bf16, int lds_bytes, int* blocks_per_cu)
{
    for (const bool solo : {true, false}) {
        if (lds_bytes <= 48 * 1024) break;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(shared_kernel_of(bf16, solo)), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, shared_kernel_of(bf16, false), kSelThreads, lds_bytes);
}

hipError_t launch_select_shared(chess_ctx* ctx, const SharedTable& tab, const int32_t* seq_lens, int batch, int cluster,
                                const SelectParams& sp, const SelectWs& ws, size_t lds_bytes, int32_t* page_ids,
                                int32_t* n_selected, hipStream_t stream)
{
    return launch(shared_kernel_of(ctx->cfg.summary_dtype == CHESS_SUMMARY_BF16, cluster == 1), dim3(cluster, 1, batch), dim3(kSelThreads),
                  lds_bytes, stream, tab, seq_lens, ctx->geom, sp, ws, page_ids, n_selected);
}

}  // namespace chess

// Coarse-to-fine page selection (Sec. 3.2, Eq. 4, Alg. 1 stage 2) as a call of its own: one launch, a
// cluster of C workgroups per (sequence, KV head); the levels themselves are in select_device.h.
// Member 0 of a cluster writes the list: sink pages, kept pages, window pages.
#include "select_device.h"

namespace chess {

// grid = (C, H_kv, batch); T = storage type of the summaries (float or bf16 bits)
// Three workgroups a compute unit.  Alone on its row, with fp32 vectors, a workgroup has half as many of them in flight: with all, the
// registers of three do not suffice (eight spilled), and of two make a second round.  us, spilled / two / half in flight: 32
// sequences of 8K 11.8 / 11.3 / 11.0, 96 of 4-21K 20.9 / 27.5 / 19.0, 128 of 2K 16.8 / 17.3 / 13.0 (four fit then).
template <class T, int kMode>
__global__ __launch_bounds__(kSelThreads) __attribute__((amdgpu_waves_per_eu(3))) void select_kernel(const uint16_t* __restrict__ q,
                                                             const void* __restrict__ pages_v,
                                                             const void* __restrict__ chunks_v,
                                                             const void* __restrict__ grids_v,
                                                             const int32_t* __restrict__ seq_lens, Geom g_args,
                                                             SelectParams sp_args, SelectWs ws,
                                                             int32_t* __restrict__ page_ids,
                                                             int32_t* __restrict__ n_selected)
{
    const Geom g = own_regs(g_args);
    const SelectParams sp = own_regs(sp_args);
    extern __shared__ unsigned long long lds_raw[];
    uint64_t* keys = reinterpret_cast<uint64_t*>(lds_raw);                    // [cap_keys]
    int32_t* kept_grids = reinterpret_cast<int32_t*>(keys + sp.cap_keys);     // [cap_kg]
    int32_t* kept_chunks = kept_grids + sp.cap_kg;                            // [cap_kc]
    int32_t* sel_pages = kept_chunks + sp.cap_kc;                             // [max_sel]
    __shared__ Shared sh;

    const int m = blockIdx.x, C = gridDim.x, h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const T* pages = static_cast<const T*>(pages_v);
    const T* chunks = static_cast<const T*>(chunks_v);
    const T* grids = static_cast<const T*>(grids_v);
    Prof prof;
    prof.mark(0);
    const size_t row = (size_t)b * g.n_kv_heads + h;
    int32_t* ids = page_ids + row * g.max_sel;
    const int B = g.page_size;
    const int L_raw = seq_lens[b];
    const int k_fixed = fixed_budget(sp, g, b);
    const uint16_t* q_rows = q + ((size_t)b * g.n_q_heads + (size_t)h * g.group) * kHeadDim;
    double pr[8];
    ProbeRows<T> probe;
    if (sp.probe == CHESS_PROBE_QUERY) probe.request(q_rows, 0, g.group);   // before anything waits on the length
    init_shared(sh, sp.poll_limit);
    const int L = min(max(L_raw, 0), g.max_pages * B);
    const int P = (L + B - 1) / B;
    const int s = sp.sink, w = sp.window;
    if (P <= s + w) {                                                 // safety pages cover the sequence
        if (m == 0) {
            for (int i = tid; i < g.max_sel; i += kSelThreads) ids[i] = i < P ? i : -1;
            if (tid == 0) n_selected[row] = min(P, g.max_sel);
        }
        return;
    }
    if (sp.probe == CHESS_PROBE_ANCHOR) load_anchor<T>(pages + row * g.max_pages * kHeadDim, P, w, pr);
    __syncthreads();
    prof.mark(1);                                                     // prologue done

    const PubLayout pubs = pub_layout(ws.keys + row * ws.key_stride, g);
    CascadeResult res;
    constexpr bool kHalf = kMode == kSolo && sizeof(T) == 4;
    Vec<T> fly[kFlyOf<T, kHalf>];
    const T* pages_row = pages + row * g.max_pages * kHeadDim;
    const auto vectors = [&](const T* to) { return (int)((to - pages_row) / kHeadDim); };
    const HeadScorer<T, kHalf> scorer{pages_row, VecBases{vectors(grids + row * g.max_grids * kHeadDim), vectors(chunks + row * g.max_chunks * kHeadDim)}, pr, fly};
    const bool ok = cascade_with<kMode, false>(scorer, P, g, sp, pubs, m, C, m == 0, keys, kept_grids, kept_chunks, sel_pages, sh, &res, prof, nullptr, false,
                                      [&] { if (sp.probe == CHESS_PROBE_QUERY) probe.sum(q_rows, g.group, pr); }, [] {}, k_fixed, FirstShare{});
    if (!ok) {
        if (tid == 0) __hip_atomic_fetch_or(ws.error, kErrWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if constexpr (kMode != kSolo) {
        // whoever is last to be done with the published words clears them for the next launch
        if (arrive_last(ws.meta + row * kSelMetaStride, C, &sh.flag)) clear_published(pubs, res);
    }
    if (m != 0) return;
    if (res.overflow && tid == 0) __hip_atomic_fetch_or(ws.error, kErrOverflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // ---- union with the safety pages: sinks, kept pages, window -- already ascending
    const int n_kp = res.n_kp, n_sel = s + n_kp + w;
    for (int i = tid; i < g.max_sel; i += kSelThreads) {
        int v = -1;
        if (i < s) v = i;
        else if (i < s + n_kp) v = sel_pages[i - s];
        else if (i < n_sel) v = P - w + (i - s - n_kp);
        ids[i] = v;
    }
    if (tid == 0) n_selected[row] = n_sel;
#ifdef CHESS_PROF
    prof.mark(15);
    if (tid == 0) prof.store(ws.prof + row * Prof::kSlots);
#endif
}

size_t select_lds_bytes(const SelectParams& sp, int max_sel)
{
    return (size_t)sp.cap_keys * 8 + ((size_t)(sp.cap_kg + sp.cap_kc + max_sel) * 4 + 7) / 8 * 8;
}

using SelectKernel = void (*)(const uint16_t*, const void*, const void*, const void*, const int32_t*, Geom, SelectParams, SelectWs, int32_t*, int32_t*);
static SelectKernel select_kernel_of(bool bf16, bool solo)
{
    if (bf16) return solo ? select_kernel<uint16_t, kSolo> : select_kernel<uint16_t, kCluster>;
    return solo ? select_kernel<float, kSolo> : select_kernel<float, kCluster>;
}

// (a cluster of one needs no co-residency: what counts is how many of the clusters' workgroups fit)
hipError_t select_occupancy(bool bf16, int lds_bytes, int* blocks_per_cu)
{
    for (const bool solo : {true, false}) {
        if (lds_bytes <= 48 * 1024) break;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(select_kernel_of(bf16, solo)), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        if (e != hipSuccess) return e;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, select_kernel_of(bf16, false), kSelThreads, lds_bytes);
}

hipError_t launch_select(chess_ctx* ctx, const uint16_t* q, const void* pages, const void* chunks,
                         const void* grids, const int32_t* seq_lens, int batch, int cluster, const SelectParams& sp,
                         const SelectWs& ws, size_t lds_bytes, int32_t* page_ids, int32_t* n_selected,
                         hipStream_t stream)
{
    return launch(select_kernel_of(ctx->cfg.summary_dtype == CHESS_SUMMARY_BF16, cluster == 1), dim3(cluster, ctx->geom.n_kv_heads, batch),
                  dim3(kSelThreads), lds_bytes, stream, q, pages, chunks, grids, seq_lens, ctx->geom, sp, ws, page_ids, n_selected);
}

}  // namespace chess

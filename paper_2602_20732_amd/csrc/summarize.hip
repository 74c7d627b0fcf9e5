// Hierarchical key summaries (Sec. 3.1): page vector = mean of the page's key rows (Eq. 1),
// chunk / grid vector = mean of the child vectors that exist (Eq. 2).
//
// One workgroup owns one (sequence, KV head, grid).  A 16-lane group streams one page: every lane
// issues 128-bit loads of 8 consecutive dims of one token row, so one wave instruction covers four
// 256-byte rows.  Each lane adds its 8 columns over the tokens in token order in fp64, so the sum
// is the same number whatever the launch shape; the mean is rounded to fp32 once.  Page vectors of
// the grid stay in LDS, chunk and grid means are formed from them without re-reading HBM.
#include <algorithm>

#include "select_device.h"

namespace chess {

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ void add_row(double (&acc)[8], const uint4& r)
{
    acc[0] += (double)bf16_lo(r.x); acc[1] += (double)bf16_hi(r.x);
    acc[2] += (double)bf16_lo(r.y); acc[3] += (double)bf16_hi(r.y);
    acc[4] += (double)bf16_lo(r.z); acc[5] += (double)bf16_hi(r.z);
    acc[6] += (double)bf16_lo(r.w); acc[7] += (double)bf16_hi(r.w);
}

// Eight consecutive elements of a stored vector (dims 8 ln .. 8 ln + 7), to and from memory (global or LDS).
template <class T>
struct Row8;
template <>
struct Row8<float> {
    float4 lo, hi;
    __device__ __forceinline__ void set(const double (&m)[8])
    {
        lo = make_float4((float)m[0], (float)m[1], (float)m[2], (float)m[3]);
        hi = make_float4((float)m[4], (float)m[5], (float)m[6], (float)m[7]);
    }
    __device__ __forceinline__ void load(const float* p) { lo = reinterpret_cast<const float4*>(p)[0]; hi = reinterpret_cast<const float4*>(p)[1]; }
    __device__ __forceinline__ void store(float* p) const { reinterpret_cast<float4*>(p)[0] = lo; reinterpret_cast<float4*>(p)[1] = hi; }
};
template <>
struct Row8<uint16_t> {
    uint4 v;
    // fp64 mean -> fp32 -> nearest-even bf16 (finite inputs), two per word
    static __device__ __forceinline__ uint32_t bf(double m)
    {
        const uint32_t u = __float_as_uint((float)m);
        return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    }
    __device__ __forceinline__ void set(const double (&m)[8])
    {
        v = make_uint4(bf(m[0]) | (bf(m[1]) << 16), bf(m[2]) | (bf(m[3]) << 16), bf(m[4]) | (bf(m[5]) << 16), bf(m[6]) | (bf(m[7]) << 16));
    }
    __device__ __forceinline__ void load(const uint16_t* p) { v = *reinterpret_cast<const uint4*>(p); }
    __device__ __forceinline__ void store(uint16_t* p) const { *reinterpret_cast<uint4*>(p) = v; }
};

__device__ __forceinline__ double as_f64(float v) { return (double)v; }
__device__ __forceinline__ double as_f64(uint16_t v) { return (double)__uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ void put_mean(float* p, double m) { *p = (float)m; }
__device__ __forceinline__ void put_mean(uint16_t* p, double m) { *p = (uint16_t)Row8<uint16_t>::bf(m); }

// T = storage type of the summaries (float, or bf16 bits: each stored mean is the fp32 mean rounded to nearest-even
// bf16, and a parent averages its children as they are stored)
template <int B, class T>
__global__ __launch_bounds__(256) void summarize_kernel(const uint16_t* __restrict__ k_pool,
                                                        const int32_t* __restrict__ block_table,
                                                        const int32_t* __restrict__ seq_lens,
                                                        const int32_t* __restrict__ from_page, int recent, Geom g,
                                                        T* __restrict__ pages, T* __restrict__ chunks,
                                                        T* __restrict__ grids)
{
    extern __shared__ float lds_f[];                  // [n_c * n_g][128] page vectors, then [n_g][128] chunk vectors, as stored
    T* lds = reinterpret_cast<T*>(lds_f);
    const int b = blockIdx.z, h = blockIdx.y, tid = threadIdx.x;
    const int L = min(seq_lens[b], g.max_pages * B);
    if (L <= 0) return;
    const int P = (L + B - 1) / B;
    const int nc = (P + g.n_c - 1) / g.n_c, ng = (nc + g.n_g - 1) / g.n_g;
    // recent > 0: only the last `recent` pages are new; the grid's workgroups count back from the last grid
    const int gk = recent > 0 ? ng - 1 - (int)blockIdx.x : (int)blockIdx.x;
    if (gk >= ng || gk < 0) return;
    int fp = recent > 0 ? P - recent : (from_page ? from_page[b] : 0);
    fp = fp < 0 ? 0 : fp;
    const int ppg = g.n_c * g.n_g;
    if (gk < fp / ppg) return;                        // every unit of this grid is older than from_page
    const int fc = fp / g.n_c;
    const int p_lo = gk * ppg, p_hi = min(P, p_lo + ppg);
    const int c_lo = gk * g.n_g, c_hi = min(nc, c_lo + g.n_g);
    const size_t row = (size_t)b * g.n_kv_heads + h;
    T* pg = pages + row * g.max_pages * kHeadDim;
    T* cg = chunks + row * g.max_chunks * kHeadDim;
    T* gg = grids + row * g.max_grids * kHeadDim;
    T* lds_chunk = lds + (size_t)ppg * kHeadDim;

    const int grp = tid >> 4, ln = tid & 15;
    for (int j = p_lo + grp; j < p_hi; j += 16) {
        T* dst = lds + (size_t)(j - p_lo) * kHeadDim + ln * 8;
        Row8<T> r8;
        if (j >= fp) {
            const int64_t phys = block_table[(size_t)b * g.max_pages + j];
            const int n = (j == P - 1) ? L - j * B : B;
            const uint4* src = reinterpret_cast<const uint4*>(k_pool + ((phys * g.n_kv_heads + h) * B) * kHeadDim) + ln;
            double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (n == B) {
#pragma unroll
                for (int t0 = 0; t0 < B; t0 += 16) {
                    uint4 r[16];
#pragma unroll
                    for (int t = 0; t < 16; ++t) r[t] = src[(t0 + t) * 16];
#pragma unroll
                    for (int t = 0; t < 16; ++t) add_row(acc, r[t]);
                }
            } else {
                for (int t = 0; t < n; ++t) add_row(acc, src[t * 16]);
            }
            const double dn = (double)n;
            double mean[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) mean[i] = acc[i] / dn;
            r8.set(mean);
            r8.store(pg + (size_t)j * kHeadDim + ln * 8);
        } else if (j / g.n_c >= fc) {                 // unchanged page whose chunk is being refreshed
            r8.load(pg + (size_t)j * kHeadDim + ln * 8);
        } else {
            continue;
        }
        r8.store(dst);
    }
    __syncthreads();

    for (int idx = tid; idx < (c_hi - c_lo) * kHeadDim; idx += 256) {
        const int c = c_lo + idx / kHeadDim, dim = idx % kHeadDim;
        T v;
        if (c >= fc) {
            const int lo = c * g.n_c, hi = min(P, lo + g.n_c);
            double acc = 0.0;
            for (int j = lo; j < hi; ++j) acc += as_f64(lds[(size_t)(j - p_lo) * kHeadDim + dim]);
            put_mean(&v, acc / (double)(hi - lo));
            cg[(size_t)c * kHeadDim + dim] = v;
        } else {
            v = cg[(size_t)c * kHeadDim + dim];
        }
        lds_chunk[idx] = v;
    }
    __syncthreads();

    if (tid < kHeadDim) {
        double acc = 0.0;
        for (int c = 0; c < c_hi - c_lo; ++c) acc += as_f64(lds_chunk[c * kHeadDim + tid]);
        T v;
        put_mean(&v, acc / (double)(c_hi - c_lo));
        gg[(size_t)gk * kHeadDim + tid] = v;
    }
}

// The same for the last few pages of every sequence (the per-step refresh, the catch-up before a reselection): one workgroup per
// (sequence, KV head), a 16-lane group per page and per unchanged page or chunk that a refreshed chunk or grid still averages, so
// everything is requested in two round trips behind the length (block-table entries, siblings; key rows) and the sums meet in LDS
// once a level.  The kernel above walks a grid's pages sixteen at a time and asks for an unchanged chunk when it comes to it.
// Bound: that chain.  us, 8 KV heads, sixteen draws of lengths of 8-16K, the kernel above / this one, 1 page, 10 and 16: 96 sequences 13.6 /
// 6.6, 23.9 / 12.4, 29.3 / 15.6; 32 11.0 / 5.3, 12.0 / 6.8, 15.3 / 8.3; one 5.5 / 4.2, 6.2 / 4.7, 7.4 / 5.1; pages of 32, 96 sequences 20.9 / 8.2,
// 38.6 / 18.8, 49.6 / 24.5 (all rows of a page at once: 12.0, 20.4, 26.8); 32 18.3 / 6.9, 20.5 / 9.3, 26.9 / 11.9; one 7.1 / 5.3, 8.7 / 6.0,
// 10.2 / 6.8.  With every last page full, where the kernel above is at its best: 96 11.6 / 8.5 (13.6 at once), 24.2 / 19.2, 35.1 / 25.0.
// shape: recent | n_c << 5 | n_g << 10 | KV heads << 15.  The arguments up to inv_ng are preloaded (see build.py).
constexpr int kRecentMost = 16;                       // pages, and children of a unit: one per group
template <int B, class T>
__global__ __launch_bounds__(256) void summarize_recent_kernel(uint64_t seq_lens_at, uint64_t block_table_at, uint64_t k_pool_at, uint64_t pages_at,
                                                               int max_pages, int shape, int rows, int max_chunks, uint32_t inv_nc,
                                                               uint32_t inv_ng, int max_grids)
{
    extern __shared__ float lds_f[];                  // page vectors from the first refreshed chunk's first page on, then chunk vectors
    const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, grp = tid >> 4, ln = tid & 15;
    const int recent = shape & 31, n_c = (shape >> 5) & 31, n_g = (shape >> 10) & 31, H = shape >> 15;
    T* lds_page = reinterpret_cast<T*>(lds_f);
    T* lds_chunk = lds_page + (n_c - 1 + recent) * kHeadDim;
    const int L = min(__builtin_amdgcn_readfirstlane(load_by_lane(device_pointer<const int32_t>(seq_lens_at) + b)), max_pages * B);
    if (L <= 0) return;
    const int P = (L + B - 1) / B, fp = max(P - recent, 0), n_new = P - fp;
    const int fc = div_by(fp, inv_nc), lc = div_by(P - 1, inv_nc), fg = div_by(fc, inv_ng), lg = div_by(lc, inv_ng);
    const int p0 = fc * n_c, c0 = fg * n_g;
    const int j = fp + min(grp, n_new - 1);           // this group's page
    const int64_t phys = device_pointer<const int32_t>(block_table_at)[(size_t)b * max_pages + j];
    const int row = b * H + h;
    const VecBases at = bases_of(rows, row, max_pages, max_chunks, max_grids);
    T* pg = device_pointer<T>(pages_at) + (size_t)row * max_pages * kHeadDim;
    T* cg = pg + (int64_t)at.chunks * kHeadDim;
    T* gg = pg + (int64_t)at.grids * kHeadDim;
    // (as words, not as Row8 and not as arrays: those went through scratch memory)
    constexpr int kHi = sizeof(T) == 4 ? 1 : 0;       // eight elements are two 16-byte words, or one
    const uint4* from_page = reinterpret_cast<const uint4*>(pg + (size_t)min(p0 + grp, P - 1) * kHeadDim + ln * 8);
    const uint4* from_chunk = reinterpret_cast<const uint4*>(cg + (size_t)min(c0 + grp, lc) * kHeadDim + ln * 8);
    const uint4 page_lo = from_page[0], page_hi = from_page[kHi], chunk_lo = from_chunk[0], chunk_hi = from_chunk[kHi];
    asm volatile("" : : : "memory");                  // (requested here, not where they are stored)
    if (grp < n_new) {                                // (a wave whose groups have no page skips the rows)
        const int n = j == P - 1 ? L - j * B : B;
        const uint4* src = reinterpret_cast<const uint4*>(device_pointer<const uint16_t>(k_pool_at) + ((phys * H + h) * B) * kHeadDim) + ln;
        double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, mean[8];
        // (sixteen at a time: 32 rows of a page at once are 172 registers, two workgroups to a compute unit)
#pragma unroll
        for (int t0 = 0; t0 < B; t0 += 16) {
            uint4 r[16];
#pragma unroll
            for (int t = 0; t < 16; ++t) r[t] = src[min(t0 + t, n - 1) * 16];      // (rows past the last token repeat it and are not added)
#pragma unroll
            for (int t = 0; t < 16; ++t)
                if (t0 + t < n) add_row(acc, r[t]);
        }
        const double dn = (double)n;
#pragma unroll
        for (int i = 0; i < 8; ++i) mean[i] = acc[i] / dn;
        Row8<T> mean8;
        mean8.set(mean);
        mean8.store(lds_page + (j - p0) * kHeadDim + ln * 8);
        mean8.store(pg + (size_t)j * kHeadDim + ln * 8);
    }
    if (p0 + grp < fp) {
        uint4* to = reinterpret_cast<uint4*>(lds_page + grp * kHeadDim + ln * 8);
        to[0] = page_lo;
        if (kHi) to[kHi] = page_hi;
    }
    if (c0 + grp < fc) {
        uint4* to = reinterpret_cast<uint4*>(lds_chunk + grp * kHeadDim + ln * 8);
        to[0] = chunk_lo;
        if (kHi) to[kHi] = chunk_hi;
    }
    __syncthreads();

    // a unit's mean, one dim a thread: its children [lo, hi), in order, eight read at a time
    const int dim = tid % kHeadDim;
    const auto mean_of = [&](const T* children, int lo, int hi, int from) {
        double sum = 0.0;
        for (int k0 = lo; k0 < hi; k0 += 8) {
            T v[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) v[x] = children[(min(k0 + x, hi - 1) - from) * kHeadDim + dim];
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (k0 + x < hi) sum += as_f64(v[x]);
        }
        T m;
        put_mean(&m, sum / (double)(hi - lo));
        return m;
    };
    for (int c = fc + tid / kHeadDim; c <= lc; c += 2) {
        const T v = mean_of(lds_page, c * n_c, min(P, c * n_c + n_c), p0);
        cg[(size_t)c * kHeadDim + dim] = v;
        lds_chunk[(c - c0) * kHeadDim + dim] = v;
    }
    __syncthreads();
    for (int k = fg + tid / kHeadDim; k <= lg; k += 2) gg[(size_t)k * kHeadDim + dim] = mean_of(lds_chunk, k * n_g, min(lc + 1, k * n_g + n_g), c0);
}

static hipError_t launch_recent(chess_ctx* ctx, const uint16_t* k_pool, const int32_t* block_table, const int32_t* seq_lens, int batch, int recent,
                                void* pages, hipStream_t stream)
{
    const Geom& g = ctx->geom;
    const bool bf16 = ctx->cfg.summary_dtype == CHESS_SUMMARY_BF16;
    // pages of the first refreshed chunk and the new ones, chunks of the first refreshed grid and the new ones
    const int new_chunks = (recent + g.n_c - 2) / g.n_c + 1;
    const size_t lds = (size_t)(g.n_c - 1 + recent + g.n_g - 1 + new_chunks) * kHeadDim * (bf16 ? sizeof(uint16_t) : sizeof(float));
    const auto kern = bf16 ? (g.page_size == 16 ? summarize_recent_kernel<16, uint16_t> : summarize_recent_kernel<32, uint16_t>)
                           : (g.page_size == 16 ? summarize_recent_kernel<16, float> : summarize_recent_kernel<32, float>);
    return launch(kern, dim3(g.n_kv_heads, batch), dim3(256), lds, stream, (uint64_t)seq_lens, (uint64_t)block_table, (uint64_t)k_pool, (uint64_t)pages,
                  g.max_pages, recent | g.n_c << 5 | g.n_g << 10 | g.n_kv_heads << 15, ctx->cfg.max_batch * g.n_kv_heads, g.max_chunks, g.inv_nc,
                  g.inv_ng, g.max_grids);
}

hipError_t launch_summarize(chess_ctx* ctx, const uint16_t* k_pool, const int32_t* block_table,
                            const int32_t* seq_lens, int batch, const int32_t* from_page, int recent,
                            void* pages, void* chunks, void* grids, hipStream_t stream)
{
    const Geom& g = ctx->geom;
    // (at its least favourable, one sequence whose last page is full, the kernel above and this one, 16 pages: of 32 8.0 / 6.8 us, of 16 6.0 / 5.1;
    // hierarchies of 4 x 4, where a grid is one trip for it, 5.9 / 7.1 and 4.7 / 5.3, but 8.4 / 7.1 and 5.4 / 5.4 over all lengths)
    if (recent > 0 && recent <= kRecentMost && g.n_c <= kRecentMost && g.n_g <= kRecentMost && g.n_kv_heads < 1 << 16)
        return launch_recent(ctx, k_pool, block_table, seq_lens, batch, recent, pages, stream);
    const bool bf16 = ctx->cfg.summary_dtype == CHESS_SUMMARY_BF16;
    const size_t lds = (size_t)(g.n_c * g.n_g + g.n_g) * kHeadDim * (bf16 ? sizeof(uint16_t) : sizeof(float));
    const int ppg = g.n_c * g.n_g;
    const int span = recent > 0 ? std::min(g.max_grids, (recent + ppg - 2) / ppg + 1) : g.max_grids;   // grids `recent` pages can touch
    const dim3 grid(span, g.n_kv_heads, batch), block(256);
    const void* kern = bf16 ? (g.page_size == 16 ? reinterpret_cast<const void*>(summarize_kernel<16, uint16_t>)
                                                 : reinterpret_cast<const void*>(summarize_kernel<32, uint16_t>))
                            : (g.page_size == 16 ? reinterpret_cast<const void*>(summarize_kernel<16, float>)
                                                 : reinterpret_cast<const void*>(summarize_kernel<32, float>));
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    if (bf16) {
        auto k = g.page_size == 16 ? summarize_kernel<16, uint16_t> : summarize_kernel<32, uint16_t>;
        return launch(k, grid, block, lds, stream, k_pool, block_table, seq_lens, from_page, recent, g,
                      static_cast<uint16_t*>(pages), static_cast<uint16_t*>(chunks), static_cast<uint16_t*>(grids));
    }
    auto k = g.page_size == 16 ? summarize_kernel<16, float> : summarize_kernel<32, float>;
    return launch(k, grid, block, lds, stream, k_pool, block_table, seq_lens, from_page, recent, g,
                  static_cast<float*>(pages), static_cast<float*>(chunks), static_cast<float*>(grids));
}

}  // namespace chess

// The quality monitor of Sec. 3.3: the entropy of each decode step's output distribution, and per generated
// page the average entropy and the variance of the entropy over the page's steps; reselection is asked for when
// either is above its threshold.
//
// entropy_kernel: grid (splits, batch).  A workgroup streams its slice of the sequence's logits row (bf16,
// 16-byte loads) keeping, per thread, the running maximum m, s0 = sum e^(z - m) and s1 = sum e^(z - m) (z - m);
// waves, the workgroup, then the splits (by the last one to finish) merge such triplets, in a fixed order, and
// H = log s0 - s1 / s0.  Bound: latency (a row of 150K logits is 300 KB; a batch of 32 moves 10 MB).
// trigger_kernel: one thread per sequence appends the step's entropy to the page's history and, when the page is
// complete, takes mean and population variance in fp64 in step order.
#include "chess_internal.h"

namespace chess {

struct Ent {
    float m, s0, s1;
};

__device__ __forceinline__ Ent ent_merge(const Ent& a, const Ent& b)
{
    const float M = fmaxf(a.m, b.m);
    if (M == -INFINITY) return Ent{M, 0.f, 0.f};
    const float da = a.m - M, db = b.m - M;              // <= 0; -inf for an empty side
    const float ea = a.s0 > 0.f ? __expf(da) : 0.f, eb = b.s0 > 0.f ? __expf(db) : 0.f;
    Ent r;
    r.m = M;
    r.s0 = a.s0 * ea + b.s0 * eb;
    r.s1 = (a.s0 > 0.f ? (a.s1 + da * a.s0) * ea : 0.f) + (b.s0 > 0.f ? (b.s1 + db * b.s0) * eb : 0.f);
    return r;
}

__device__ __forceinline__ void trigger_update_one(float Hb, int b, int count_before, int page_steps, double tau_h, double tau_v,
                                                   float* __restrict__ history, int32_t* __restrict__ count,
                                                   int32_t* __restrict__ fire, double* __restrict__ stats);

// Sum / maximum of a value over the wave (row shifts and row broadcasts, no LDS), in every lane.
template <class Op>
__device__ __forceinline__ float wave_all(float v, float identity, Op op)
{
    const int id = __float_as_int(identity);
#define CHESS_WAVE_STEP(ctrl, rows) v = op(v, __int_as_float(__builtin_amdgcn_update_dpp(id, __float_as_int(v), ctrl, rows, 0xf, false)));
    CHESS_WAVE_STEP(0x111, 0xf) CHESS_WAVE_STEP(0x112, 0xf) CHESS_WAVE_STEP(0x114, 0xf) CHESS_WAVE_STEP(0x118, 0xf)
    CHESS_WAVE_STEP(0x142, 0xa) CHESS_WAVE_STEP(0x143, 0xc)
#undef CHESS_WAVE_STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The triplets of a wave's lanes merged, in every lane: the maximum first, one exponential a lane to bring its sums to it, then
// plain sums in a fixed order.  (A tree of pairwise merges is two exponentials a level in one chain; twice per launch.)
__device__ __forceinline__ Ent ent_wave(const Ent& e)
{
    const float M = wave_all(e.m, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
    if (M == -INFINITY) return Ent{M, 0.f, 0.f};
    const bool some = e.s0 > 0.f;
    const float d = some ? e.m - M : 0.f, f = some ? __expf(d) : 0.f;
    const auto add = [](float a, float b) { return a + b; };
    return Ent{M, wave_all(e.s0 * f, 0.f, add), wave_all((e.s1 + d * e.s0) * f, 0.f, add)};
}

// What the entropy kernel reads late, and what the monitor call adds to it: the page statistics, done by the thread that has the entropy.
struct EntropyArgs {
    float* H;
    float* partials;                                     // [batch][splits][4]
    int32_t* arrivals;                                   // [batch] kArrivalStride apart, zero between launches
    double tau_h, tau_v;
    float* history;
    int32_t* fire;
    double* stats;
};
using EntropyKernel = void (*)(const uint16_t*, int32_t*, int64_t, int, int, int, int, EntropyArgs);

constexpr int kEntThreads = 256;
constexpr int kEntFly = 4;                               // 16-byte loads per thread and trip

// The first loads need only the arguments ahead of `tr`, which are in registers when a wave starts; the lines of the others are asked for
// with the first instruction and are there when the row has been read.  `per`: 16-byte chunks a split.  page_steps 0: entropy only.
// us, rows of 151936 logits, every argument fetched, every logit masked for itself, the counters side by side and two workgroups a compute
// unit / now: one 6.2 / 5.7, 8 rows 8.7 / 6.1, 16 12.2 / 6.6, 32 11.7 / 8.1, 96 15.1 / 12.3; preloading and masks by the word alone: 5.6, 8.1
// (8 rows), 10.8 (32), 13.6 (96).
__global__ __launch_bounds__(kEntThreads) void entropy_kernel(const uint16_t* __restrict__ logits, int32_t* __restrict__ count, int64_t row_stride,
                                                              int vocab, int n_splits, int per, int page_steps, EntropyArgs tr)
{
    ArgLinesOf<EntropyKernel, EntropyArgs> lines;
    lines.ask();
    __shared__ Ent lds[kEntThreads / 64];
    __shared__ int flag;
    const int split = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    // (asked for now: whoever ends up with the entropy would wait for it then)
    const int count_before = page_steps > 0 ? count[b] : 0;
    const auto finish = [&](const Ent& e) {
        const float Hb = e.s0 > 0.f ? logf(e.s0) - e.s1 / e.s0 : 0.f;
        tr.H[b] = Hb;
        if (page_steps > 0) trigger_update_one(Hb, b, count_before, page_steps, tr.tau_h, tr.tau_v, tr.history, count, tr.fire, tr.stats);
    };
    const uint4* row = reinterpret_cast<const uint4*>(logits + (size_t)b * row_stride);
    const int n_chunks = (vocab + 7) / 8;                                    // 8 logits per 16 bytes
    const int c_lo = split * per, c_hi = min(n_chunks, c_lo + per);
    Ent acc{-INFINITY, 0.f, 0.f};
    for (int c0 = c_lo + tid; c0 < c_hi; c0 += kEntThreads * kEntFly) {
        uint4 r[kEntFly];
#pragma unroll
        for (int x = 0; x < kEntFly; ++x) r[x] = row[min(c0 + x * kEntThreads, c_hi - 1)];
        float z[kEntFly * 8];
        float mx = -INFINITY;
#pragma unroll
        for (int x = 0; x < kEntFly; ++x) {
            const int c = c0 + x * kEntThreads;
            const uint32_t none = 0xff80ff80u;               // two times -inf
            uint32_t w[4] = {r[x].x, r[x].y, r[x].z, r[x].w};
            if (c >= n_chunks - 1) {                          // (the row's last chunk may be partly beyond the vocabulary)
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (c * 8 + i >= vocab) w[i >> 1] = (i & 1) ? (w[i >> 1] & 0xffffu) | (none & 0xffff0000u) : (w[i >> 1] & 0xffff0000u) | (none & 0xffffu);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = c < c_hi ? w[i] : none;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                z[x * 8 + i] = __uint_as_float((i & 1) ? (w[i >> 1] & 0xffff0000u) : (w[i >> 1] << 16));
                mx = fmaxf(mx, z[x * 8 + i]);
            }
        }
        if (mx == -INFINITY) continue;
        Ent e{mx, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < kEntFly * 8; ++i) {
#pragma clang fp contract(off)
            const float d = z[i] - mx;                    // -inf for a masked entry: contributes 0 (times a finite number: 0 x inf is none)
            const float p = __expf(d);
            e.s0 += p;
            e.s1 += p * fmaxf(d, -1e30f);
        }
        acc = ent_merge(acc, e);
    }
    lines.hold();
    const Ent own = ent_wave(acc);
    if ((tid & 63) == 0) lds[tid >> 6] = own;
    __syncthreads();
    if (tid < 64) {
        const Ent e = ent_wave(tid < kEntThreads / 64 ? lds[tid] : Ent{-INFINITY, 0.f, 0.f});
        if (tid == 0) {
            if (n_splits == 1) finish(e);
            else {
                float* p = tr.partials + ((size_t)b * n_splits + split) * 4;
                publish_f32(p, e.m); publish_f32(p + 1, e.s0); publish_f32(p + 2, e.s1);
            }
        }
    }
    if (n_splits == 1) return;
    if (!arrive_last(tr.arrivals + b * kArrivalStride, n_splits, &flag)) return;
    // the splits' triplets: lane s of wave 0 takes split s (at most kEntMaxSplits = 32 of them)
    if (tid < 64) {
        Ent e{-INFINITY, 0.f, 0.f};
        if (tid < n_splits) {
            const float* p = tr.partials + ((size_t)b * n_splits + tid) * 4;
            e = Ent{observe_f32(p), observe_f32(p + 1), observe_f32(p + 2)};
        }
        e = ent_wave(e);
        if (tid == 0) finish(e);
    }
}

hipError_t launch_entropy(chess_ctx* ctx, const uint16_t* logits, int batch, int vocab, int64_t row_stride, int splits,
                          float* H, float* partials, int32_t* arrivals, int page_steps, double tau_h, double tau_v,
                          float* history, int32_t* count, int32_t* fire, double* stats, hipStream_t stream)
{
    (void)ctx;
    const EntropyArgs tr{H, partials, arrivals, tau_h, tau_v, history, fire, stats};
    const int chunks = (vocab + 7) / 8;                   // (as the kernel counts them: 8 logits per 16 bytes)
    const EntropyKernel kern = entropy_kernel;            // (the signature that its argument lines follow from)
    return launch(kern, dim3(splits, batch), dim3(kEntThreads), 0, stream, logits, count, row_stride, vocab, splits,
                  (chunks + splits - 1) / splits, page_steps, tr);
}

// The page statistics of one sequence (what trigger_kernel does per thread).
__device__ __forceinline__ void trigger_update_one(float Hb, int b, int count_before, int page_steps, double tau_h, double tau_v,
                                                   float* __restrict__ history, int32_t* __restrict__ count,
                                                   int32_t* __restrict__ fire, double* __restrict__ stats)
{
    float* hist = history + (size_t)b * page_steps;
    int c = count_before;                                 // count[b] as the launch found it
    if (c < 0 || c >= page_steps) c = 0;                  // a state the caller did not initialise
    hist[c] = Hb;
    ++c;
    int f = 0;
    if (c == page_steps) {                                // the page is complete
        double s = 0.0, q = 0.0;
        for (int i = 0; i < page_steps - 1; ++i) s += (double)hist[i];
        s += (double)Hb;                                  // (the entry just stored, without reading it back)
        const double mu = s / (double)page_steps;
        for (int i = 0; i < page_steps; ++i) {
#pragma clang fp contract(off)                            // product rounded, then added: no fused multiply-add
            const double d = (double)(i == page_steps - 1 ? Hb : hist[i]) - mu;
            const double dd = d * d;
            q = q + dd;
        }
        const double var = q / (double)page_steps;
        f = (mu > tau_h || var > tau_v) ? 1 : 0;
        if (stats) { stats[2 * b] = mu; stats[2 * b + 1] = var; }
        c = 0;
    }
    fire[b] = f;
    count[b] = c;
}

// one thread per sequence
__global__ void trigger_kernel(const float* __restrict__ H, int batch, int page_steps, double tau_h, double tau_v,
                               float* __restrict__ history, int32_t* __restrict__ count, int32_t* __restrict__ fire,
                               double* __restrict__ stats)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= batch) return;
    trigger_update_one(H[b], b, count[b], page_steps, tau_h, tau_v, history, count, fire, stats);
}

hipError_t launch_trigger(const float* H, int batch, int page_steps, double tau_h, double tau_v, float* history,
                          int32_t* count, int32_t* fire, double* stats, hipStream_t stream)
{
    return launch(trigger_kernel, dim3((batch + 63) / 64), dim3(64), 0, stream, H, batch, page_steps, tau_h, tau_v, history,
                  count, fire, stats);
}

}  // namespace chess

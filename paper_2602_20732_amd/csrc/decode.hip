// Paged decode attention over a list of pages read in place (sparse: the selected page ids; dense: every
// page), split-K with an online-softmax merge; the arithmetic is in decode_device.h.
#include "decode_device.h"
#include "split_rule.h"

namespace chess {

// Workgroups dealt by length (attention over every page of a ragged batch).  A KV head has n_slots workgroups for all
// the sequences together; a sequence of t tiles takes ceil(t / u) of them, with the smallest tile count u per workgroup, of
// 64 tried, for which the slots suffice.  Lane i holds the i-th of 63 steps from "all slots equally full" to a count that
// certainly fits; the last lane's is one workgroup per sequence (the host calls with n_slots >= batch).  Every workgroup
// computes the same numbers from the lengths in device memory, so a captured launch follows them.
// A workgroup gets at least a tile per wave (u >= NW), and a sequence at most 1.5 x the count at which its own tiles and
// its merge balance (choose_splits knows the longest possible length only): split finer, 16 workgroups' partials of a
// short sequence cost more than its tiles.
// With the same number of workgroups for every sequence the longest one set the time (the waves of the others idle,
// and HBM with them): 64 sequences of 1-8192 tokens, 8 KV heads, 235 us -> 195 us dealt.
// The dealing is a chain before the first request, so it is kept short: equal lengths need no search, a search looks at
// three candidates a step (the slots needed never grow with u), and beyond 64 sequences the waves share them.  Counting all
// 64 candidates sequence by sequence in every wave took 18 us of 512 sequences' launch.  us, fixed splits / every candidate
// counted / as here:
//   8 KV heads,  16 sequences of 1024 tokens   16.4 / 18.0 / 16.3    room for 64K, 8 sequences of 1-1024   11.1 / 14.0 /  8.7
//               64 sequences of 8192 tokens   371.6 / 380.8 / 370.3
//   1 KV head,  512 sequences of 1-1024 tokens 27.4 / 52.7 / 29.7    512 sequences of 1-8192   244.7 / 240.8 / 215.9
// What remains of its cost shows where there is nothing to gain: 0.3 us with equal lengths, 0.5-1.5 us with ragged ones of
// a few tiles, 3-5 us with 512-700 of those.
struct SlotShare { int b, split, n_splits, first, len; };
struct Share { int tiles, most; };                    // of one sequence; 0, 0: a lane without one

__device__ __forceinline__ int slots_of(const Share& q, float inv_u) { return min(1 + (int)((float)(q.tiles - 1) * inv_u), q.most); }

// Inclusive sum over the lanes (row shifts and row broadcasts, no LDS); lane 63 has the total.
template <class T>
__device__ __forceinline__ T lanes_upto(T v)
{
    static_assert(sizeof(T) == 4);
#define CHESS_UPTO(ctrl, rows) v += __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, rows, 0xf, false));
    CHESS_UPTO(0x111, 0xf) CHESS_UPTO(0x112, 0xf) CHESS_UPTO(0x114, 0xf) CHESS_UPTO(0x118, 0xf) CHESS_UPTO(0x142, 0xa) CHESS_UPTO(0x143, 0xc)
#undef CHESS_UPTO
    return v;
}

template <class T>
__device__ __forceinline__ T lane_of(T v, int lane)
{
    static_assert(sizeof(T) == 4);
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// What the waves of a workgroup tell each other where a batch has more than 64 sequences.
template <int NW>
struct DealLds {
    float total[NW];
    int other[NW], c12[3][NW], c3[3][NW];
    int block[kDealMost / 64];                        // workgroups of each 64 sequences
};

template <int B, int NW>
__device__ __forceinline__ SlotShare share_slots(int slot, int n_slots, int batch, int most, int G, const int32_t* __restrict__ seq_lens,
                                                 int max_pages, int lane, int wave, DealLds<NW>& lds)
{
    const auto len_of = [&](int b) { return min(max(seq_lens[min(b, batch - 1)], 0), max_pages * B); };
    const float per_tile = 18.f / (float)G;           // (1.5 x sqrt(8 tiles / G))
    const auto share_of = [&](int b, int L) {
        const int n = max((L + kTileTokens - 1) / kTileTokens, 1);
        const int balanced = max((int)__builtin_amdgcn_sqrtf((float)n * per_tile), 1);
        return b < batch ? Share{n, min(balanced, most)} : Share{0, 0};
    };
    // up to 64 sequences: every wave has them all, one a lane.  More: a wave takes every NW-th block of 64 (the first of
    // them stays in registers, those beyond are read again for every pass, from the cache), and the sums meet in LDS.
    const bool wide = batch > 64;
    const int b00 = wide ? 64 * wave : 0, b_next = wide ? b00 + 64 * NW : batch;
    const int len0 = len_of(b00 + lane);
    const int len_first = len_of(0);
    const Share mine = share_of(b00 + lane, len0);
    const Share some = share_of(0, len_first);
    float total = (float)mine.tiles;                  // (an estimate that orders the candidates: fp32 is enough)
    int other = __ballot(mine.tiles != some.tiles && b00 + lane < batch) != 0;
    for (int b0 = b_next; b0 < batch; b0 += 64 * NW) {
        const int n = share_of(b0 + lane, len_of(b0 + lane)).tiles;
        total += (float)n;
        other |= __ballot(n != some.tiles && b0 + lane < batch) != 0;
    }
    total = lane_of(lanes_upto(total), 63);
    if (wide) {
        if (lane == 0) {
            lds.total[wave] = total;
            lds.other[wave] = other;
        }
        __syncthreads();
        total = 0.f;
        other = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            total += lds.total[w];
            other |= lds.other[w];
        }
    }
    SlotShare s = {-1, 0, 1, 0, 0};
    if (__builtin_amdgcn_readfirstlane(other) == 0) { // all as long: no search (quotients of small whole numbers: exact)
        s.n_splits = min(min((int)((float)n_slots / (float)batch), some.most), (some.tiles + NW - 1) / NW);
        const int b = (int)((float)slot / (float)s.n_splits);
        if (b < batch) {
            s.b = b;
            s.first = b * s.n_splits;
            s.split = slot - s.first;
            s.len = seq_lens[b];
        }
        return s;
    }
    const float lo = fmaxf(total / (float)n_slots, (float)NW), hi = fmaxf(total / fmaxf((float)(n_slots - batch), 1.f), lo);
    const float inv_u = lane == 63 ? 0.f : 1.f / (lo + (hi - lo) * (float)lane * (1.f / 62.f));
    int at = 0;
#pragma unroll
    for (int step = 16, i = 0; step > 0; step >>= 2, ++i) {   // the slots needed never grow with the candidate: 64 -> 16 -> 4 -> 1
        const float i1 = lane_of(inv_u, at + step - 1), i2 = lane_of(inv_u, at + 2 * step - 1), i3 = lane_of(inv_u, at + 3 * step - 1);
        // (two counts in one register: at most n_slots + batch each)
        int c12 = slots_of(mine, i1) | slots_of(mine, i2) << 16, c3 = slots_of(mine, i3);
        for (int b0 = b_next; b0 < batch; b0 += 64 * NW) {
            const Share q = share_of(b0 + lane, len_of(b0 + lane));
            c12 += slots_of(q, i1) | slots_of(q, i2) << 16;
            c3 += slots_of(q, i3);
        }
        c12 = lane_of(lanes_upto(c12), 63);
        c3 = lane_of(lanes_upto(c3), 63);
        if (wide) {
            if (lane == 0) {
                lds.c12[i][wave] = c12;
                lds.c3[i][wave] = c3;
            }
            __syncthreads();
            c12 = c3 = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                c12 += lds.c12[i][w];
                c3 += lds.c3[i][w];
            }
        }
        at += (c12 & 0xffff) <= n_slots ? 0 : (c12 >> 16) <= n_slots ? step : c3 <= n_slots ? 2 * step : 3 * step;
        at = __builtin_amdgcn_readfirstlane(at);
    }
    const float inv = lane_of(inv_u, at);             // (the last candidate always fits)
    int b0 = 0, first = 0, len = len0;
    Share own = mine;
    if (wide) {                                       // the block of 64 the slot falls in
        for (b0 = b00; b0 < batch; b0 += 64 * NW) {
            const int n = lane_of(lanes_upto(slots_of(share_of(b0 + lane, len_of(b0 + lane)), inv)), 63);
            if (lane == 0) lds.block[b0 / 64] = n;
        }
        __syncthreads();
        const int n = 64 * lane < batch ? lds.block[lane] : 0, upto = lanes_upto(n);
        const unsigned long long past = __ballot(upto > slot);
        if (past == 0) return s;
        const int j = __builtin_ctzll(past);
        b0 = 64 * j;
        first = lane_of(upto, j) - lane_of(n, j);
        len = len_of(b0 + lane);
        own = share_of(b0 + lane, len);
    }
    const int n = slots_of(own, inv), upto = first + lanes_upto(n);
    const unsigned long long past = __ballot(upto > slot);
    if (past != 0) {
        const int j = __builtin_ctzll(past);
        s.b = b0 + j;
        s.n_splits = lane_of(n, j);
        s.first = lane_of(upto, j) - s.n_splits;
        s.split = slot - s.first;
        s.len = lane_of(len, j);
    }
    return s;
}

// What the attention kernels need later than their first loads.  Those (lengths, lists, block table, queries) have their pointers and
// sizes in preloaded registers: an argument that has to be fetched is there after 1.2 us, and a length or a list asked for behind it 0.9 us
// later.  us, the pools first and loads moved behind the length / as here: reuse step, 32 layers of 1 x 32K 231.7 / 208.4, 8 layers of 32 x
// 16-32K 128.6 / 123.4; 32 layers of 4 x 24-32K and their selection 314 / 306; every page 461 / 461.  Numbers, not pointers: see step.hip.
struct DecodeArgs {
    uint16_t* k_pool;        // (written by the reuse kernel only, as v_pool)
    uint16_t* v_pool;
    float* out;
    float* ws_acc;
    float* ws_ml;
    int32_t* arrivals;
    float scale_log2;
    int batch;
    const uint16_t* k_new;   // reuse
    const uint16_t* v_new;
};
using DecodeKernel = void (*)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, int, int, int, int, DecodeArgs);   // (the launchers' tables hold the kernels to it)
using DecodeLines = ArgLinesOf<DecodeKernel, DecodeArgs>;
// What stands before is requested before what stands behind (the compiler moves a load that only a branch uses into the branch).
__device__ __forceinline__ void requested_by_here() { asm volatile("" : : : "memory"); }

// Three workgroups of four waves per compute unit (at most 170 registers a lane): see run_tiles_with, kSingle.
// One sequence's every page of 32: within the registers of four.  With 136 of them the compiler asks for a tile's value rows ahead of its
// first product and not behind it, and the few workgroups there are, which wait for their rows tile by tile, take longer: us, one KV head,
// 131072 tokens, G = 1 / 4 / 7 / 16: 26.2 / 30.3 / 39.9 / 55.7 with 136 registers, 25.3 / 28.7 / 37.0 / 50.7 so.
// heads: KV heads << 8 | group.
template <int B, int NW, bool kList, bool kDealt = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(B == 32 && NW == 4 && !kList && !kDealt ? 4 : 3))) void decode_kernel(uint64_t seq_lens_at, uint64_t block_table_at, uint64_t q_at,
                                                         uint64_t page_ids_at, uint64_t n_selected_at, int heads, int max_sel, int max_pages,
                                                         int n_splits, DecodeArgs a)
{
    constexpr int PPT = 32 / B;
    extern __shared__ float lds_f[];                  // DecodeLds<NW>::floats(G)
    __shared__ int lds_last;
    const int G = heads & 255, H = heads >> 8, h = kDealt ? blockIdx.x : blockIdx.y;
    DecodeLines lines;
    lines.ask();
    DecodeLds<NW> lds(lds_f, G);
    const int32_t* seq_lens = device_pointer<const int32_t>(seq_lens_at);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m16 = lane & 15, grp = lane >> 4;
    // the workgroup's sequence, its place among that row's splits, and where the row's partials start
    int split = blockIdx.x, b = blockIdx.z, ns = n_splits, L_raw;
    size_t part0 = ((size_t)b * H + h) * n_splits;
    if constexpr (kDealt) {                           // grid = (H_kv, n_slots): the heads of a page are read at about the same time
        __shared__ DealLds<NW> deal_lds;
        const SlotShare sh = share_slots<B, NW>(blockIdx.y, gridDim.y, a.batch, n_splits, G, seq_lens, max_pages, lane, wave, deal_lds);
        if (sh.b < 0) return;                         // (uniform: nobody waits for a slot without work)
        split = sh.split;
        b = sh.b;
        ns = sh.n_splits;
        L_raw = sh.len;
        part0 = (size_t)h * gridDim.y + sh.first;
    }
    const size_t row = (size_t)b * H + h;
    const int32_t* ids = kList ? device_pointer<const int32_t>(page_ids_at) + row * max_sel : nullptr;
    const int32_t* bt_row = device_pointer<const int32_t>(block_table_at) + (size_t)b * max_pages;
    // tiles are dealt round-robin: tile = split + n_splits * (wave + NW * i), so the first tile of a wave
    // is known before the list length is, and its page numbers can be fetched alongside the lengths
    const int stride = ns * NW;
    const int t = split + ns * wave;
    int raw_cur[PPT], raw_nxt[PPT];
    if constexpr (!kDealt) L_raw = load_by_lane(seq_lens + b);
    int n_raw = kList ? load_by_lane(device_pointer<const int32_t>(n_selected_at) + row) : 0;
    fetch_ids<B, kList>(raw_cur, t, ids, max_sel);
    fetch_ids<B, kList>(raw_nxt, t + stride, ids, max_sel);
    WaveAcc<B> acc;
    acc.request(device_pointer<const uint16_t>(q_at) + ((size_t)b * H * G + (size_t)h * G) * kHeadDim, G, m16, grp);
    requested_by_here();
    if constexpr (!kDealt) L_raw = __builtin_amdgcn_readfirstlane(L_raw);
    if (kList) n_raw = __builtin_amdgcn_readfirstlane(n_raw);
    const int L = min(max(L_raw, 0), max_pages * B);
    const int P = (L + B - 1) / B;
    const int n_pages = P == 0 ? 0 : (kList ? min(max(n_raw, 0), max_sel) : P);
    const int n_tiles = (n_pages + PPT - 1) / PPT;

    lines.hold();
    acc.start(G, m16);
    NewToken<B> none;
    none.tile = -1;
    run_tiles_with<B, kList, false, false, true>(acc, t, stride, n_tiles, n_pages, raw_cur, raw_nxt, ids, max_sel, bt_row, nullptr,
                                                 a.k_pool, a.v_pool, H, h, L, P, a.scale_log2, m16, grp, none, 1 << 30);

    float* out_rows = a.out + ((size_t)b * H * G + (size_t)h * G) * kHeadDim;
    if (!combine_waves<NW>(acc.o, acc.m_run, acc.l_run, lds, G, ns, split, part0, out_rows, a.ws_acc, a.ws_ml)) return;
    if (!arrive_last(a.arrivals + row * kArrivalStride, ns, &lds_last)) return;
    if constexpr (kDealt) {                           // (the same in every lane, which the compiler cannot tell)
        ns = own_reg(__builtin_amdgcn_readfirstlane(ns));
        part0 = own_reg((unsigned)__builtin_amdgcn_readfirstlane((int)part0));
    }
    merge_splits<NW, kDealt ? kMergeDealt : kMergePlain>(G, ns, part0, out_rows, a.ws_acc, a.ws_ml);
}

// The step between reselections (Sec. 3.3) in one launch: attention over the kept list for the sequence WITH the
// token that is being appended, whose key / value rows are not in the pools yet.  Every split takes them from
// k_new / v_new straight into the operands of the tile that holds the tail page; the last split of a (sequence,
// KV head) to finish -- after which nobody reads the tail page or the list any more -- writes the rows to the pools
// and, when the token opens a new page, the page to the list.  The lists must end with the tail page of seq_lens
// (as a selection on these lengths, chess_append_kv with the lists, or this call leave them).
// grid = (n_splits, H_kv, batch), NW waves (4 or 8: see split_rule.h).
// kSingle: one tile in registers at a time; faster while a wave has only a few tiles (the host decides).
// Two workgroups per compute unit either way (squeezed into the registers of three, the kernel was slower).
template <int B, bool kSingle, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void reuse_kernel(uint64_t seq_lens_at, uint64_t block_table_at, uint64_t q_at,
                                                    uint64_t page_ids_at, uint64_t n_selected_at, int heads, int max_sel, int max_pages,
                                                    int n_splits, DecodeArgs a)
{
    constexpr int PPT = 32 / B;
    extern __shared__ float lds_f[];
    __shared__ int lds_last;
    const int G = heads & 255, H = heads >> 8;
    DecodeLines lines;
    lines.ask();
    DecodeLds<NW> lds(lds_f, G);

    const int split = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m16 = lane & 15, grp = lane >> 4;
    const size_t row = (size_t)b * H + h;
    int32_t* ids = device_pointer<int32_t>(page_ids_at) + row * max_sel;
    int32_t* n_selected = device_pointer<int32_t>(n_selected_at) + row;
    const int32_t* bt_row = device_pointer<const int32_t>(block_table_at) + (size_t)b * max_pages;
    const int stride = n_splits * NW;
    const int t = split + n_splits * wave;
    int raw_cur[PPT], raw_nxt[PPT];
    int L_before = load_by_lane(device_pointer<const int32_t>(seq_lens_at) + b);
    int n_raw = load_by_lane(n_selected);
    fetch_ids<B, true>(raw_cur, t, ids, max_sel);
    fetch_ids<B, true>(raw_nxt, t + stride, ids, max_sel);
    WaveAcc<B> acc;
    acc.request(device_pointer<const uint16_t>(q_at) + ((size_t)b * H * G + (size_t)h * G) * kHeadDim, G, m16, grp);
    requested_by_here();
    L_before = __builtin_amdgcn_readfirstlane(L_before);
    n_raw = __builtin_amdgcn_readfirstlane(n_raw);
    lines.hold();
    NewToken<B> nt;
    nt.k_row = a.k_new + row * kHeadDim;
    nt.v_row = a.v_new + row * kHeadDim;

    const bool room = L_before >= 0 && L_before < max_pages * B;
    const int L = room ? L_before + 1 : min(max(L_before, 0), max_pages * B);
    const int P = (L + B - 1) / B;
    const int n_stored = min(max(n_raw, 0), max_sel);
    const bool grow = room && L_before % B == 0 && n_stored < max_sel;       // the token opens a page
    const int n_pages = P == 0 ? 0 : n_stored + (grow ? 1 : 0);
    const int n_tiles = (n_pages + PPT - 1) / PPT;
    // the tail page is the list's last entry -- unless the token opens a page and the row has no room for it: then
    // (and in the steps after: run_tiles_with looks at the entry) the token is stored but not attended, as with
    // chess_append_kv + chess_sparse_decode
    nt.tile = room && n_pages > 0 && (grow || L_before % B != 0) ? (n_pages - 1) / PPT : -1;
    nt.T = ((n_pages - 1) % PPT) * B + L_before % B;

    // what the last split to finish stores, and where: asked for ahead of the rows (behind the last arrival it was two round trips, 0.6 us)
    const int dim = min((int)threadIdx.x, kHeadDim - 1), page = room ? L_before / B : 0;
    const uint16_t k_tok = nt.k_row[dim], v_tok = nt.v_row[dim];
    const int tok_phys = load_by_lane(bt_row + page);

    acc.start(G, m16);
    run_tiles_with<B, true, false, true, kSingle>(acc, t, stride, n_tiles, n_pages, raw_cur, raw_nxt, ids, max_sel, bt_row, nullptr, a.k_pool,
                                         a.v_pool, H, h, L, P, a.scale_log2, m16, grp, nt, n_stored);

    float* out_rows = a.out + ((size_t)b * H * G + (size_t)h * G) * kHeadDim;
    const bool split_up = combine_waves<NW>(acc.o, acc.m_run, acc.l_run, lds, G, n_splits, split, row * n_splits, out_rows, a.ws_acc, a.ws_ml);
    if (split_up && !arrive_last(a.arrivals + row * kArrivalStride, n_splits, &lds_last)) return;
    // every split of the row is past its reads: the token and the page go where the next step looks for them
    if (room) {
        if (threadIdx.x < kHeadDim) {
            const size_t blk = ((size_t)__builtin_amdgcn_readfirstlane(tok_phys) * H + h) * B * kHeadDim;
            const int tok = L_before % B;
            a.k_pool[blk + (size_t)tok * kHeadDim + dim] = k_tok;
            a.v_pool[blk + (size_t)dim * B + tok] = v_tok;
        }
        if (grow && threadIdx.x == 0) {
            ids[n_stored] = P - 1;
            *n_selected = n_stored + 1;
        }
    }
    if (split_up) merge_splits<NW, kMergePlain>(G, n_splits, row * n_splits, out_rows, a.ws_acc, a.ws_ml);
}

hipError_t launch_reuse(chess_ctx* ctx, const uint16_t* q, const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool,
                        uint16_t* v_pool, const int32_t* block_table, const int32_t* seq_lens, int32_t* page_ids,
                        int32_t* n_selected, int batch, int n_splits, int waves, float* out, float* ws_acc, float* ws_ml,
                        int32_t* arrivals, hipStream_t stream)
{
    const Geom& g = ctx->geom;
    const float scale_log2 = ctx->sm_scale * 1.4426950408889634f;
    const int nw = waves == 8 ? 8 : 4;
    const dim3 grid(n_splits, g.n_kv_heads, batch), block(64 * nw);
    const size_t lds = (size_t)(nw * g.group * kHeadDim + 2 * nw * g.group) * sizeof(float);
    // without the prefetch of the next tile while a wave has at most four tiles of the longest possible list
    const int tiles = (g.max_sel + kTileTokens / g.page_size - 1) / (kTileTokens / g.page_size);
    const int single = tiles <= 4 * nw * n_splits;
    // [page size 16 / 32][waves 4 / 8][prefetch / single]
    static const DecodeKernel table[2][2][2] = {
        {{reuse_kernel<16, false, 4>, reuse_kernel<16, true, 4>}, {reuse_kernel<16, false, 8>, reuse_kernel<16, true, 8>}},
        {{reuse_kernel<32, false, 4>, reuse_kernel<32, true, 4>}, {reuse_kernel<32, false, 8>, reuse_kernel<32, true, 8>}}};
    const DecodeKernel kern = table[g.page_size == 16 ? 0 : 1][nw == 8][single];
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return launch(kern, grid, block, lds, stream, (uint64_t)seq_lens, (uint64_t)block_table, (uint64_t)q, (uint64_t)page_ids, (uint64_t)n_selected,
                  g.n_kv_heads << 8 | g.group, g.max_sel, g.max_pages, n_splits,
                  DecodeArgs{k_pool, v_pool, out, ws_acc, ws_ml, arrivals, scale_log2, batch, k_new, v_new});
}

hipError_t launch_decode(chess_ctx* ctx, const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool,
                         const int32_t* block_table, const int32_t* seq_lens, const int32_t* page_ids,
                         const int32_t* n_selected, int batch, int n_splits, int waves, int n_slots, float* out,
                         float* ws_acc, float* ws_ml, int32_t* arrivals, hipStream_t stream)
{
    const Geom& g = ctx->geom;
    const float scale_log2 = ctx->sm_scale * 1.4426950408889634f;
    const bool dealt = n_slots > 0;                   // (every page, four waves: see choose_splits)
    const dim3 grid = dealt ? dim3(g.n_kv_heads, n_slots) : dim3(n_splits, g.n_kv_heads, batch), block(64 * waves);
    const size_t lds = (size_t)(waves * g.group * kHeadDim + 2 * waves * g.group) * sizeof(float);
    // [page size 16 / 32][waves 4 / 1][list / every page], eight waves for a list, every page dealt by length
    static const DecodeKernel table[2][2][2] = {
        {{decode_kernel<16, 4, true>, decode_kernel<16, 4, false>}, {decode_kernel<16, 1, true>, decode_kernel<16, 1, false>}},
        {{decode_kernel<32, 4, true>, decode_kernel<32, 4, false>}, {decode_kernel<32, 1, true>, decode_kernel<32, 1, false>}}};
    static const DecodeKernel wide[2] = {decode_kernel<16, 8, true>, decode_kernel<32, 8, true>};
    static const DecodeKernel by_length[2] = {decode_kernel<16, 4, false, true>, decode_kernel<32, 4, false, true>};
    const int by_page = g.page_size == 16 ? 0 : 1;
    const DecodeKernel kern = dealt ? by_length[by_page] : waves == 8 ? wide[by_page] : table[by_page][waves == 4 ? 0 : 1][page_ids ? 0 : 1];
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return launch(kern, grid, block, lds, stream, (uint64_t)seq_lens, (uint64_t)block_table, (uint64_t)q, (uint64_t)page_ids, (uint64_t)n_selected,
                  g.n_kv_heads << 8 | g.group, g.max_sel, g.max_pages, n_splits,
                  DecodeArgs{const_cast<uint16_t*>(k_pool), const_cast<uint16_t*>(v_pool), out, ws_acc, ws_ml, arrivals, scale_log2, batch, nullptr, nullptr});
}

// Four-wave workgroups of attention over every page that fit on a compute unit, dealt or not, whichever are fewer (lists
// go by the number of compute units alone).
hipError_t dense_occupancy(int page_size, int group, int* blocks_per_cu)
{
    const size_t lds = (size_t)(4 * group * kHeadDim + 2 * 4 * group) * sizeof(float);
    int fixed = 0, dealt = 0;
    hipError_t e = page_size == 16 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&fixed, decode_kernel<16, 4, false>, 256, lds)
                                   : hipOccupancyMaxActiveBlocksPerMultiprocessor(&fixed, decode_kernel<32, 4, false>, 256, lds);
    if (e != hipSuccess) return e;
    e = page_size == 16 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&dealt, decode_kernel<16, 4, false, true>, 256, lds)
                        : hipOccupancyMaxActiveBlocksPerMultiprocessor(&dealt, decode_kernel<32, 4, false, true>, 256, lds);
    if (e != hipSuccess) return e;
    *blocks_per_cu = fixed < dealt ? fixed : dealt;
    return hipSuccess;
}

// One new token per sequence into the paged pools: K row-major [phys][H][B][128], V token-minor [phys][H][128][B].
// grid = batch * H_kv workgroups of 128 threads, thread = dim.
__global__ __launch_bounds__(kHeadDim) void append_kernel(const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new,
                                                          uint16_t* __restrict__ k_pool, uint16_t* __restrict__ v_pool,
                                                          const int32_t* __restrict__ block_table,
                                                          const int32_t* __restrict__ seq_lens, Geom g,
                                                          int32_t* __restrict__ page_ids, int32_t* __restrict__ n_selected)
{
    const int row = blockIdx.x, b = row / g.n_kv_heads, h = row - b * g.n_kv_heads, dim = threadIdx.x;
    const int L = seq_lens[b], B = g.page_size;
    if (L < 0 || L >= g.max_pages * B) return;        // no room: the sequence is left as it is
    if (page_ids != nullptr && dim == 0) {            // the row's list follows the tail (what extend_kernel does)
        const int P = L / B + 1;                      // pages once the token is in
        int32_t* ids = page_ids + (size_t)row * g.max_sel;
        int n = min(max(n_selected[row], 0), g.max_sel);
        int last = n > 0 ? ids[n - 1] : -1;
        while (last < P - 1 && n < g.max_sel) ids[n++] = ++last;
        n_selected[row] = n;
    }
    const int64_t phys = block_table[(size_t)b * g.max_pages + L / B];
    const int t = L % B;
    const size_t blk = ((size_t)phys * g.n_kv_heads + h) * B * kHeadDim;
    k_pool[blk + (size_t)t * kHeadDim + dim] = k_new[(size_t)row * kHeadDim + dim];
    v_pool[blk + (size_t)dim * B + t] = v_new[(size_t)row * kHeadDim + dim];
}

hipError_t launch_append(chess_ctx* ctx, const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool, uint16_t* v_pool,
                         const int32_t* block_table, const int32_t* seq_lens, int batch, int32_t* page_ids,
                         int32_t* n_selected, hipStream_t stream)
{
    return launch(append_kernel, dim3(batch * ctx->geom.n_kv_heads), dim3(kHeadDim), 0, stream, k_new, v_new, k_pool, v_pool,
                  block_table, seq_lens, ctx->geom, page_ids, n_selected);
}

// Between reselections the recent window follows the tail: every list is extended by the pages after its last
// entry, up to the sequence's current last page (as far as the row has room).  One thread per (sequence, KV head).
__global__ void extend_kernel(const int32_t* __restrict__ seq_lens, int rows, Geom g, int32_t* __restrict__ page_ids,
                              int32_t* __restrict__ n_selected)
{
    const int row = blockIdx.x * blockDim.x + threadIdx.x;
    if (row >= rows) return;
    const int L = min(max(seq_lens[row / g.n_kv_heads], 0), g.max_pages * g.page_size);
    const int P = (L + g.page_size - 1) / g.page_size;
    int32_t* ids = page_ids + (size_t)row * g.max_sel;
    int n = min(max(n_selected[row], 0), g.max_sel);
    int last = n > 0 ? ids[n - 1] : -1;
    while (last < P - 1 && n < g.max_sel) ids[n++] = ++last;
    n_selected[row] = n;
}

hipError_t launch_extend(chess_ctx* ctx, const int32_t* seq_lens, int batch, int32_t* page_ids, int32_t* n_selected,
                         hipStream_t stream)
{
    const int rows = batch * ctx->geom.n_kv_heads;
    return launch(extend_kernel, dim3((rows + 63) / 64), dim3(64), 0, stream, seq_lens, rows, ctx->geom, page_ids, n_selected);
}

__global__ void zero_kernel(int32_t* p, size_t n, int stride)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i * stride] = 0;
}

hipError_t launch_zero(chess_ctx* ctx, int32_t* p, size_t n_words, int stride, hipStream_t stream)
{
    (void)ctx;
    return launch(zero_kernel, dim3((unsigned)((n_words + 255) / 256)), dim3(256), 0, stream, p, n_words, stride);
}

}  // namespace chess

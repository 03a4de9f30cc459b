// Tenant segmentation and grouped-work descriptors (see mt_device.h for the overview).
#include "mt_device.h"
#include <type_traits>

namespace mt {

// Index of the segment that holds submission row r (segments are sorted by row_begin).
__device__ __forceinline__ uint32_t find_segment(const Segment* segs, uint32_t n, uint32_t r)
{
    uint32_t lo = 0, hi = n;            // invariant: segs[lo].row_begin <= r
    while (hi - lo > 1) {
        uint32_t mid = (lo + hi) >> 1;
        if (segs[mid].row_begin <= r) lo = mid; else hi = mid;
    }
    return lo;
}

// Exclusive scan of data[0..n) in LDS by the whole workgroup (n <= kMaxTenantsPadded);
// returns the total.  tmp must hold 17 words.
__device__ uint32_t block_exclusive_scan(uint32_t* data, uint32_t n, uint32_t* tmp)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t ipt = ceil_div(n, kBatchThreads);
    const uint32_t begin = tid * ipt, end = min(begin + ipt, n);
    static_assert(kBatchThreads / 64 == 16, "the wave totals are one row of 16 lanes");
    uint32_t s = 0;
    for (uint32_t i = begin; i < end; ++i) s += data[i];
    const uint32_t incl = wave_inclusive_scan(s);
    if (lane == 63) tmp[w] = incl;
    __syncthreads();
    if (w == 0) {
        const uint32_t c = lane < 16 ? tmp[lane] : 0;
        const uint32_t inc = row16_inclusive_scan(c);
        if (lane < 16) tmp[lane] = inc - c;
        if (lane == 15) tmp[16] = inc;
    }
    __syncthreads();
    uint32_t run = tmp[w] + incl - s;
    for (uint32_t i = begin; i < end; ++i) { uint32_t c = data[i]; data[i] = run; run += c; }
    uint32_t total = tmp[16];
    __syncthreads();
    return total;
}

// Placement pass for large batches (after rank_kernel and the batcher): one row per thread;
// position = the tenant's first row + rows of the tenant in earlier ranking workgroups + rank.
__global__ __launch_bounds__(kBatchThreads) void place_kernel(BatchArgs a)
{
    const uint32_t r = blockIdx.x * kRankRows + threadIdx.x;
    if (r >= a.R) return;
    uint32_t Tp = 64;
    while (Tp < a.T) Tp <<= 1;
    const int32_t t = a.row_tenant[r];
    place_row(a, r, t, t >= 0 ? a.off[t] + a.hist_g[blockIdx.x * Tp + t] + a.row_rank[r] : 0);
}

// Ranking pass for large batches, spread over the chip: workgroup g takes rows
// [g * kRankRows, (g + 1) * kRankRows), one per thread.  Equal tenants inside a wave are matched
// with ballots as in the batcher; the 16 waves' counts are combined in wave order, so a row's
// rank counts the earlier rows of its tenant in the workgroup (arrival order is kept).
template <bool ONE_SEG>
__global__ __launch_bounds__(kBatchThreads) void rank_kernel(BatchArgs a)
{
    static_assert(kRankRows == (int)kBatchThreads, "one row per thread");
    __shared__ uint32_t whist[(kBatchThreads / 64) * kRankMaxTenants];
    __shared__ Segment seg_l[kSegsInLds];
    const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t T = a.T, R = a.R, r = blockIdx.x * kRankRows + tid;
    uint32_t Tp = 64;
    while (Tp < T) Tp <<= 1;
    const uint32_t bits = T > 1 ? 32 - __builtin_clz(T - 1) : 0;
    const Segment* segs = a.segs;
    if (!ONE_SEG && a.n_segs <= kSegsInLds) {
        for (uint32_t i = tid; i < a.n_segs; i += kBatchThreads) seg_l[i] = a.segs[i];
        segs = seg_l;
    }
    for (uint32_t i = tid; i < (kBatchThreads / 64) * Tp; i += kBatchThreads) whist[i] = 0;
    __syncthreads();
    int32_t t = -1;
    if (r < R) {
        if (ONE_SEG) {
            a.row_src[r] = (const uint8_t*)a.first.src + (size_t)r * a.first.row_stride * a.elem_size;
            t = a.first.ids ? a.first.ids[r] : a.first.tenant;
        } else {
            const Segment& sg = segs[find_segment(segs, a.n_segs, r)];
            a.row_src[r] = (const uint8_t*)sg.src + (size_t)(r - sg.row_begin) * sg.row_stride * a.elem_size;
            t = sg.ids ? sg.ids[r - sg.row_begin] : sg.tenant;
        }
        if (t < 0 || (uint32_t)t >= T || !serves(a, a.tenants[t])) t = -1;
        a.row_tenant[r] = t;
    }
    uint64_t peers = __ballot(t >= 0);
    for (uint32_t b = 0; b < bits; ++b) {
        const bool bit = (t >> b) & 1;
        const uint64_t m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    const uint32_t rank = __popcll(peers & ((1ull << lane) - 1));
    if (t >= 0 && rank == 0) whist[w * Tp + t] = __popcll(peers);        // the first of its tenant in this wave
    __syncthreads();
    for (uint32_t u = tid; u < Tp; u += kBatchThreads) {
        uint32_t cnt[kBatchThreads / 64];
#pragma unroll
        for (uint32_t i = 0; i < kBatchThreads / 64; ++i) cnt[i] = whist[i * Tp + u];
        uint32_t run = 0;
#pragma unroll
        for (uint32_t i = 0; i < kBatchThreads / 64; ++i) { whist[i * Tp + u] = run; run += cnt[i]; }
        a.hist_g[blockIdx.x * Tp + u] = run;
    }
    __syncthreads();
    if (t >= 0) a.row_rank[r] = whist[w * Tp + t] + rank;
}

// Tenant segmentation and grouped-work descriptors.  One workgroup; every step is deterministic: rows of a tenant keep their
// arrival order (stable counting sort).  Equal tenant ids inside a wavefront are found with one ballot per id bit, so a step
// costs the same whatever the tenant mix is.  Latency, not bandwidth, bounds this kernel, so everything that does not depend on the
// rows (tenant and layer facts) is fetched up front, and waves wait for each other as little as possible: with at most
// 64 tenants every wave holds all of them in its lanes and works out totals and offsets for itself (two barriers in the whole
// kernel, a third where big tiles are possible), and a tile list belongs to one wave.
// Kernel trace, this form against one whose 1024 threads were the tenants and built the lists of eight layer indices
// at a time with three barriers per eight: 1 request to 8 three-layer models 7.8 -> 4.0 us, 4096 requests to 64 of
// them 13.0 -> 10.6, 1 request to 26-layer models 20.4 -> 5.8, behind the ranking kernel (32768 rows, 8 tenants) 13.9 -> 6.1.
// Many tenants, three layers, 256 / 4096 / 16384 requests: 256 tenants 11.0 -> 8.8 / 15.6 -> 13.2 / 20.0 -> 15.5 (three kernels), 1024 15.1 -> 12.4 /
// 33.2 -> 29.0 / 53.2 -> 49.8, 2048 25.0 -> 19.2 / 58.3 -> 51.0 / 118.1 -> 108.9; thirteen layers, 2048 tenants 38.2 -> 28.6 / 70.5 -> 70.1 /
// 132.4 -> 122.4.  (Lists walked 64 tenants at a time, facts of a tenant's layers side by side, rows placed by the waves that
// ranked them: 29.3 / 64.8 / 150.1, thirteen layers 45.0 / 84.9 / 152.5.)
// ITERS: rows a lane may keep in registers (64 * ITERS rows per wave); the launcher picks the smallest
// instantiation that covers the batch, because the unrolled steps of a larger one cost small batches microseconds.
template <bool ONE_SEG, int ITERS, bool PRE = false>
__global__ __launch_bounds__(kBatchThreads) void batcher_kernel(BatchArgs a)
{
    constexpr uint32_t kWaves = kBatchThreads / 64;
    __shared__ uint32_t hist[kHistEntries];
    __shared__ __attribute__((aligned(16))) uint32_t Ml[kMaxTenantsPadded];
    __shared__ uint32_t offl[kMaxTenantsPadded];
    __shared__ uint8_t regl[kMaxTenantsPadded];
    __shared__ uint32_t tmp[17];
    __shared__ Segment seg_l[kSegsInLds];
    __shared__ uint32_t big_l;                         // layer indices served with big tiles

    const uint32_t tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t T = a.T, R = a.R;
    uint32_t Tp = 64;
    while (Tp < T) Tp <<= 1;
    const bool one_wave = Tp == 64;                    // every tenant has a lane: no tables in LDS
    const uint32_t bits = T > 1 ? 32 - __builtin_clz(T - 1) : 0;      // valid ids are below T
    constexpr uint32_t kRegIters = ITERS;

    // Every global load the kernel depends on is issued before the first wait: the segment table (it
    // sits in host memory; staged in LDS when it is small), the lane's tenant ids of a batch that is one
    // submission, the tenant facts and the first layer facts of this wave's tile lists.
    // PRE: the rows were ranked by rank_kernel; its workgroups stand where the waves stand otherwise
    const Segment* segs = a.segs;
    if (!ONE_SEG && a.n_segs <= kSegsInLds) {
        for (uint32_t i = tid; i < a.n_segs; i += kBatchThreads) seg_l[i] = a.segs[i];
        segs = seg_l;
    }
    const uint32_t nw = PRE ? a.n_rank_groups : min(kWaves, (uint32_t)kHistEntries / Tp);
    const uint32_t chunk = PRE ? (uint32_t)kRankRows : ceil_div(ceil_div(R, nw), 64) * 64;          // rows per wave
    const bool in_regs = !PRE && chunk <= 64 * kRegIters;                // a lane keeps its rows' ids and ranks in registers
    const uint32_t begin = w * chunk, end = w < nw ? min(begin + chunk, R) : begin;
    int32_t tq[kRegIters];               // first the submitted id, then rank << 11 | tenant (or -1): ids and in-wave ranks are below 2048
    static_assert(kMaxTenantsPadded <= 2048 && 64 * kRegIters <= (1u << 21), "packing of tenant and rank");
    // the submitted id of row r (also notes where its input lies)
    auto fetch_id = [&](uint32_t r) -> int32_t {
        if (r >= end) return -1;
        if (ONE_SEG) {                          // the whole batch is one submission: no table lookup
            a.row_src[r] = (const uint8_t*)a.first.src + (size_t)r * a.first.row_stride * a.elem_size;
            return a.first.ids ? a.first.ids[r] : a.first.tenant;
        }
        const Segment& sg = segs[find_segment(segs, a.n_segs, r)];
        a.row_src[r] = (const uint8_t*)sg.src + (size_t)(r - sg.row_begin) * sg.row_stride * a.elem_size;
        return sg.ids ? sg.ids[r - sg.row_begin] : sg.tenant;
    };
    if (ONE_SEG && in_regs) {
#pragma unroll
        for (uint32_t it = 0; it < kRegIters; ++it) tq[it] = fetch_id(begin + it * 64 + lane);
    }
    // The tile lists of layer index l (three kinds) belong to wave l % 16, which walks them 64 tenants at a time, or 256
    // (four neighbours a lane) where there are more than 64.  A step needs the fact words of its tenant-layers
    // (BatchArgs::facts); those of the wave's first steps are fetched here: four layer indices of up to 64 tenants, or 256 tenants of one.
    constexpr uint32_t kPre = 4;
    static_assert(MT_MAX_LAYERS <= kPre * kWaves, "with at most 64 tenants, every step of a wave is fetched ahead");
    auto load_fact = [&](uint32_t l, uint32_t t) -> uint4 {
        return l < a.n_layer_slots && t < T ? ((const uint4*)a.facts)[(size_t)l * T + t] : uint4{0, 0, 0, 0};
    };
    uint4 fq[kPre];
#pragma unroll
    for (uint32_t i = 0; i < kPre; ++i) fq[i] = one_wave ? load_fact(w + i * kWaves, lane) : load_fact(w, lane * kPre + i);
    for (uint32_t t = tid; t < Tp; t += kBatchThreads) regl[t] = t < T && serves(a, a.tenants[t]);
    for (uint32_t i = tid; i < nw * Tp; i += kBatchThreads) hist[i] = PRE ? a.hist_g[i] : 0;
    if (tid == 0) big_l = 0;
    __syncthreads();

    // pass 1: per-wave histograms and in-wave ranks.  One step ranks 64 rows: equal tenant ids
    // are matched with one ballot per id bit.
    auto rank_step = [&](int32_t& t, uint32_t& rank_out) {
        if (t < 0 || (uint32_t)t >= T || !regl[t]) t = -1;
        uint64_t peers = __ballot(t >= 0);
        for (uint32_t b = 0; b < bits; ++b) {
            const bool bit = (t >> b) & 1;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const bool ok = t >= 0;
        const uint32_t leader = ok ? (uint32_t)__ffsll((unsigned long long)peers) - 1 : lane;
        const uint32_t rank = __popcll(peers & ((1ull << lane) - 1));
        uint32_t old = 0;
        if (ok && lane == leader) {
            old = hist[w * Tp + t];
            hist[w * Tp + t] = old + __popcll(peers);
        }
        old = __shfl(old, leader);
        rank_out = old + rank;
    };
    if (in_regs) {
#pragma unroll
        for (uint32_t it = 0; it < kRegIters; ++it) {
            if (begin + it * 64 < end) {                     // wave-uniform
                const uint32_t r = begin + it * 64 + lane;
                if (!ONE_SEG) tq[it] = fetch_id(r);
                uint32_t rank;
                rank_step(tq[it], rank);
                if (r < end) a.row_tenant[r] = tq[it];
                if (tq[it] >= 0) tq[it] |= (int32_t)(rank << 11);
            } else if (!ONE_SEG) tq[it] = -1;
        }
    } else if (!PRE && w < nw) {
        int32_t t_next = begin < end ? fetch_id(begin + lane) : -1;
        for (uint32_t base = begin; base < end; base += 64) {
            const uint32_t r = base + lane;
            int32_t t = t_next;
            if (base + 64 < end) t_next = fetch_id(r + 64);
            uint32_t rank;
            rank_step(t, rank);
            if (r < end) { a.row_tenant[r] = t; if (t >= 0) a.row_rank[r] = rank; }
        }
    }
    if (!PRE) __syncthreads();

    // pass 2: per-tenant totals, per-wave bases, tenant offsets (each tenant starts a 32-row block)
    uint32_t Mt1 = 0, base1 = 0;                       // one_wave: lane t holds tenant t's total, and where this wave's rows of it begin
    auto publish = [&](uint32_t t, uint32_t Mt, uint32_t off) {
        a.M[t] = Mt; a.off[t] = off;
        if (Mt) { atomicAdd(&a.served[2 * t], (unsigned long long)Mt); atomicAdd(&a.served[2 * t + 1], 1ull); }
    };
    auto pad_rows = [&](uint32_t Mt, uint32_t off) {   // padding rows of a tenant's last block
        const uint32_t pend = off + ceil_div(Mt, kBrickRows) * kBrickRows;
        for (uint32_t p = off + Mt; p < pend; ++p) a.perm[p] = -1;
    };
    if (one_wave) {
        uint32_t before = 0;
        for (uint32_t i0 = 0; i0 < nw; i0 += 16) {            // 16 reads in flight together
            uint32_t cnt[16];
#pragma unroll
            for (uint32_t i = 0; i < 16; ++i) cnt[i] = i0 + i < nw ? hist[(i0 + i) * 64 + lane] : 0;
#pragma unroll
            for (uint32_t i = 0; i < 16; ++i) {
                if (PRE && i == w && i0 + i < nw) a.hist_g[(i0 + i) * 64 + lane] = Mt1;      // prefix over the ranking workgroups, for place_kernel
                if (!PRE && i0 + i == w) before = Mt1;
                Mt1 += cnt[i];
            }
        }
        const uint32_t padded = ceil_div(Mt1, kBrickRows) * kBrickRows, incl = wave_inclusive_scan(padded), off = incl - padded;
        base1 = off + before;
        if (w == 0) {
            if (lane < T) publish(lane, Mt1, off);
            if (lane == 63) a.off[T] = incl;
        } else if (w == 1) {
            if (lane < T) pad_rows(Mt1, off);
        }
    } else {
        for (uint32_t t = tid; t < Tp; t += kBatchThreads) {
            uint32_t s = 0;
            for (uint32_t i0 = 0; i0 < nw; i0 += 16) {            // 16 reads in flight together
                uint32_t cnt[16];
#pragma unroll
                for (uint32_t i = 0; i < 16; ++i) cnt[i] = i0 + i < nw ? hist[(i0 + i) * Tp + t] : 0;
#pragma unroll
                for (uint32_t i = 0; i < 16; ++i) { if (i0 + i < nw) hist[(i0 + i) * Tp + t] = s; s += cnt[i]; }
            }
            Ml[t] = s; offl[t] = ceil_div(s, kBrickRows) * kBrickRows;
        }
        __syncthreads();
        const uint32_t total = block_exclusive_scan(offl, Tp, tmp);
        for (uint32_t t = tid; t < T; t += kBatchThreads) { publish(t, Ml[t], offl[t]); pad_rows(Ml[t], offl[t]); }
        if (tid == 0) a.off[T] = total;
        if (PRE) for (uint32_t i = tid; i < nw * Tp; i += kBatchThreads) a.hist_g[i] = hist[i];
    }

    // pass 3: packed position of every row (pre-ranked batches: place_kernel, from the prefixes
    // over the ranking workgroups that were handed back above); a wave places the rows it ranked
    auto place = [&](uint32_t r, int32_t t, uint32_t rank) {
        const uint32_t tl = t >= 0 ? (uint32_t)t : 0;
        const uint32_t base = one_wave ? (uint32_t)__shfl((int)base1, (int)(tl & 63)) : offl[tl] + hist[w * Tp + tl];
        if (r < end) place_row(a, r, t, base + rank);
    };
    // (unless most waves ranked none: with more than 512 tenants the histograms leave room for eight or four of the sixteen)
    if (in_regs) {
#pragma unroll
        for (uint32_t it = 0; it < kRegIters; ++it)
            if (begin + it * 64 < end) place(begin + it * 64 + lane, tq[it] < 0 ? -1 : (tq[it] & 2047), (uint32_t)tq[it] >> 11);
    } else if (!PRE && nw < kWaves) {
#pragma unroll 4
        for (uint32_t r = tid; r < R; r += kBatchThreads) {
            const int32_t t = a.row_tenant[r];
            place_row(a, r, t, t >= 0 ? offl[t] + hist[r / chunk * Tp + t] + a.row_rank[r] : 0);
        }
    } else if (!PRE) {
        for (uint32_t r0 = begin; r0 < end; r0 += 64) {
            const uint32_t r = r0 + lane;
            const int32_t t = r < end ? a.row_tenant[r] : -1;
            place(r, t, t >= 0 ? a.row_rank[r] : 0);
        }
    }

    // pass 4: the tile lists.  Big tiles pay only when a layer index has enough of them to fill the chip; below
    // that the streaming kernel takes those tenants too, side by side with everyone else's tiles.
    // One step: the J tenants a lane from t0 on, of layer index l; f: their facts, Mt: their rows.
    uint32_t run_fc, run_conv, run_big;                        // tiles of the tenants before this step
    auto list_step = [&](auto J_, uint32_t l, uint32_t t0, const uint4* f, const uint32_t* Mt, bool big_here, bool last) {
        constexpr uint32_t J = decltype(J_)::value;
        const uint32_t lm = a.list_mask[l / kLayerGroup] >> (l % kLayerGroup);      // bit kind * kLayerGroup: some registered model has such tiles here
        const bool split = (a.conv_split[l / 32] >> (l % 32)) & 1;      // this run's convolution tiles: 32 pixels, one channel block
        uint32_t n_fc[J], n_conv[J], n_big[J];
#pragma unroll
        for (uint32_t j = 0; j < J; ++j) {
            const uint32_t x = f[j].x, y = f[j].y, M = Mt[j];
            const bool conv = x >> 31, sk = a.fc_split_k && !conv && x;                // this run's FC tiles: one column block each, 32 rows
            const uint32_t blocks = x & 0x7fffffffu;                                   // (a convolution's)
            const uint32_t groups = sk ? ((x >> 29) & 1 && a.fc_whole ? 1 : y / kBrickRows) : x & 0x1fffffffu;
            const bool big = big_here && !conv && x && fc_is_big(M, y);
            // conv: rows = requests * output pixels per tile; FC: tiles of 64 or 32 rows over the rows that big tiles leave
            // (the few rows that big tiles leave in a narrow layer are tiled one column block and 32 rows at a time,
            // with K split among the waves: see big_remainder_split_k)
            static_assert(kTileRows == 64, "FC tiles have 64 or 32 rows");
            const uint32_t Mb = big ? big_rows(M) : 0;
            const bool rem_sk = big && big_remainder_split_k(y);
            const uint32_t sh = sk || rem_sk || ((x >> 30) & 1) ? 5 : 6, gq = rem_sk ? y / kBrickRows : groups;
            n_fc[j] = !conv && groups && M ? ((M - Mb + (1u << sh) - 1) >> sh) * gq : 0;
            n_conv[j] = conv && M ? (split ? ceil_div(M * f[j].z, kBrickRows) * blocks : ceil_div(M * y, kConvTileRows) * ceil_div(blocks, kTileCols / kBrickRows)) : 0;
            n_big[j] = ceil_div(Mb, kBigTile) * ceil_div(y, kBigTile);
        }
        auto emit = [&](uint32_t kind, const uint32_t (&n)[J], uint32_t& run) {
            if (!((lm >> (kind * kLayerGroup)) & 1)) return;                              // lists no registered model contributes to are never read
            uint32_t* base = a.tile_base + ((size_t)kind * MT_MAX_LAYERS + l) * (T + 1);
            uint32_t mine = 0;
#pragma unroll
            for (uint32_t j = 0; j < J; ++j) mine += n[j];
            const uint32_t incl = wave_inclusive_scan(mine);
            uint32_t at = run + incl - mine;
#pragma unroll
            for (uint32_t j = 0; j < J; ++j) {
                if (t0 + j < T) base[t0 + j] = at;
                at += n[j];
            }
            run += __builtin_amdgcn_readlane(incl, 63);
            if (last && lane == 0) base[T] = run;
        };
        emit(0, n_fc, run_fc);
        emit(1, n_conv, run_conv);
        emit(2, n_big, run_big);
    };
    auto big_possible = [&](uint32_t l) {
        return a.big_enabled && l < (uint32_t)kBigMaxLayer && ((a.list_mask[l / kLayerGroup] >> (2 * kLayerGroup + l % kLayerGroup)) & 1);
    };
    auto big_tiles = [&](uint4 f, uint32_t M) {
        return f.x && !(f.x >> 31) && fc_is_big(M, f.y) ? ceil_div(big_rows(M), kBigTile) * ceil_div(f.y, kBigTile) : 0u;
    };
    auto take_big = [&](uint32_t l, uint32_t n) {              // n: big tiles of this lane's tenants at layer index l
        const bool yes = __builtin_amdgcn_readlane(wave_inclusive_scan(n), 63) >= a.big_min_tiles;
        if (yes && lane == 0) atomicOr(&big_l, 1u << l);
        return yes;
    };
    if (one_wave) {
#pragma unroll
        for (uint32_t i = 0; i < kPre; ++i) {
            const uint32_t l = w + i * kWaves;
            if (l >= a.n_layer_slots) break;
            run_fc = run_conv = run_big = 0;
            list_step(std::integral_constant<uint32_t, 1>{}, l, lane, &fq[i], &Mt1, big_possible(l) && take_big(l, big_tiles(fq[i], Mt1)), true);
        }
    } else {
        constexpr uint32_t kStep = 64 * kPre;
        auto rows_of = [&](uint32_t t0, uint32_t (&M)[kPre]) {
            static_assert(kPre == 4 && kMaxTenantsPadded % kStep == 0, "one 16-byte read; tables of whole steps");
            const u32x4 m = *(const u32x4*)(Ml + t0);          // (entries from T on may never have been written)
#pragma unroll
            for (uint32_t j = 0; j < kPre; ++j) M[j] = t0 + j < T ? m[j] : 0;
        };
        for (uint32_t l = w; l < a.n_layer_slots; l += kWaves) {
            run_fc = run_conv = run_big = 0;
            bool big_here = false;
            if (l != w) {
#pragma unroll
                for (uint32_t j = 0; j < kPre; ++j) fq[j] = load_fact(l, lane * kPre + j);
            }
            if (big_possible(l)) {
                uint32_t n = 0;
                for (uint32_t t0 = lane * kPre; t0 - lane * kPre < T; t0 += kStep) {
                    uint32_t M[kPre];
                    rows_of(t0, M);
#pragma unroll
                    for (uint32_t j = 0; j < kPre; ++j) n += big_tiles(t0 < kStep ? fq[j] : load_fact(l, t0 + j), M[j]);
                }
                big_here = take_big(l, n);
            }
            for (uint32_t first = 0; first < T; first += kStep) {
                const uint32_t t0 = first + lane * kPre;
                uint4 ahead[kPre];                             // the next step's facts are asked for before this step's stores
#pragma unroll
                for (uint32_t j = 0; j < kPre; ++j) ahead[j] = load_fact(l, t0 + kStep + j);
                uint32_t M[kPre];
                rows_of(t0, M);
                list_step(std::integral_constant<uint32_t, kPre>{}, l, t0, fq, M, big_here, first + kStep >= T);
#pragma unroll
                for (uint32_t j = 0; j < kPre; ++j) fq[j] = ahead[j];
            }
        }
    }
    // First convolutions on the submitted images, alone or with the ones behind them: a list of rows of tiles, which the code above does not make
    // (list_mask).  Apart from it, by the wave that has the fewest lists: every instruction in its unrolled steps costs each run its fetch (1.4 us
    // with this in them, of a batcher of 4.2).
    if (a.first_cap && w == kWaves - 1) {
        uint32_t* base = a.tile_base + (size_t)MT_MAX_LAYERS * (T + 1);
        uint32_t run = 0;
        for (uint32_t t0 = 0; t0 < T; t0 += 64) {
            const uint32_t t = t0 + lane, M = one_wave ? Mt1 : t < T ? Ml[t] : 0;
            const uint4 f = load_fact(0, t);
            const uint32_t rows = a.first_pair ? load_fact(1, t).w : f.w;
            // (a replay during a registration may find the tenant and not yet its facts)
            const uint32_t n = f.x >> 31 && rows >> 16 && M ? M * first_strips(rows & 0xffffu, rows >> 16, a.first_cap) * ceil_div(f.x & 0x7fffffffu, kFirstBlocks) : 0;
            const uint32_t incl = wave_inclusive_scan(n);
            if (t < T) base[t] = run + incl - n;
            run += __builtin_amdgcn_readlane(incl, 63);
        }
        if (lane == 0) base[T] = run;
    }
    if (a.big_enabled) __syncthreads();
    if (tid == 0) *a.big_layers = big_l;               // the FC kernels split a qualifying tenant's rows by it
}

// ---- launcher ------------------------------------------------------------
hipError_t launch_batcher(const BatchArgs& a, hipStream_t s)
{
    const bool one = a.n_segs == 1;
    // rows per lane of the register path, as the kernel derives them
    uint32_t Tp = 64;
    while (Tp < a.T) Tp <<= 1;
    const uint32_t nw = std::min<uint32_t>(kBatchThreads / 64, kHistEntries / Tp);
    const uint32_t iters = (((a.R + nw - 1) / nw) + 63) / 64;
    if (a.n_rank_groups) {                  // large batch: ranked across the chip first
        if (a.T > (uint32_t)kRankMaxTenants || (uint64_t)a.n_rank_groups * Tp > (uint64_t)kHistEntries ||
            (uint64_t)a.n_rank_groups * kRankRows < a.R) return hipErrorInvalidValue;
        if (one) hipLaunchKernelGGL(rank_kernel<true>, dim3(a.n_rank_groups), dim3(kBatchThreads), 0, s, a);
        else hipLaunchKernelGGL(rank_kernel<false>, dim3(a.n_rank_groups), dim3(kBatchThreads), 0, s, a);
        hipLaunchKernelGGL((batcher_kernel<true, 4, true>), dim3(1), dim3(kBatchThreads), 0, s, a);
        hipLaunchKernelGGL(place_kernel, dim3(a.n_rank_groups), dim3(kBatchThreads), 0, s, a);
        return hipGetLastError();
    }
#define MT_BATCHER(SEG, IT) hipLaunchKernelGGL((batcher_kernel<SEG, IT>), dim3(1), dim3(kBatchThreads), 0, s, a)
    if (!one) { if (iters <= 1) MT_BATCHER(false, 1); else MT_BATCHER(false, 4); }
    else if (iters <= 1) MT_BATCHER(true, 1);
    else if (iters <= 4) MT_BATCHER(true, 4);
    else if (iters <= 8) MT_BATCHER(true, 8);
    else if (iters <= 16) MT_BATCHER(true, 16);
    else MT_BATCHER(true, 32);
#undef MT_BATCHER
    return hipGetLastError();
}

}  // namespace mt

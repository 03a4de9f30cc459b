// Tenant segmentation and grouped-work descriptors (see mt_device.h for the overview).
#include "mt_device.h"

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

// Tenant segmentation and grouped-work descriptors.  One workgroup; every step is
// deterministic: rows of a tenant keep their arrival order (stable counting sort).  Equal
// tenant ids inside a wavefront are found with one ballot per id bit, so a step costs the
// same whatever the tenant mix is.  Latency, not bandwidth, bounds this kernel, so everything
// that does not depend on the rows (tenant and layer facts) is fetched up front, and waves wait
// for each other as little as possible: with at most 64 tenants every wave holds all of
// them in its lanes and works out totals and offsets for itself (two barriers in the whole kernel),
// and a tile list belongs to one wave, which scans it 64 tenants at a time.
// Kernel trace, this form against one whose 1024 threads were the tenants and built the lists of eight layer indices
// at a time with three barriers per eight: 1 request to 8 three-layer models 7.8 -> 4.0 us, 4096 requests to 64 of
// them 13.0 -> 10.6, 1 request to 26-layer models 20.4 -> 5.8, behind the ranking kernel (32768 rows, 8 tenants)
// 13.9 -> 6.1, with 256 tenants 14.4 -> 13.6.
// ITERS: rows a lane may keep in registers (64 * ITERS rows per wave); the launcher picks the smallest
// instantiation that covers the batch, because the unrolled steps of a larger one cost small batches microseconds.
// A row's packed position is known: note it both ways; a rejected row (t < 0: unknown tenant or
// no model) is answered at once with label -1 and zero rows.
__device__ __forceinline__ void place_row(const BatchArgs& a, uint32_t r, int32_t t, uint32_t position)
{
    int32_t pos = -1;
    if (t >= 0) {
        pos = (int32_t)position;
        a.perm[pos] = (int32_t)r;
    } else {
        a.out.labels[r] = -1;
        if (a.out.n_classes) a.out.n_classes[r] = 0;
        for (uint32_t c = 0; c < a.out.row_stride; ++c) {
            if (a.out.probs) a.out.probs[(size_t)r * a.out.row_stride + c] = 0.0f;
            if (a.out.logits) a.out.logits[(size_t)r * a.out.row_stride + c] = 0.0f;
        }
    }
    a.pos_of[r] = pos;
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
        if (t < 0 || (uint32_t)t >= T || !a.tenants[t].registered) t = -1;
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

template <bool ONE_SEG, int ITERS, bool PRE = false>
__global__ __launch_bounds__(kBatchThreads) void batcher_kernel(BatchArgs a)
{
    constexpr uint32_t kWaves = kBatchThreads / 64;
    __shared__ uint32_t hist[kHistEntries];
    __shared__ uint32_t Ml[kMaxTenantsPadded];
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
    // The tile lists of layer index l (three kinds) belong to wave l % 16, which walks them 64 tenants at a time:
    // step i of the wave is chunk i % n_chunks of its (i / n_chunks)-th layer index.  A step needs the fact words
    // of its 64 tenant-layers (BatchArgs::facts); the first kPre steps' are fetched here.
    constexpr uint32_t kPre = 4;
    const uint32_t n_chunks = ceil_div(T, 64), n_steps = w < a.n_layer_slots ? ceil_div(a.n_layer_slots - w, kWaves) * n_chunks : 0;
    auto load_facts = [&](uint32_t l, uint32_t c) -> uint4 {
        const uint32_t t = c * 64 + lane;
        return t < T ? ((const uint4*)a.facts)[(size_t)t * MT_MAX_LAYERS + l] : uint4{0, 0, 0, 0};
    };
    auto next_step = [&](uint32_t& l, uint32_t& c) { if (++c == n_chunks) { c = 0; l += kWaves; } };
    uint4 fq[kPre];
    uint32_t l = w, c = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPre; ++i) {
        fq[i] = i < n_steps ? load_facts(l, c) : uint4{0, 0, 0, 0};
        next_step(l, c);
    }
    for (uint32_t t = tid; t < Tp; t += kBatchThreads) regl[t] = t < T && a.tenants[t].registered;
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
    if (in_regs) {
#pragma unroll
        for (uint32_t it = 0; it < kRegIters; ++it)
            if (begin + it * 64 < end) place(begin + it * 64 + lane, tq[it] < 0 ? -1 : (tq[it] & 2047), (uint32_t)tq[it] >> 11);
    } else if (!PRE) {
        for (uint32_t r0 = begin; r0 < end; r0 += 64) {
            const uint32_t r = r0 + lane;
            const int32_t t = r < end ? a.row_tenant[r] : -1;
            place(r, t, t >= 0 ? a.row_rank[r] : 0);
        }
    }

    // pass 4: the tile lists.  Big tiles pay only when a layer index has enough of them to fill the chip; below
    // that the streaming kernel takes those tenants too, side by side with everyone else's tiles.
    uint32_t run_fc = 0, run_conv = 0, run_big = 0;            // tiles of the tenants before this chunk
    bool big_here = false;
    auto tenant_rows = [&](uint32_t c) { return one_wave ? Mt1 : (c * 64 + lane < T ? Ml[c * 64 + lane] : 0u); };
    auto list_step = [&](uint32_t l, uint32_t c, uint4 f) {
        const uint32_t lm = a.list_mask[l / kLayerGroup] >> (l % kLayerGroup);      // bit kind * kLayerGroup: some registered model has such tiles here
        if (c == 0) {
            run_fc = run_conv = run_big = 0; big_here = false;
            if (a.big_enabled && l < (uint32_t)kBigMaxLayer && ((lm >> (2 * kLayerGroup)) & 1)) {
                uint32_t n = 0;
                for (uint32_t i = 0; i < n_chunks; ++i) {
                    const uint4 g = i == 0 ? f : load_facts(l, i);
                    const uint32_t Mt = tenant_rows(i);
                    const bool big = g.x && !(g.x >> 31) && fc_is_big(Mt, g.y);
                    n += __builtin_amdgcn_readlane(wave_inclusive_scan(big ? ceil_div(big_rows(Mt), kBigTile) * ceil_div(g.y, kBigTile) : 0), 63);
                }
                big_here = n >= a.big_min_tiles;
                if (big_here && lane == 0) atomicOr(&big_l, 1u << l);
            }
        }
        const uint32_t t = c * 64 + lane, Mt = tenant_rows(c);
        const bool conv = f.x >> 31, sk = a.fc_split_k && !conv && f.x;                // this run's FC tiles: one column block each, 32 rows
        const bool split = (a.conv_split[l / 32] >> (l % 32)) & 1;      // this run's convolution tiles: 32 pixels, one channel block
        const uint32_t groups = sk ? f.y / kBrickRows : conv ? ceil_div(f.x & 0x7fffffffu, split ? 1 : kTileCols / kBrickRows) : f.x & 0x3fffffffu;
        const bool big = big_here && !conv && f.x && fc_is_big(Mt, f.y);
        // conv: rows = requests * output pixels per tile; FC: tiles of 64 or 32 rows over the rows that big tiles leave
        // (the few rows that big tiles leave in a narrow layer are tiled one column block and 32 rows at a time,
        // with K split among the waves: see big_remainder_split_k)
        static_assert(kTileRows == 64, "FC tiles have 64 or 32 rows");
        const uint32_t Mb = big ? big_rows(Mt) : 0;
        const bool rem_sk = big && big_remainder_split_k(f.y);
        const uint32_t sh = sk || rem_sk || ((f.x >> 30) & 1) ? 5 : 6, gq = rem_sk ? f.y / kBrickRows : groups;
        auto emit = [&](uint32_t kind, uint32_t n, uint32_t& run) {
            if (!((lm >> (kind * kLayerGroup)) & 1)) return;                              // lists no registered model contributes to are never read
            uint32_t* base = a.tile_base + ((size_t)kind * MT_MAX_LAYERS + l) * (T + 1);
            const uint32_t incl = wave_inclusive_scan(n);
            if (t < T) base[t] = run + incl - n;
            run += __builtin_amdgcn_readlane(incl, 63);
            if (c + 1 == n_chunks && lane == 0) base[T] = run;
        };
        emit(0, !conv && groups && Mt ? ((Mt - Mb + (1u << sh) - 1) >> sh) * gq : 0, run_fc);
        emit(1, conv && Mt ? (split ? ceil_div(Mt * f.z, kBrickRows) : ceil_div(Mt * f.y, kConvTileRows)) * groups : 0, run_conv);
        emit(2, ceil_div(Mb, kBigTile) * ceil_div(f.y, kBigTile), run_big);
    };
    l = w; c = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPre; ++i) {
        if (i < n_steps) list_step(l, c, fq[i]);
        next_step(l, c);
    }
    for (uint32_t i = kPre; i < n_steps; ++i) {
        list_step(l, c, load_facts(l, c));
        next_step(l, c);
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

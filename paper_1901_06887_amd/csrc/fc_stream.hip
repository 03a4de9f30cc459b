// Grouped FC layer, weight-streaming tiles (see mt_device.h for the overview).
#include "mt_device.h"
#include <type_traits>

namespace mt {

// ---- grouped FC ------------------------------------------------------------------------------
// A workgroup of four waves owns up to 64 rows (RB row blocks of 32) of one tenant and
// `split` column blocks of 32.  Weight bricks never touch LDS: every wave streams the bricks
// of its own column block straight from memory into MFMA B operands through a ring of
// registers that keeps P bricks in flight.
//   split == 4 (the common case): the four waves share the same activation bricks, so those
//     are staged once per workgroup in LDS, 16 bricks per chunk, double buffered, one barrier
//     per chunk; LDS reads of a brick are 16 contiguous bytes per lane, conflict free.
//   split < 4 (layers with at most 64 outputs): the waves also split K between them, read
//     their own activation bricks directly, and the partial sums are added in a fixed order
//     through LDS (deterministic, no atomics).
constexpr uint32_t kRedFloats = 4 * 16 * 64;                 // one f32x16 per lane per wave
constexpr uint32_t kTrRowBytes = 32 * 4 + 16;                // transposition scratch row (fp32 worst case)
constexpr uint32_t kTrBytes = 32 * kTrRowBytes;
constexpr uint32_t kChunkBricks = 16;                        // activation bricks per LDS stage
constexpr uint32_t kStageBytes = kChunkBricks * kBrickBytes;
// LDS of the FC kernel, 34 KiB so that four workgroups fit a CU.  K loop: two activation
// stages (split == 4).  After the K loop: reduction scratch (split < 4 only) at offset 0 and
// transposition scratch at kTrOffset; both alias the stages, separated from them by barriers.
constexpr uint32_t kTrOffset = kRedFloats * 4;
constexpr uint32_t kFcLdsBytes = kTrOffset + 4 * kTrBytes;
template <int ROWS> constexpr uint32_t fc_lds_bytes() { return kFcLdsBytes + (ROWS == kRowsAny ? 4 * kBrickBytes : 0); }      // (the tails of rows of any length)
static_assert(kFcLdsBytes >= 2 * kStageBytes, "the two activation stages must fit");

// A lane's row of any length at any address: chunks that lie in it whole come as 16 bytes, wherever they begin; the others from a block of zeros (no lane reads past
// its row), and the elements behind the last whole chunk, asked for one by one up front, take the place of the chunk that they begin.
template <typename T> struct AnyChunk;
template <> struct AnyChunk<__bf16> { typedef u32x4 type __attribute__((aligned(2))); };
template <> struct AnyChunk<float> { typedef u32x4 type __attribute__((aligned(4))); };
template <typename T> struct AnyRow {
    static constexpr uint32_t EPC = 16 / sizeof(T);
    typedef const __attribute__((address_space(1))) typename AnyChunk<T>::type* cptr_t;
    typedef const __attribute__((address_space(1))) T* eptr_t;
    eptr_t row;
    uint32_t whole;            // elements in whole chunks (none: a padding row)
    uint32_t rest;             // where the tail belongs
    u32x4 tail;
    __device__ __forceinline__ void init(const void* at, bool ok, uint32_t n)
    {
        row = (eptr_t)at;
        rest = n / EPC * EPC;
        whole = ok ? rest : 0;
        T t[EPC];
#pragma unroll
        for (uint32_t e = 0; e < EPC; ++e) t[e] = row[min(rest + e, n - 1)];
#pragma unroll
        for (uint32_t e = 0; e < EPC; ++e) t[e] = ok && rest + e < n ? t[e] : (T)0.0f;
        tail = __builtin_bit_cast(u32x4, t);
    }
    __device__ __forceinline__ u32x4 load(uint32_t k, const void* zeros) const { return *(k < whole ? (cptr_t)(row + k) : (cptr_t)zeros); }
    __device__ __forceinline__ u32x4 at(uint32_t k, const u32x4& v) const { return k == rest ? tail : v; }
};

// split == 4: activations through LDS, weights through the register ring.
// row_of(block of 32 rows of the tile, lane, real): the submitted row of a lane (GATHER).
template <typename T, int RB, int GATHER, typename ROWS>
__device__ __forceinline__ void fc_accumulate_shared(const GemmArgs& a, const Tile& tl, const LayerDev& L, uint32_t seg0,
                                                     uint32_t nb, bool active, const ROWS& row_of, uint8_t* stages, f32x16 (&acc)[RB])
{
    constexpr uint32_t EPC = 16 / sizeof(T), KB = 2 * EPC;
    constexpr uint32_t KC = kChunkBricks / RB;               // k steps per chunk: 16 or 8
    constexpr uint32_t P = 16;                               // weight bricks in flight per wave
    constexpr uint32_t U = P > KC ? P : KC;                  // unrolled block of k steps
    static_assert(U == P && U % KC == 0, "the tail relies on U == P");
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t nKB = L.K / KB;
    const uint32_t nrb = (tl.rows + kBrickRows - 1) / kBrickRows;
    const uint32_t nb_eff = active ? nb : 0;                 // idle waves still help staging; they stream block 0 and drop it
    const u32x4* wp = (const u32x4*)(a.arena + L.w_off) + (size_t)nb_eff * nKB * 64 + lane;
    const u32x4* xbase = (const u32x4*)((const T*)act_of(a.act, L.in_buf) + (size_t)seg0 * a.S) + lane;

    // this wave stages bricks q = 4*wave .. 4*wave+3 of every chunk: row block q / KC, k step q % KC
    const u32x4* xsrc[4]; uint32_t xkk[4];
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t q = wave * 4 + j, r = q / KC;
        xkk[j] = q % KC;
        const uint32_t rbi = tl.m0 / kBrickRows + min(r, nrb - 1);     // blocks past the tile repeat its last one
        xsrc[j] = xbase + (size_t)rbi * nKB * 64;
    }
    // GATHER (layer 0): the bricks are formed on the fly from the submitted rows; this wave's
    // four bricks lie in one row block, so a lane reads from one row (null for padding rows)
    typedef const __attribute__((address_space(1))) u32x4* gptr_t;     // submitted rows live in global memory
    gptr_t rowp = nullptr;
    bool row_ok = false;
    AnyRow<T> any;
    if (GATHER) {
        const void* at = row_of(min(wave * 4 / KC, nrb - 1), lane & 31, &row_ok);
        rowp = (gptr_t)at;
        if constexpr (GATHER == kRowsAny) {                  // the tail waits in LDS: these tiles use all the registers there are
            any.init(at, row_ok, L.k_valid);
            *(u32x4*)(stages + kFcLdsBytes + wave * kBrickBytes + lane * 16) = any.tail;
        }
    }
    auto load_chunk = [&](uint32_t c, u32x4 (&xr)[4]) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            if (GATHER == kRowsAny) {
                xr[j] = any.load((c * KC + xkk[j]) * KB + (lane >> 5) * EPC, a.zeros);
            } else if (GATHER) {
                const uint32_t k = (c * KC + xkk[j]) * KB + (lane >> 5) * EPC;
                const bool ok = row_ok && k < L.k_valid;
                const u32x4 v = rowp[(ok ? k : 0) / EPC];
                xr[j] = ok ? v : u32x4{0, 0, 0, 0};
            } else {
                xr[j] = xsrc[j][(size_t)min(c * KC + xkk[j], nKB - 1) * 64];
            }
        }
    };
    auto store_chunk = [&](uint32_t c, const u32x4 (&xr)[4]) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            u32x4 v = xr[j];
            if constexpr (GATHER == kRowsAny) {
                const uint32_t k = (c * KC + xkk[j]) * KB;
                if (k == any.rest / KB * KB) {                // (uniform: one step of all; the address is worked out there, see fc_tile)
                    uint32_t at = lane;
                    asm("" : "+v"(at));
                    if (any.rest - k == (at >> 5) * EPC) v = *(const u32x4*)(stages + kFcLdsBytes + wave * kBrickBytes + at * 16);
                }
            }
            *(u32x4*)(stages + (c & 1) * kStageBytes + (wave * 4 + j) * kBrickBytes + lane * 16) = v;
        }
    };

    // K is walked in blocks of U steps, unrolled, so that ring slots (step % P) and, where a
    // block spans two chunks, LDS stages are compile-time constants.  Slot s % P holds step s
    // from P steps before its use until its MFMAs; it is refilled with step s + P right after.
    // Loads return in order, so waiting for an activation load also waits for every weight
    // load issued before it.  The activation bricks of a chunk are therefore fetched as far
    // ahead as the weight ring reaches (NX chunks = P steps): by the time they are waited for,
    // every older weight load is one whose MFMA is due anyway, and the ring keeps its depth
    // across chunk boundaries (with one chunk of lookahead the 64-row tiles, whose chunks are 8
    // steps, had only the newest 8 weight loads in flight at every boundary; worth 1-2 % on the
    // skewed mixes).
    constexpr uint32_t NX = P / KC;                           // 1 (32-row tiles) or 2
    static_assert(NX >= 1 && U % (NX * KC) == 0, "a block of U steps starts with staging slot 0");
    u32x4 bq[P], xr[NX][4];
#pragma unroll
    for (uint32_t j = 0; j < P; ++j) bq[j] = wp[(size_t)min(j, nKB - 1) * 64];
    load_chunk(0, xr[0]);
    store_chunk(0, xr[0]);
#pragma unroll
    for (uint32_t i = 1; i <= NX; ++i) load_chunk(i, xr[i % NX]);   // zeros / clamped past the last chunk
    uint32_t c = 0;                                           // chunk being consumed; it lives in stage c & 1
    const uint8_t* st = stages + lane * 16;
    auto next_chunk = [&](uint32_t slot) {                    // slot = (c + 1) % NX, a constant at every call site
        lds_barrier();                                        // stage c&1 is complete; stage (c+1)&1 is free again
        store_chunk(c + 1, xr[slot]);
        load_chunk(c + 1 + NX, xr[slot]);
        st = stages + (c & 1) * kStageBytes + lane * 16;
        ++c;
    };
    const uint32_t n_blocks = nKB / U;
    for (uint32_t blk = 0; blk < n_blocks; ++blk) {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (u % KC == 0) next_chunk((u / KC + 1) % NX);
            u32x4 av[RB];
#pragma unroll
            for (int r = 0; r < RB; ++r) av[r] = *(const u32x4*)(st + (r * KC + u % KC) * kBrickBytes);
#pragma unroll
            for (int r = 0; r < RB; ++r) Mma<T>::run(acc[r], av[r], bq[u % P]);
            bq[u % P] = wp[(size_t)min(blk * U + u + P, nKB - 1) * 64];
            // keeps the compiler from hoisting every LDS read of the block to its top (registers)
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const uint32_t rem = nKB - n_blocks * U;                  // < U == P: the ring already holds these steps
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
        if (u < rem) {
            if (u % KC == 0) next_chunk((u / KC + 1) % NX);
#pragma unroll
            for (int r = 0; r < RB; ++r) Mma<T>::run(acc[r], *(const u32x4*)(st + (r * KC + u % KC) * kBrickBytes), bq[u % P]);
        }
    }
}

// split < 4: every wave reads the activation bricks of its own K range directly.
// NB: column blocks at once (nb, and nb2).
template <typename T, int GATHER, int NB = 1>
__device__ __forceinline__ void fc_accumulate_direct(const GemmArgs& a, const Tile& tl, const LayerDev& L, uint32_t seg0,
                                                     uint32_t nb, uint32_t nb2, uint32_t kq, uint32_t ks, const void* row, bool row_ok, f32x16 (&acc)[NB])     // GATHER: this lane's submitted row (a padding row: any)
{
    constexpr uint32_t EPC = 16 / sizeof(T), KB = 2 * EPC;
    constexpr int P = NB == 1 ? 8 : 4;                        // steps in flight per wave
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t nKB = L.K / KB;
    const uint32_t cnt = nKB / ks, kb0 = kq * cnt;
    const u32x4* wp[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) wp[c] = (const u32x4*)(a.arena + L.w_off) + ((size_t)(c ? nb2 : nb) * nKB + kb0) * 64 + lane;
    const u32x4* xp = (const u32x4*)((const T*)act_of(a.act, L.in_buf) + (size_t)seg0 * a.S) + lane + ((size_t)(tl.m0 / kBrickRows) * nKB + kb0) * 64;
    typedef const __attribute__((address_space(1))) u32x4* gptr_t;     // submitted rows live in global memory
    const gptr_t rowp = (gptr_t)row;
    AnyRow<T> any;
    if constexpr (GATHER == kRowsAny) any.init(row, row_ok, L.k_valid);
    // (a submitted row's chunk is masked where it is used, not where it is asked for: that would wait for it)
    auto chunk_of = [&](uint32_t kk) { return (kb0 + kk) * KB + (lane >> 5) * EPC; };
    auto in_row = [&](uint32_t k) { return row_ok && k < L.k_valid; };
    auto load_x = [&](uint32_t kk) -> u32x4 {
        if (!GATHER) return xp[(size_t)kk * 64];
        const uint32_t k = chunk_of(kk);
        if (GATHER == kRowsAny) return any.load(k, a.zeros);
        return rowp[(in_row(k) ? k : 0) / EPC];
    };
    auto masked = [&](const u32x4& v, uint32_t kk) -> u32x4 {
        if (GATHER == kRowsAny) return any.at(chunk_of(kk), v);
        return !GATHER || in_row(chunk_of(kk)) ? v : u32x4{0, 0, 0, 0};
    };
    u32x4 bq[P][NB], aq[P];
    auto load_w = [&](int j, uint32_t kk) {
#pragma unroll
        for (int c = 0; c < NB; ++c) bq[j][c] = wp[c][(size_t)kk * 64];
    };
    auto step = [&](int j, uint32_t kk) {
        const u32x4 x = masked(aq[j], kk);
#pragma unroll
        for (int c = 0; c < NB; ++c) Mma<T>::run(acc[c], x, bq[j][c]);
    };
#pragma unroll
    for (int j = 0; j < P; ++j) {
        const uint32_t kk = min((uint32_t)j, cnt - 1);
        load_w(j, kk);
        aq[j] = load_x(kk);
        __builtin_amdgcn_sched_barrier(0);
    }
    // steady state: straight-line groups of P bricks, each slot refilled right after use; the
    // clamped refill index re-reads the last brick instead of branching.  The fences keep the loads in the order of their
    // use, one step's behind the other's: left to itself the compiler gathers a group's MFMAs behind a wait for all its loads
    const uint32_t full = cnt / P;
    for (uint32_t g = 0; g < full; ++g) {
#pragma unroll
        for (int j = 0; j < P; ++j) {
            step(j, g * P + j);
            const uint32_t kk = min(g * P + j + P, cnt - 1);
            load_w(j, kk);
            aq[j] = load_x(kk);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const uint32_t rem = cnt - full * P;                      // the slots already hold the remaining bricks
#pragma unroll
    for (int j = 0; j < P; ++j)
        if ((uint32_t)j < rem) step(j, full * P + j);
}

__device__ __forceinline__ int32_t submission_of(const GemmArgs& a, const LayerDev& L, uint32_t seg0, uint32_t m0) { return L.is_last ? a.perm[seg0 + m0 + (threadIdx.x >> 3)] : -1; }

// The rows of a tile whose logits stand in LDS as [row][class], LRS floats to a row, at most 32 Q classes: softmax, argmax, outputs in submission order, eight
// threads a row, whose place there they have asked for before the sums (submission_of).
template <uint32_t Q, uint32_t LRS>
__device__ __forceinline__ void fc_finish_rows(const GemmArgs& a, const float* lt, uint32_t C, uint32_t mb, uint32_t Mt, int32_t submitted)
{
    const uint32_t tid = threadIdx.x, row = tid >> 3, part = tid & 7, m = mb + row, sub = (uint32_t)submitted;
    if (m >= Mt) return;                                                 // the eight threads of a row are neighbours in one wave
    f32x4 z[Q], ez[Q];
    float mx = -INFINITY; int32_t best = 0x7fffffff;
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q) {                                   // thread `part` holds classes 4 part + 32 q + {0..3}
        z[q] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (q * kBrickRows < C) z[q] = *(const f32x4*)(lt + row * LRS + q * kBrickRows + part * 4);
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) {
            const uint32_t c = q * kBrickRows + part * 4 + e;
            if (c >= C) z[q][e] = -INFINITY;
            if (z[q][e] > mx) { mx = z[q][e]; best = (int32_t)c; }      // increasing index: the first hit is this thread's lowest
        }
    }
#pragma unroll
    for (int d = 4; d >= 1; d >>= 1) {
        const float omx = __shfl_xor(mx, d);
        const int32_t ob = __shfl_xor(best, d);
        if (omx > mx || (omx == mx && ob < best)) { mx = omx; best = ob; }
    }
    best = head_label(best, lt[row * LRS]);
    float sum = 0.0f;
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q)
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) { ez[q][e] = q * kBrickRows + part * 4 + e < C ? __expf(z[q][e] - mx) : 0.0f; sum += ez[q][e]; }
#pragma unroll
    for (int d = 4; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
    const float inv = 1.0f / sum;
    if (part == 0) {
        a.out.labels[sub] = best;
        if (a.out.n_classes) a.out.n_classes[sub] = (int32_t)C;
    }
    float* pr = a.out.probs ? a.out.probs + (size_t)sub * a.out.row_stride : nullptr;
    float* lg = a.out.logits ? a.out.logits + (size_t)sub * a.out.row_stride : nullptr;
#pragma unroll
    for (uint32_t q = 0; q < Q; ++q) {
        const uint32_t c0 = q * kBrickRows + part * 4;
        f32x4 pv, lv;
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) { const bool in = c0 + e < C; pv[e] = in ? ez[q][e] * inv : 0.0f; lv[e] = in ? z[q][e] : 0.0f; }
        if (a.out_vec_ok) {
            if (c0 < a.out.row_stride) { if (pr) *(f32x4*)(pr + c0) = pv; if (lg) *(f32x4*)(lg + c0) = lv; }
        } else {
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e)
                if (c0 + e < a.out.row_stride) { if (pr) pr[c0 + e] = pv[e]; if (lg) lg[c0 + e] = lv[e]; }
        }
    }
    for (uint32_t c = Q * kBrickRows + part; c < a.out.row_stride; c += 8) {      // wider output rows: zeros past the tile
        if (pr) pr[c] = 0.0f;
        if (lg) lg[c] = 0.0f;
    }
}

// End of a tile whose waves split K (split < 4; ks = 4 / split waves share a column block): the partial sums meet in LDS and are
// added in wave order, and what follows is dealt to all the waves: wave kq takes the output rows 8 g + 4 lh + {0..3} of
// its 4 / ks values of g, then a share of the finished bricks, or, in a last layer whose classes are all in this tile, of the
// rows (eight threads each: softmax, argmax, outputs in submission order).  These tiles live for a few microseconds, of which a
// single wave's finish was one to three: 48 LDS reads, the activation of 16 values a lane, loops over the classes by one thread per row.
// Passes, one wave's finish -> this -> with a kernel of their own for such tiles (fc_kernel's NARROW): one request to a 784-1024-1024-10
// model 26.6 -> 25.7 -> 24.6 us, 64 fp32 requests to 256-512-512-10 models 30.7 -> 29.7 -> 28.6, 777 requests to 301-333-520-97-37 models
// with GELU 59.0 -> 57.1 -> 57.0; the last layer of 64 residual nets 8.6 -> 6.9.
template <typename T>
__device__ __forceinline__ void fc_finish_split(const GemmArgs& a, const Tile& tl, const LayerDev& L, uint32_t Mt, uint32_t seg0,
                                                uint32_t nb, uint32_t kq, uint32_t ks, bool active, float bv, int32_t sub, T* xout, const f32x16& acc, uint8_t* smem)
{
    constexpr uint32_t EPC = 16 / sizeof(T), KB = 2 * EPC, MAXG = 2;         // (ks is 2 or 4)
    constexpr uint32_t TRS = 32 * sizeof(T) + 16;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 31, lh = lane >> 5;
    const uint32_t split = tl.split, cb = wave % split, ng = 4 / ks;
    const uint32_t n = nb * kBrickRows + li;
    float* red = (float*)smem;
    uint8_t* trw = smem + kTrOffset + cb * kTrBytes;
    const bool head = L.is_last && a.fuse_head && L.N <= a.fuse_head_max && L.N_pad <= split * kBrickRows;
    constexpr uint32_t LRS = 2 * kBrickRows + 4;                             // floats per row of the logits tile
    static_assert(kBrickRows * LRS * 4 <= 4 * kTrBytes, "the logits tile lies where the transposition scratch does");
    float* lt = (float*)(smem + kTrOffset);
    __syncthreads();
    if (active) {
#pragma unroll
        for (uint32_t g = 0; g < 4; ++g) *(f32x4*)(red + wave * 1024 + g * 256 + lane * 4) = f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    }
    __syncthreads();
    f32x4 y[MAXG];
#pragma unroll
    for (uint32_t i = 0; i < MAXG; ++i) {
        y[i] = f32x4{0, 0, 0, 0};
        if (active && i < ng) {
            const float* src = red + cb * 1024 + (kq * ng + i) * 256 + lane * 4;
            y[i] = *(const f32x4*)src;
            for (uint32_t q = 1; q < ks; ++q) y[i] += *(const f32x4*)(src + q * split * 1024);
#pragma unroll
            for (int e = 0; e < 4; ++e) y[i][e] += bv;
        }
    }
    const uint32_t mb = tl.m0;
    if (head) {
#pragma unroll
        for (uint32_t i = 0; i < MAXG; ++i)
            if (active && i < ng) {
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) lt[(8 * (kq * ng + i) + 4 * lh + e) * LRS + cb * kBrickRows + li] = y[i][e];
            }
        __syncthreads();
        fc_finish_rows<MAXG, LRS>(a, lt, L.N, mb, Mt, sub);
        return;
    }
    if (L.is_last) {
#pragma unroll
        for (uint32_t i = 0; i < MAXG; ++i)
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) {
                const uint32_t m = mb + 8 * (kq * ng + i) + 4 * lh + e;
                if (active && i < ng && n < L.N && m < Mt) a.logits[(size_t)(seg0 + m) * a.C_pad + n] = y[i][e];
            }
        return;
    }
    // hidden layer: activation, rounding; the 32x32 block through LDS as [row][column], out as whole bricks.  Outputs past N are
    // masked: a zero weight row against an infinite input is NaN, and the next layer reads them with zero weights
    activate_block<MAXG>(y, L.act);
#pragma unroll
    for (uint32_t i = 0; i < MAXG; ++i)
        if (active && i < ng) {
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) *(T*)(trw + (8 * (kq * ng + i) + 4 * lh + e) * TRS + li * sizeof(T)) = (T)(n < L.N ? y[i][e] : 0.0f);
        }
    __syncthreads();
    if (active) {
        u32x4* out = (u32x4*)xout + ((size_t)(mb / kBrickRows) * (L.out_fill / KB) + nb * (kBrickRows / KB)) * 64 + lane;
        for (uint32_t c = kq; c < kBrickRows / KB; c += ks) out[c * 64] = *(const u32x4*)(trw + li * TRS + (c * KB + lh * EPC) * sizeof(T));
    }
}

// A tile whose waves split K: 32 rows (fc_shape).
template <typename T, int GATHER>
__device__ __forceinline__ void fc_split_tile(const GemmArgs& a, const Tile& tl, const LayerDev& L, uint32_t Mt, uint32_t seg0, const void* row, bool row_ok, T* xout, uint8_t* smem)
{
    const uint32_t split = tl.split, ks = 4 / split, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t nb = tl.n0 / kBrickRows + (wave % split), kq = wave / split;
    const bool active = nb < L.N_pad / kBrickRows;
    // what the end of the tile needs is asked for in front of the sums: behind them it was a trip to memory each (64 fp32 requests to MLPs 20.7 -> 20.6 us, one bf16 19.7 -> 19.4)
    const float bv = active ? ((const float*)(a.arena + L.b_off))[nb * kBrickRows + (threadIdx.x & 31)] : 0.0f;
    const int32_t sub = submission_of(a, L, seg0, tl.m0);
    f32x16 acc[1];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = 0.0f;
    if (active) fc_accumulate_direct<T, GATHER>(a, tl, L, seg0, nb, nb, kq, ks, row, row_ok, acc);
    fc_finish_split<T>(a, tl, L, Mt, seg0, nb, kq, ks, active, bv, sub, xout, acc[0], smem);
}

// A last layer of 33 to 128 classes in a run whose tiles split K: the tile takes all its column blocks, two at a time, and finishes its rows, where a tile per block left them to a
// launch of their own.  Sums as in those.  Bound by its chain of trips like them: the second pair of blocks adds 1 us, the head's launch took 4 (and 3 of the host).
template <typename T>
__device__ __forceinline__ void fc_whole_tile(const GemmArgs& a, const Tile& tl, const LayerDev& L, uint32_t Mt, uint32_t seg0, uint8_t* smem)
{
    constexpr uint32_t LRS = kTileCols + 4;                                  // floats per row of the logits tile
    static_assert(kTrOffset + kBrickRows * LRS * 4 <= kFcLdsBytes, "behind the partial sums");
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 31, lh = lane >> 5, blocks = L.N_pad / kBrickRows;
    float *red = (float*)smem, *lt = (float*)(smem + kTrOffset);
    const float* bias = (const float*)(a.arena + L.b_off);
    const int32_t sub = submission_of(a, L, seg0, tl.m0);
    for (uint32_t nb = 0; nb < blocks; nb += 2) {
        const uint32_t nb2 = min(nb + 1, blocks - 1);
        const float bv[2] = {bias[nb * kBrickRows + li], bias[nb2 * kBrickRows + li]};
        f32x16 acc[2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[c][v] = 0.0f;
        fc_accumulate_direct<T, kRowsStaged, 2>(a, tl, L, seg0, nb, nb2, wave, 4, nullptr, false, acc);
#pragma unroll
        for (uint32_t c = 0; c < 2; ++c) {
            __syncthreads();
#pragma unroll
            for (uint32_t g = 0; g < 4; ++g) *(f32x4*)(red + wave * 1024 + g * 256 + lane * 4) = f32x4{acc[c][4 * g], acc[c][4 * g + 1], acc[c][4 * g + 2], acc[c][4 * g + 3]};
            __syncthreads();
            f32x4 y = *(const f32x4*)(red + wave * 256 + lane * 4);
#pragma unroll
            for (uint32_t q = 1; q < 4; ++q) y += *(const f32x4*)(red + q * 1024 + wave * 256 + lane * 4);
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) lt[(8 * wave + 4 * lh + e) * LRS + (c ? nb2 : nb) * kBrickRows + li] = y[e] + bv[c];      // (an odd last block is written twice)
        }
    }
    __syncthreads();
    fc_finish_rows<kTileCols / kBrickRows, LRS>(a, lt, L.N, tl.m0, Mt, sub);
}

// LAST: the layer may be a last one (not in fc_entry_wide_kernel, whose models all have a second).
template <typename T, int RB, int GATHER, bool LAST, typename ROWS>
__device__ __forceinline__ void fc_tile(const GemmArgs& a, const Tile& tl, const LayerDev& L, uint32_t Mt, uint32_t seg0, const ROWS& row_of, T* xout, uint8_t* smem)     // xout: the tenant's first output row
{
    const uint32_t split = tl.split;
    constexpr uint32_t EPC = 16 / sizeof(T), KB = 2 * EPC;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t nb = tl.n0 / kBrickRows + wave;            // (split == 4)
    const bool active = nb < L.N_pad / kBrickRows;
    const uint32_t nrb = (tl.rows + kBrickRows - 1) / kBrickRows;
    uint8_t* tr = smem + kTrOffset;                           // aliases the stages, used after the K loop only

    f32x16 acc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] = 0.0f;

    const float bv = active ? ((const float*)(a.arena + L.b_off))[nb * kBrickRows + (threadIdx.x & 31)] : 0.0f;      // (asked for in front of the sums: 4096 requests to 64 MLPs 99.4 -> 97.3 us)
    fc_accumulate_shared<T, RB, GATHER>(a, tl, L, seg0, nb, active, row_of, smem, acc);
    // What follows goes by the lane, and is worked out from here on: kept through the K loop, which uses all the registers there are, it went to scratch memory in
    // fc_entry_wide_kernel (64 tenants of 784-1024-1024-10, 1024 / 2048 requests 55.4 / 63.2 -> 54.0 / 60.5 us a pass; rows of 787 values, 32 tenants, 38.9 / 51.9 -> 36.4 / 48.6)
    uint32_t tid_behind = threadIdx.x;
    asm volatile("" : "+v"(tid_behind));
    const uint32_t lane = tid_behind & 63, li = lane & 31, lh = lane >> 5, n = nb * kBrickRows + li;
    if (LAST && L.is_last && a.fuse_head && L.N <= a.fuse_head_max && L.N_pad <= split * kBrickRows) {
        // 33 .. 128 classes, all of them inside this tile (one column group): the waves put their
        // 32x32 blocks of logits side by side in LDS as [row][class], then eight threads share a
        // row: softmax, argmax (lowest index on ties) and the outputs in submission order.
        constexpr uint32_t LRS = kTileCols + 4;                 // floats per row of the logits tile (16-byte aligned rows)
        static_assert(kBrickRows * LRS * 4 <= kFcLdsBytes, "the logits tile of one row block must fit the kernel's LDS");
        float* lt = (float*)smem;
        const uint32_t C = L.N, tid = tid_behind, row = tid >> 3, part = tid & 7;
        const bool vec = a.out_vec_ok;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            __syncthreads();
            if (active && (uint32_t)r < nrb) {
#pragma unroll
                for (int v = 0; v < 16; ++v) lt[(8 * (v >> 2) + 4 * lh + (v & 3)) * LRS + n] = acc[r][v] + bv;
            }
            __syncthreads();
            const uint32_t m = tl.m0 + r * kBrickRows + row;
            if ((uint32_t)r < nrb && m < Mt) {                   // the eight threads of a row are neighbours in one wave
                f32x4 z[4];
                float mx = -INFINITY; int32_t best = 0x7fffffff;
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    z[q] = *(const f32x4*)(lt + row * LRS + part * 16 + q * 4);
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) {
                        const uint32_t c = part * 16 + q * 4 + i;
                        if (c >= C) z[q][i] = -INFINITY;       // also hides what idle waves did not write
                        if (z[q][i] > mx) { mx = z[q][i]; best = (int32_t)c; }      // increasing index: the first hit is the lowest
                    }
                }
#pragma unroll
                for (int d = 4; d >= 1; d >>= 1) {
                    const float omx = __shfl_xor(mx, d);
                    const int32_t ob = __shfl_xor(best, d);
                    if (omx > mx || (omx == mx && ob < best)) { mx = omx; best = ob; }
                }
                best = head_label(best, lt[row * LRS]);
                f32x4 e[4];
                float sum = 0.0f;
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q)
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) { e[q][i] = __expf(z[q][i] - mx); sum += e[q][i]; }   // exp(-inf) = 0 past the last class
#pragma unroll
                for (int d = 4; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
                const float inv = 1.0f / sum;
                const uint32_t sub = (uint32_t)a.perm[seg0 + m];
                if (part == 0) {
                    a.out.labels[sub] = best;
                    if (a.out.n_classes) a.out.n_classes[sub] = (int32_t)C;
                }
                float* pr = a.out.probs ? a.out.probs + (size_t)sub * a.out.row_stride : nullptr;
                float* lg = a.out.logits ? a.out.logits + (size_t)sub * a.out.row_stride : nullptr;
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    const uint32_t c0 = part * 16 + q * 4;
                    f32x4 pv, lv;
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) { const bool in = c0 + i < C; pv[i] = in ? e[q][i] * inv : 0.0f; lv[i] = in ? z[q][i] : 0.0f; }
                    if (vec) {
                        if (c0 < a.out.row_stride) { if (pr) *(f32x4*)(pr + c0) = pv; if (lg) *(f32x4*)(lg + c0) = lv; }
                    } else {
#pragma unroll
                        for (uint32_t i = 0; i < 4; ++i)
                            if (c0 + i < a.out.row_stride) { if (pr) pr[c0 + i] = pv[i]; if (lg) lg[c0 + i] = lv[i]; }
                    }
                }
                for (uint32_t c = kTileCols + part; c < a.out.row_stride; c += 8) {      // wider output rows: zeros past the tile
                    if (pr) pr[c] = 0.0f;
                    if (lg) lg[c] = 0.0f;
                }
            }
        }
        return;
    }
    if (LAST && L.is_last) {
        if (!active || n >= L.N) return;
#pragma unroll
        for (int r = 0; r < RB; ++r) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint32_t m = tl.m0 + r * kBrickRows + 8 * (v >> 2) + 4 * lh + (v & 3);
                if ((uint32_t)r < nrb && m < Mt) a.logits[(size_t)(seg0 + m) * a.C_pad + n] = acc[r][v] + bv;
            }
        }
        return;
    }
    // hidden layer: bias, activation, rounding; transpose the 32x32 block through LDS so that
    // every lane ends up with 16 contiguous output bytes, then store whole bricks
    constexpr uint32_t TRS = 32 * sizeof(T) + 16;
    uint8_t* trw = tr + wave * kTrBytes;
    const uint32_t nKB_out = L.out_fill / KB;
    u32x4* obase = (u32x4*)xout + lane;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        __syncthreads();
        if (active && (uint32_t)r < nrb) {
            f32x4 y[4];
#pragma unroll
            for (int v = 0; v < 16; ++v) y[v >> 2][v & 3] = acc[r][v] + bv;
            activate_block<4>(y, L.act);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint32_t ml = 8 * (v >> 2) + 4 * lh + (v & 3);
                *(T*)(trw + ml * TRS + li * sizeof(T)) = (T)(n < L.N ? y[v >> 2][v & 3] : 0.0f);
            }
        }
        __syncthreads();
        if (active && (uint32_t)r < nrb) {
#pragma unroll
            for (uint32_t c = 0; c < kBrickRows / KB; ++c) {
                const u32x4 chunk = *(const u32x4*)(trw + li * TRS + (c * KB + lh * EPC) * sizeof(T));
                const uint32_t kb_out = nb * (kBrickRows / KB) + c;
                obase[((size_t)(tl.m0 / kBrickRows + r) * nKB_out + kb_out) * 64] = chunk;
            }
        }
    }
}

// FEW: at most 64 tenants (for launches of nothing but K-split tiles; those of many tiles gain nothing: 1024 tiles of 64 tenants
// 99.3 -> 100.0 us a pass).  NARROW: every tile of the launch splits K (small runs, layer indices with at most 64 outputs): a kernel a
// third the size, with registers for four workgroups per CU.  WHOLE: some last layer of the index takes tiles of all its column blocks
// (fc_whole_tile), which need the registers of three: in the plain narrow kernel they spilled, and every launch brought their code
// (64 bf16 requests to 256-256-256-256-256-256-256-10 models 35.9 -> 34.8 us a pass without, four 256-512-512-40 20.3 -> 20.5).
// GATHER: layer 0 reads the submitted rows itself.  In the general kernel the wide tiles stand first
// and the two kinds of layer 0 in kernels of their own: with both and the K-split tiles in front, 40 scalar registers were
// spilled and layer 0 of 256 models of mixed depths took 175.9 us instead of 171.3.
template <typename T, bool NARROW, int GATHER, bool FEW, bool WHOLE = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NARROW && !WHOLE ? 4 : 3, NARROW && !WHOLE ? 4 : 3))) void fc_kernel(GemmArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t smem[NARROW ? kFcLdsBytes : fc_lds_bytes<GATHER>()];
    __shared__ uint32_t owner_part[4];
    TileLookup<256, FEW ? 64 : 0> lookup;
    lookup.fetch(a);
    const uint32_t n_tiles = a.tile_base[a.T];
    uint32_t idx;
    if (!logical_tile(n_tiles, &idx)) return;
    Tile tl;
    LayerDev L;
    uint32_t Mt, seg0, local;
    static_assert(kStageBytes + ahead_bytes() <= kFcLdsBytes, "the second stage, and the scratch of the K-split tiles, are first written behind a barrier");
    lookup.find(a, idx, owner_part, smem + kStageBytes, &tl.tenant, &L, &Mt, &seg0, &local);
    asm volatile("" :: "s"(seg0), "s"(local));                // keeps those loads here, next to the others, instead of at their first use
    // where big tiles serve this tenant-layer, only the rows they leave are tiled here (in the shape that
    // big_remainder_split_k says: the batcher counted the tiles by the same rule)
    const bool big = ((*a.big_layers >> a.layer) & 1) && fc_is_big(Mt, L.N_pad);
    uint32_t groups, trows;
    fc_shape(L.N_pad, a.fc_split_k || (big && big_remainder_split_k(L.N_pad)), &tl.split, &groups, &trows);
    static_assert(!WHOLE || (NARROW && GATHER == kRowsStaged), "in runs whose tiles split K, behind layer 0");
    const uint32_t first = big ? big_rows(Mt) : 0;
    const uint32_t mt_ = ceil_div(Mt - first, trows);
    tl.m0 = first + (local % mt_) * trows;
    tl.rows = min(trows, Mt - tl.m0);
    tl.n0 = (local / mt_) * tl.split * kBrickRows;
    const uint32_t nrb = (tl.rows + kBrickRows - 1) / kBrickRows;
    T* xout = (T*)act_of(a.act, L.out_buf) + (size_t)seg0 * a.S;
    auto row_of = [&](uint32_t block, uint32_t i, bool* real) {
        const uint32_t p0 = seg0 + tl.m0 + block * kBrickRows;
        const int32_t r = a.perm[p0 + i];
        *real = r >= 0;
        return a.row_src[r >= 0 ? r : a.perm[p0]];            // padding rows read the block's first row (always a real request) and discard it: no branch around the loads
    };
    if constexpr (!NARROW) {
        if (__builtin_expect(tl.split == 4, 1)) {
            if (__builtin_expect(nrb > 1, 1)) fc_tile<T, 2, GATHER, true>(a, tl, L, Mt, seg0, row_of, xout, smem);
            else fc_tile<T, 1, GATHER, true>(a, tl, L, Mt, seg0, row_of, xout, smem);
            return;
        }
    }
    const void* row = nullptr;
    bool row_ok = false;
    if (GATHER) {
        row = row_of(0, threadIdx.x & 31, &row_ok);
    }
    if constexpr (WHOLE) {                                    // (local / mt_ is 0)
        if (L.is_last && fc_whole(L.N_pad)) { fc_whole_tile<T>(a, tl, L, Mt, seg0, smem); return; }
    }
    fc_split_tile<T, GATHER>(a, tl, L, Mt, seg0, row, row_ok, xout, smem);
}

// ---- layer 0 of a small run, with the segmentation in it ------------------------------------------
__device__ __forceinline__ uint32_t entry_tiles(const BatchArgs& b, const uint4& f, uint32_t M)      // streaming FC tiles of a tenant, as the batcher counts them
{
    const bool sk = b.fc_split_k && f.x;
    const uint32_t groups = sk ? ((f.x >> 29) & 1 && b.fc_whole ? 1 : f.y / kBrickRows) : f.x & 0x1fffffffu, sh = sk || ((f.x >> 30) & 1) ? 5 : 6;
    return f.x >> 31 ? 0 : ((M + (1u << sh) - 1) >> sh) * groups;
}
// What the launches behind the first one read, by one wave: counts and offsets (a lane is a tenant), padding rows.
__device__ __forceinline__ void entry_publish(const BatchArgs& b, uint32_t lane, uint32_t M, uint32_t off, uint32_t padded, uint32_t total)
{
    if (lane < b.T) {
        b.M[lane] = M; b.off[lane] = off;
        if (M) { atomicAdd(&b.served[2 * lane], (unsigned long long)M); atomicAdd(&b.served[2 * lane + 1], 1ull); }
        for (uint32_t p = off + M; p < off + padded; ++p) b.perm[p] = -1;
    }
    if (lane == 63) b.off[b.T] = total;
    if (lane == 0) *b.big_layers = 0;
}
// ... and the tile lists of layers first, first + step, ...
__device__ __forceinline__ void entry_lists(const BatchArgs& b, uint32_t lane, uint32_t M, uint32_t first, uint32_t step)
{
    for (uint32_t l = first; l < b.n_layer_slots; l += step) {
        if (!((b.list_mask[l / kLayerGroup] >> (l % kLayerGroup)) & 1)) continue;
        const uint4 f = lane < b.T ? ((const uint4*)b.facts)[(size_t)l * b.T + lane] : uint4{0, 0, 0, 0};
        const uint32_t n = entry_tiles(b, f, M), incl = wave_inclusive_scan(n);
        uint32_t* base = b.tile_base + (size_t)l * (b.T + 1);
        if (lane < b.T) base[lane] = incl - n;
        if (lane == 63) base[b.T] = incl;
    }
}

// One submission of at most 256 rows, at most 64 tenants: the batcher's launch, one workgroup, is a sixth of such a pass.
// Here every wave of every workgroup works the segmentation out for itself, with the tenants in its lanes: the rows of a lane's tenant
// are a bit mask per 64 rows, from one ballot per id bit; tile counts and offsets are two wave scans, a tile's owner one
// ballot.  That takes one round trip to memory (ids, tenants, facts) where the tile list, the row order and the rows' addresses took
// three.  The last workgroup has no tile and writes what the launches behind this one read, as the batcher leaves it: counts, offsets,
// row order and the tile lists of layers 1 on (streaming FC tiles only: models with images are not served this way).
// 1 request to 8 tenants' 784-1024-1024-10 models: 23.8 -> 20.2 us, 64 fp32 requests to four 256-512-512-10 models 26.5 -> 23.1.
template <typename T, int ROWS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void fc_entry_kernel(GemmArgs a, BatchArgs b)
{
    constexpr uint32_t NIT = kEntryMaxRows / 64;
    __shared__ __attribute__((aligned(16))) uint8_t smem[kFcLdsBytes];
    __shared__ int32_t rows_of[4][kBrickRows];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_tenants = b.T, R = b.R;
    // a lane is a row of every 64, and a tenant
    int32_t id[NIT];
#pragma unroll
    for (uint32_t i = 0; i < NIT; ++i) {
        const uint32_t r = i * 64 + lane;
        id[i] = r < R ? (b.first.ids ? b.first.ids[r] : b.first.tenant) : -1;
    }
    const uint4 f0 = lane < n_tenants ? ((const uint4*)b.facts)[lane] : uint4{0, 0, 0, 0};
    // (every workgroup looks for itself: a run that is not captured serves what was registered when it was enqueued, which no registration since can change)
    const uint64_t registered = __ballot(lane < n_tenants && serves(b, b.tenants[lane]));
    uint64_t has[NIT];                                        // the rows of this lane's tenant
    uint32_t M = 0;
#pragma unroll
    for (uint32_t i = 0; i < NIT; ++i) {
        has[i] = 0;
        if (i * 64 >= R) continue;                            // uniform
        const uint32_t t = (uint32_t)id[i];
        const bool ok = t < n_tenants && ((registered >> t) & 1);
        uint64_t m = __ballot(ok);
#pragma unroll
        for (uint32_t bit = 0; bit < 6; ++bit) {
            const uint64_t s = __ballot((t >> bit) & 1);
            m &= (lane >> bit) & 1 ? s : ~s;
        }
        has[i] = m;
        M += (uint32_t)__popcll(m);
        id[i] = ok ? (int32_t)t : -1;
    }
    const uint32_t padded = ceil_div(M, kBrickRows) * kBrickRows, off_incl = wave_inclusive_scan(padded), off = off_incl - padded;

    if (blockIdx.x == gridDim.x - 1) {
        if (wave == 0) {
            entry_publish(b, lane, M, off, padded, off_incl);
        } else if (wave == 1) {
#pragma unroll
            for (uint32_t i = 0; i < NIT; ++i) {
                if (i * 64 >= R) break;
                const int32_t t = id[i], tl = max(t, 0);
                uint32_t rank = 0;                            // rows of the same tenant in front of this one
#pragma unroll
                for (uint32_t j = 0; j <= i; ++j) {
                    const uint64_t m = (uint64_t)(uint32_t)__shfl((int)(uint32_t)has[j], tl) | (uint64_t)(uint32_t)__shfl((int)(uint32_t)(has[j] >> 32), tl) << 32;
                    rank += (uint32_t)__popcll(j < i ? m : m & ((1ull << lane) - 1));
                }
                const uint32_t position = (uint32_t)__shfl((int)off, tl) + rank, r = i * 64 + lane;
                if (r < R) { b.row_tenant[r] = t; place_row(b, r, t, position); }
            }
        }
        entry_lists(b, lane, M, 1 + (wave + 2) % 4, 4);       // (waves 2 and 3, which have nothing else to do, first)
        return;
    }

    const uint32_t n = entry_tiles(b, f0, M), incl = wave_inclusive_scan(n);
    uint32_t idx;
    if (!logical_tile(__builtin_amdgcn_readlane(incl, 63), &idx)) return;
    Tile tl;
    tl.tenant = (uint32_t)__popcll(__ballot(incl <= idx));    // (a lane without a tenant holds the total)
    const LayerDev L = a.layers[tl.tenant * MT_MAX_LAYERS];
    const uint32_t Mt = __builtin_amdgcn_readlane(M, tl.tenant), seg0 = __builtin_amdgcn_readlane(off, tl.tenant), local = idx - __builtin_amdgcn_readlane(incl - n, tl.tenant);
    uint32_t groups, trows;
    fc_shape(L.N_pad, a.fc_split_k, &tl.split, &groups, &trows);
    const uint32_t mt_ = ceil_div(Mt, trows);
    tl.m0 = (local % mt_) * trows;
    tl.rows = min(trows, Mt - tl.m0);
    tl.n0 = (local / mt_) * tl.split * kBrickRows;
    // the tile's rows in submission order, for this wave's lanes
    uint32_t at = 0;
#pragma unroll
    for (uint32_t i = 0; i < NIT; ++i) {
        const uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)has[i], tl.tenant) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(has[i] >> 32), tl.tenant) << 32;
        const uint32_t p = at + (uint32_t)__popcll(m & ((1ull << lane) - 1)) - tl.m0;
        if ((m >> lane) & 1 && p < (uint32_t)kBrickRows) rows_of[wave][p] = (int32_t)(i * 64 + lane);
        at += (uint32_t)__popcll(m);
    }
    const bool row_ok = (lane & 31) < tl.rows;
    const int32_t r = rows_of[wave][row_ok ? lane & 31 : 0];
    const void* row = (const uint8_t*)b.first.src + (size_t)(uint32_t)r * b.first.row_stride * sizeof(T);
    fc_split_tile<T, ROWS>(a, tl, L, Mt, seg0, row, row_ok, (T*)act_of(a.act, L.out_buf) + (size_t)seg0 * a.S, smem);
}

// The same for one submission of at most 4096 rows and any tiles: the workgroup's waves take a quarter of the rows each, count them by tenant in LDS and, once the
// tile's tenant is known, note those that are the tile's.  A tile waits for ids and facts, the layer's row and the submitted rows, in place of the tile list, that row,
// the rows' addresses and the rows; the batcher's launch, alone on the chip for 5-7 us, is gone.  Passes and the line beside run_entry.  Bound as fc_kernel is: by the
// weight stream, behind 2-3 us until the first weight load.  (With the ids in registers and masks from ballots, as above, 16 unrolled steps of them spilled 91 registers
// and the tiles took half as long again.  Of 64 rows the first one's tenant is counted at once, every other row by an addition of its lane: without that, all rows one
// tenant's, 4096 requests 113 -> 123 us.)
template <typename T, int ROWS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void fc_entry_wide_kernel(GemmArgs a, BatchArgs b)
{
    constexpr uint32_t NIT = kEntryWideRows / 256;
    __shared__ __attribute__((aligned(16))) uint8_t smem[fc_lds_bytes<ROWS>()];
    __shared__ uint32_t counts[4][65];                        // (the last one: rows of no tenant)
    __shared__ int32_t rows_of[kTileRows];
    uint8_t* const ids = smem + kStageBytes;                  // every row's tenant (0xff: none); until the second stage is written, behind a barrier
    static_assert(kStageBytes + kEntryWideRows <= kFcLdsBytes && kEntryMaxTenants <= 64, "a byte per row");
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_tenants = b.T, R = b.R;
    const uint32_t per = ceil_div(R, 256), begin = wave * per * 64, chunks = begin < R ? min(per, ceil_div(R - begin, 64)) : 0;      // this wave's rows, 64 at a time
    int32_t id[NIT];
    if (b.first.ids) {
#pragma unroll
        for (uint32_t i = 0; i < NIT; ++i) id[i] = b.first.ids[min(begin + min(i, per - 1) * 64 + lane, R - 1)];
    } else {
#pragma unroll
        for (uint32_t i = 0; i < NIT; ++i) id[i] = b.first.tenant;
    }
    const uint4 f0 = lane < n_tenants ? ((const uint4*)b.facts)[lane] : uint4{0, 0, 0, 0};
    const uint64_t registered = __ballot(lane < n_tenants && serves(b, b.tenants[lane]));
    counts[wave][lane] = 0;
#pragma unroll
    for (uint32_t i = 0; i < NIT; ++i) {
        if (i >= chunks) break;                               // uniform
        const uint32_t t = (uint32_t)id[i], r = begin + i * 64 + lane;
        const bool ok = (r < R) & (t < n_tenants) & (((registered >> (t & 63)) & 1) != 0);
        // (lanes of one tenant would add one after the other: those of the first lane's are added at once)
        const uint32_t bin = ok ? t : 64, first = __builtin_amdgcn_readfirstlane(bin);
        const uint32_t same = (uint32_t)__popcll(__ballot(bin == first));
        if (bin != first || lane == 0) atomicAdd(&counts[wave][bin], lane == 0 ? same : 1u);
        ids[r] = ok ? (uint8_t)t : (uint8_t)0xff;
    }
    lds_barrier();
    uint32_t M = 0, before = 0;                               // this lane's tenant: its rows, and those of them in front of this wave's
#pragma unroll
    for (uint32_t w = 0; w < 4; ++w) {
        before = w == wave ? M : before;
        M += counts[w][lane];
    }
    const uint32_t padded = ceil_div(M, kBrickRows) * kBrickRows, off_incl = wave_inclusive_scan(padded), off = off_incl - padded;

    if (blockIdx.x == gridDim.x - 1) {                        // the batcher's part
        if (wave == 0) entry_publish(b, lane, M, off, padded, off_incl);
        entry_lists(b, lane, M, 1 + (wave + 3) % 4, 4);
        uint32_t at = off + before;                           // where the next row of this lane's tenant goes
#pragma unroll 1
        for (uint32_t i = 0; i < chunks; ++i) {
            const uint32_t r = begin + i * 64 + lane;
            const int32_t t = (int8_t)ids[r], tl = max(t, 0);
            uint64_t has = __ballot(t >= 0);                  // the rows of this lane's tenant among these 64
#pragma unroll
            for (uint32_t bit = 0; bit < 6; ++bit) {
                const uint64_t s = __ballot((t >> bit) & 1);
                has &= (lane >> bit) & 1 ? s : ~s;
            }
            const uint64_t same = (uint64_t)(uint32_t)__shfl((int)(uint32_t)has, tl) | (uint64_t)(uint32_t)__shfl((int)(uint32_t)(has >> 32), tl) << 32;
            const uint32_t position = (uint32_t)__shfl((int)at, tl) + (uint32_t)__popcll(same & ((1ull << lane) - 1));
            at += (uint32_t)__popcll(has);
            if (r < R) { b.row_tenant[r] = t; place_row(b, r, t, position); }
        }
        return;
    }

    const uint32_t n = entry_tiles(b, f0, M), incl = wave_inclusive_scan(n);
    uint32_t idx;
    if (!logical_tile(__builtin_amdgcn_readlane(incl, 63), &idx)) return;
    Tile tl;
    tl.tenant = (uint32_t)__popcll(__ballot(incl <= idx));    // (a lane without a tenant holds the total)
    const LayerDev L = a.layers[tl.tenant * MT_MAX_LAYERS];
    const uint32_t Mt = __builtin_amdgcn_readlane(M, tl.tenant), seg0 = __builtin_amdgcn_readlane(off, tl.tenant), local = idx - __builtin_amdgcn_readlane(incl - n, tl.tenant);
    uint32_t groups, trows;
    fc_shape(L.N_pad, a.fc_split_k, &tl.split, &groups, &trows);
    const uint32_t mt_ = ceil_div(Mt, trows);
    tl.m0 = (local % mt_) * trows;
    tl.rows = min(trows, Mt - tl.m0);
    tl.n0 = (local / mt_) * tl.split * kBrickRows;
    uint32_t at = __builtin_amdgcn_readlane(before, tl.tenant);
#pragma unroll 1
    for (uint32_t i = 0; i < chunks; ++i) {
        const uint64_t m = __ballot(ids[begin + i * 64 + lane] == tl.tenant);
        const uint32_t p = at + (uint32_t)__popcll(m & ((1ull << lane) - 1)) - tl.m0;
        if (((m >> lane) & 1) && p < tl.rows) rows_of[p] = (int32_t)(begin + i * 64 + lane);
        at += (uint32_t)__popcll(m);
    }
    lds_barrier();
    auto row_of = [&](uint32_t block, uint32_t i, bool* real) -> const void* {
        const uint32_t p = block * kBrickRows + i;
        *real = p < tl.rows;
        const int32_t r = rows_of[*real ? p : block * kBrickRows];
        return (const uint8_t*)b.first.src + (size_t)(uint32_t)r * b.first.row_stride * sizeof(T);
    };
    T* xout = (T*)act_of(a.act, L.out_buf) + (size_t)seg0 * a.S;
    if (__builtin_expect(tl.split == 4, 1)) {
        if (__builtin_expect(tl.rows > (uint32_t)kBrickRows, 1)) fc_tile<T, 2, ROWS, false>(a, tl, L, Mt, seg0, row_of, xout, smem);
        else fc_tile<T, 1, ROWS, false>(a, tl, L, Mt, seg0, row_of, xout, smem);
        return;
    }
    bool row_ok;
    const void* row = row_of(0, lane & 31, &row_ok);
    fc_split_tile<T, ROWS>(a, tl, L, Mt, seg0, row, row_ok, xout, smem);
}

// ---- launcher ------------------------------------------------------------
template <typename T>
static void launch_fc_t(const GemmArgs& a, bool narrow, uint32_t grid, hipStream_t s)
{
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, a); };
    auto with = [&](auto rows_) {
        constexpr int rows = decltype(rows_)::value;
        if (!narrow) launch(fc_kernel<T, false, rows, false>);
        else if (a.T <= 64) launch(fc_kernel<T, true, rows, true>);
        else launch(fc_kernel<T, true, rows, false>);
    };
    if (a.fc_whole && a.T <= 64) { launch(fc_kernel<T, true, kRowsStaged, true, true>); return; }
    if (a.fc_whole) { launch(fc_kernel<T, true, kRowsStaged, false, true>); return; }
    if (a.gather == kRowsAny) with(std::integral_constant<int, kRowsAny>{});
    else if (a.gather) with(std::integral_constant<int, kRowsChunked>{});
    else with(std::integral_constant<int, kRowsStaged>{});
}

// grid: a bound of the tiles; eight workgroups more, of which the last does the batcher's part
hipError_t launch_fc_entry(const GemmArgs& a, const BatchArgs& b, uint32_t dtype, bool wide, uint32_t grid, hipStream_t s)
{
    if (b.R > kEntryWideRows || b.T > kEntryMaxTenants || (!wide && b.R > kEntryMaxRows)) return hipErrorInvalidValue;
    grid = (grid + 7) / 8 * 8 + 8;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, a, b); };
    auto with = [&](auto rows_) {
        constexpr int rows = decltype(rows_)::value;
        if (wide) { if (dtype == MT_BF16) launch(fc_entry_wide_kernel<__bf16, rows>); else launch(fc_entry_wide_kernel<float, rows>); }
        else if (dtype == MT_BF16) launch(fc_entry_kernel<__bf16, rows>);
        else launch(fc_entry_kernel<float, rows>);
    };
    if (a.gather == kRowsAny) with(std::integral_constant<int, kRowsAny>{}); else with(std::integral_constant<int, kRowsChunked>{});
    return hipGetLastError();
}

// narrow: every tile of the launch splits K
hipError_t launch_fc(const GemmArgs& a, uint32_t dtype, bool narrow, uint32_t grid, hipStream_t s)
{
    if (grid == 0) return hipSuccess;
    if (a.fc_whole && (!narrow || a.gather != kRowsStaged)) return hipErrorInvalidValue;
    grid = (grid + 7) / 8 * 8;
    if (dtype == MT_BF16) launch_fc_t<__bf16>(a, narrow, grid, s); else launch_fc_t<float>(a, narrow, grid, s);
    return hipGetLastError();
}

}  // namespace mt

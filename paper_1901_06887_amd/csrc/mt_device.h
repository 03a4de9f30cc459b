// Device-side helpers shared by the kernels of the multi-tenant worker runtime, written for
// gfx950 (CDNA4, wave64).  The kernels live in:
//
//   batcher.hip     batcher_kernel (+ rank_kernel, place_kernel for large batches): tenant
//                   segmentation of the pending requests (counts, 32-aligned offsets, stable
//                   permutation) and the per-layer grouped-work tile lists, on device
//   fc_stream.hip   fc_kernel: one FC layer index for all tenants, weight-streaming tiles: weight
//                   bricks go from memory into MFMA operands through a register ring, activation
//                   bricks are shared through LDS; fused bias + activation (+ rounding), brick
//                   output, fp32 logits, or softmax/argmax where one tile holds all classes (at most
//                   128).  Narrow layers and small runs take tiles of 32 rows whose waves split K;
//                   fc_entry_kernel: layer 0 of a small run with the segmentation in it
//   fc_big.hip      fc_big_walk_kernel / fc_big_kernel: the same layer index, compute-bound tenant-layers:
//                   256x256 tiles, both operands through an LDS ring filled by direct global->LDS loads;
//                   one workgroup per compute unit walks the tiles (or, for short K, one workgroup per tile)
//   conv.hip        conv_kernel (layers at most 32 channels wide: every wave gathers its own
//                   pixels) and conv_lds_kernel (wider layers: activation bricks gathered once
//                   per tile into LDS and shared by waves side by side over channels; pools on
//                   the way out where it can) and conv_img_kernel (layers whose tiles are whole
//                   output rows of an image or whole small images: the tile's input rows are
//                   copied to LDS once and every tap is read from there) and conv_split_kernel
//                   (launches of few tiles: 32 pixels and 32 channels to a tile, whose 4 to 16 waves
//                   share K): implicit-GEMM convolution for all tenants
//   conv_first.hip  conv_first_kernel: first convolutions of images with at most four channels, from the
//                   submitted images themselves; takes the max-pool behind the layer with it; conv_pair_kernel: those and
//                   the 3x3 convolution behind them
//   small.hip       gather_kernel / gather_image_kernel (submitted rows -> bricks / padded NHWC),
//                   gap_kernel (global average pooling), head_kernel (softmax + argmax in
//                   submission order), copy_kernel (the yardstick for byte counters)
//
// A DNN is a fixed sequence of layers applied in turn (paper, section 1.1); a worker
// hosts many tenants' DNNs and multiplexes their requests (section 3).  The grouping
// of all tenants' work for one layer index into one launch is this runtime's way of
// doing that multiplexing on one GPU.
#pragma once
#include <algorithm>
#include "mt_internal.h"

namespace mt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kBatchThreads = 1024;
constexpr uint32_t kMaxTenantsPadded = 2048;
constexpr uint32_t kSegsInLds = 64;

__device__ __forceinline__ uint32_t ceil_div(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

// One of the run's activation buffers by its number (a layer names the ones it reads and writes);
// selects instead of indexing, so that the kernel arguments stay in scalar registers.
__device__ __forceinline__ void* act_of(const ActBufs& b, uint32_t i)
{
    return i == 0 ? b.p[0] : i == 1 ? b.p[1] : i == 2 ? b.p[2] : b.p[3];
}

// A wave-uniform value in scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t x)
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)x) | (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(x >> 32)) << 32;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also drains every global
// load in flight (it fences all address spaces), which would empty the prefetch rings of the
// GEMM loops at each LDS hand-over; here only the LDS counter is waited on.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Direct global -> LDS load of 16 bytes per lane: lane l's bytes land at lds_dst + 16 l
// (lds_dst is wave-uniform and travels in M0).  Written as asm on purpose: the compiler's
// wait-count pass gives up exact vmcnt bookkeeping (it waits for zero) once it sees such loads
// in flight together with ordinary register loads.  A kernel that uses this helper issues no
// register loads while such loads are in flight and waits for the LDS data itself, with an
// explicit vmcnt before the barrier that publishes it.  Nothing else keeps a value in M0.
__device__ __forceinline__ void lds_dma16(const __attribute__((address_space(1))) void* src, void* lds_dst)
{
    const uint32_t m0v = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds_dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(m0v), "v"(src) : "memory", "m0");
}

// The same through a buffer descriptor: lane l's 16 bytes at byte `voff` of the buffer land at lds_dst + 16 l, and a
// lane whose offset lies outside the buffer gets zeros (the hardware's range check of untyped buffers; checked on
// the device: the lane layout is that of the global form, offsets from num_records - 15 on deliver zeros).
// The descriptor: base address, stride 0 (untyped), size in bytes, 32-bit data format.
__device__ __forceinline__ u32x4 buffer_descriptor(const void* base, uint32_t bytes)
{
    const uint64_t b = (uint64_t)base;
    u32x4 d;
    d[0] = __builtin_amdgcn_readfirstlane((uint32_t)b);
    d[1] = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32) & 0xffffu);
    d[2] = __builtin_amdgcn_readfirstlane(bytes);
    d[3] = 0x00020000u;
    return d;
}
__device__ __forceinline__ void lds_dma16_buffer(const u32x4& desc, uint32_t voff, void* lds_dst)
{
    const uint32_t m0v = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds_dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(m0v), "v"(voff), "s"(desc) : "memory", "m0");
}

// 16 bytes per lane through the XCD's L2 to memory (agent scope).  An ordinary store stays in L2 and is written back when the kernel
// ends, with nothing else running: a convolution launch that writes some 10-50 MB ends 1.2-1.7 us earlier with these (residual nets, 64
// images, 19 such launches: 30.5 -> 28.8, 36.3 -> 34.8, 20.0 -> 18.4 us).  Passes that write all the time lose (image gather 26 -> 37 us).
// In asm: the compiler has no store of this size and scope; its wait counts only become stricter by stores that it does not know of.
// Two wait states, in the asm because the compiler does not know that it is a store: from gfx940 on a vector instruction
// may overwrite the data of a store wider than 8 bytes only behind them.
__device__ __forceinline__ void store_through(u32x4* dst, const u32x4& v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(dst), "v"(v) : "memory");
}

// Inclusive prefix sums across lanes with data-parallel-primitive moves (no LDS traffic): shifts
// by 1, 2, 4, 8 inside each row of 16 lanes (lanes without a source add 0), then lane 15 of rows
// 0 and 2 is added to rows 1 and 3, then lane 31 to the upper half.
#define MT_DPP_ADD(v, ctrl, rows) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false)
__device__ __forceinline__ uint32_t row16_inclusive_scan(uint32_t v)
{
    MT_DPP_ADD(v, 0x111, 0xf); MT_DPP_ADD(v, 0x112, 0xf); MT_DPP_ADD(v, 0x114, 0xf); MT_DPP_ADD(v, 0x118, 0xf);   // row_shr:1,2,4,8
    return v;
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v)
{
    v = row16_inclusive_scan(v);
    MT_DPP_ADD(v, 0x142, 0xa);      // row_bcast:15 into rows 1 and 3
    MT_DPP_ADD(v, 0x143, 0xc);      // row_bcast:31 into rows 2 and 3
    return v;
}
#undef MT_DPP_ADD

// How an FC layer is cut into workgroup tiles: `split` column blocks side by side per
// group (the four waves cover them; with split < 4 they also split K), `groups` column
// groups, and the rows of a tile: 64 normally, 32 for the K-split shapes (layers with at
// most 64 outputs): their tiles are short-lived and latency bound, so more and smaller ones
// finish sooner.
__device__ __forceinline__ void fc_shape(uint32_t n_pad, uint32_t split_k, uint32_t* split, uint32_t* groups, uint32_t* tile_rows)
{
    const uint32_t nblk = n_pad / kBrickRows;
    uint32_t s = split_k ? 1u : (nblk >= 3 ? 4u : nblk);
    *split = s;
    *groups = ceil_div(nblk, s);
    *tile_rows = s == 4 ? kTileRows : kTileRows / 2;
}

// ---- shared pieces of the GEMM kernels -----------------------------------------------------
// GELU(x) = x * Phi(x) with the exact (erf) definition, evaluated through the complementary
// error function of z = |x|/sqrt(2) (Abramowitz & Stegun 7.1.26: a degree-5 polynomial in
// t = 1/(1 + p z) times exp(-z^2), absolute error below 1.5e-7).  With h = erfc(z)/2, Phi is
// 1 - h on the positive side and h on the negative one, so x Phi(x) = max(x, 0) - |x| h on both
// (the small negative tail keeps its relative accuracy).  z is carried pre-scaled by
// sqrt(log2 e) so that exp(-z^2) is one multiply and one exp2; the 1/2 sits in the polynomial's
// coefficients.  The error is far below half a bfloat16 ulp of the result, and a library erf
// costs four times as much, which showed in the epilogue of the compute-bound tiles.
// max(x, 0) in one instruction: the compiler's own maximum first quiets a possible signalling NaN with a second
// v_max (it cannot know that MFMA results hold none), one issue slot in fifteen of the GELU below.
__device__ __forceinline__ float max0(float x)
{
    float r;
    asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(x));
    return r;
}

__device__ __forceinline__ float gelu(float x)
{
    constexpr float kScale = 0.84932180028801904f;           // sqrt(log2(e) / 2): zs = z * sqrt(log2 e)
    constexpr float kP = 0.3275911f / 1.2011224087864498f;   // p / sqrt(log2 e)
    const float ax = fabsf(x);
    const float zs = ax * kScale;
    const float t = __builtin_amdgcn_rcpf(fmaf(kP, zs, 1.0f));   // one instruction, within 1 ulp: far inside the formula's own 1.5e-7
    const float poly = t * (0.127414796f + t * (-0.142248368f + t * (0.7107068705f + t * (-0.7265760135f + t * 0.5307027145f))));
    const float h = poly * __builtin_amdgcn_exp2f(-zs * zs);
    return fmaf(-ax, h, max0(x));
}

__device__ __forceinline__ float activate(float z, uint32_t act)
{
    if (act == MT_ACT_RELU) return max0(z);
    if (act == MT_ACT_GELU) return gelu(z);
    return z;
}

// The same on a block of values, with the choice made once, outside the loops.
template <int G>
__device__ __forceinline__ void activate_block(f32x4 (&y)[G], uint32_t act)
{
    if (act == MT_ACT_GELU) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) y[g][e] = gelu(y[g][e]);
    } else if (act == MT_ACT_RELU) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) y[g][e] = max0(y[g][e]);
    }
}

// A residual addition done by the convolution in front of it.  y holds this lane's four runs of four
// channels (8 g + 4 lh + {0..3}) of one pixel, bias and the convolution's activation applied: they are
// rounded to T, as the addition would have read them, the other operand's values of the same pixel and
// channels are added, and the addition's activation follows.  `skip` points into the other operand
// where `out` points into the output (null for lanes without a pixel); channels from `nvalid` on do not exist.
template <typename T>
__device__ __forceinline__ void add_residual(f32x4 (&y)[4], const T* skip, uint32_t lh, uint32_t nvalid, uint32_t act)
{
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        if (skip != nullptr && 8 * g + 4 * lh < nvalid) {        // channel counts are multiples of 8: a run exists whole or not at all
            T sv[4];
            if constexpr (sizeof(T) == 2) *(uint64_t*)sv = *(const uint64_t*)(skip + 8 * g + 4 * lh);
            else *(u32x4*)sv = *(const u32x4*)(skip + 8 * g + 4 * lh);
#pragma unroll
            for (int e = 0; e < 4; ++e) y[g][e] = (float)(T)y[g][e] + (float)sv[e];
        }
    }
    activate_block<4>(y, act);
}

// The same in two parts: the other operand is asked for long before the sums are there, as a memory trip per unit (1.5-2 thousand clocks) at the end of a tile
// has nothing to hide behind.  Lanes and channels that do not exist read some that do (`any`: the tenant's first row).
template <typename T> struct Residual {
    typedef T vec __attribute__((ext_vector_type(4)));
    vec v[4];
    __device__ __forceinline__ void fetch(const T* skip, const T* any, uint32_t lh, uint32_t nvalid)
    {
        typedef const __attribute__((address_space(1))) vec* vptr_t;
#pragma unroll
        for (uint32_t g = 0; g < 4; ++g) {
            const uint32_t c = 8 * g + 4 * lh;
            v[g] = *(vptr_t)(skip ? skip + (c < nvalid ? c : 0) : any);
        }
    }
    __device__ __forceinline__ void add(f32x4 (&y)[4], uint32_t act) const
    {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) y[g][e] = (float)(T)y[g][e] + (float)v[g][e];
        activate_block<4>(y, act);
    }
};

// Quotient and remainder by a wave-uniform divisor; image sizes are mostly powers of two, and a
// general 32-bit division costs some thirty vector instructions per lane.
__device__ __forceinline__ void divmod_uniform(uint32_t x, uint32_t d, uint32_t* q, uint32_t* r)
{
    if ((d & (d - 1)) == 0) { *q = x >> __builtin_ctz(d); *r = x & (d - 1); }
    else { *q = x / d; *r = x - *q * d; }
}

// ---- NHWC store of one 32-pixel x 32-channel unit held in the transposed accumulator layout ----
// After an MFMA with the filter brick as row operand, lane (li, lh) holds channels 8g + 4 lh +
// {0..3} of pixel li: stored from there, a wave instruction writes 64 separate 8- or 16-byte
// pieces, and the texture path counts (and takes time for) every one of them; the counters
// showed the convolution kernels bound by exactly that rate.  So the unit goes through a
// wave-private LDS scratch as [pixel][channel] rows and is read back so that consecutive
// lanes hold consecutive 16-byte chunks of a pixel's row: a pixel's 64 (bf16) or 128 (fp32)
// bytes leave in one piece.  Each pixel's destination travels through the scratch as well
// (null for pixels past the end), so the storing lane needs no index arithmetic.
template <typename T> constexpr uint32_t unit_row_stride() { return kBrickRows * sizeof(T) + 16; }
template <typename T> constexpr uint32_t unit_scratch_bytes() { return kBrickRows * unit_row_stride<T>() + kBrickRows * 8; }

// Four values rounded to the element type, as they lie in memory.  (Converted as a vector: two instructions for bf16.  Element by element the compiler
// converts each for itself and puts the pairs together again.)
template <typename T> struct Packed4;
template <> struct Packed4<__bf16> {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ uint64_t of(const f32x4& y) { return __builtin_bit_cast(uint64_t, __builtin_convertvector(y, bf16x4)); }
};
template <> struct Packed4<float> {
    static __device__ __forceinline__ f32x4 of(const f32x4& y) { return y; }
};
template <typename T> __device__ __forceinline__ void put4(void* p, const f32x4& y)
{
    auto v = Packed4<T>::of(y);
    *(decltype(v)*)p = v;
}

template <typename T>
__device__ __forceinline__ void store_unit_nhwc(const f32x4 (&y)[4], T* my_pixel_out, uint32_t n_valid, uint32_t through, uint8_t* scratch)
{
    constexpr uint32_t EPC = 16 / sizeof(T), RS = unit_row_stride<T>();
    constexpr uint32_t CP = kBrickRows / EPC;                       // 16-byte chunks per pixel row: 4 (bf16) or 8 (fp32)
    const uint32_t lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    T** dests = (T**)(scratch + kBrickRows * RS);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        put4<T>(scratch + li * RS + (8 * g + 4 * lh) * sizeof(T), y[g]);
    }
    if (lh == 0) dests[li] = my_pixel_out;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // the wave's own LDS writes have landed
#pragma unroll
    for (uint32_t pass = 0; pass < CP / 2; ++pass) {
        const uint32_t px = pass * (64 / CP) + lane / CP, ch = lane % CP;
        T* dst = dests[px];
        const u32x4 v = *(const u32x4*)(scratch + px * RS + ch * 16);
        if (dst != nullptr && ch * EPC < n_valid) {
            if (through) store_through((u32x4*)(dst + ch * EPC), v);      // the same for the whole launch
            else *(u32x4*)(dst + ch * EPC) = v;
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // reads done before the next unit overwrites the scratch
}

// The label of a row whose classes were compared in parts with `>` from -inf on: best is the first class with the largest logit, 0x7fffffff
// where none is above -inf; z0: the first class's logit.  A walk from the first class stays there if its logit is NaN or nothing is larger.
__device__ __forceinline__ int32_t head_label(int32_t best, float z0) { return best == 0x7fffffff || z0 != z0 ? 0 : best; }

template <typename T> struct Mma;
// bf16: one 16-byte chunk is a whole MFMA operand (8 consecutive k of one row).
template <> struct Mma<__bf16> {
    static __device__ __forceinline__ void run(f32x16& acc, const u32x4& a, const u32x4& b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
    }
};
// fp32: a chunk holds 4 consecutive k; four 32x32x2 MFMAs consume it, the two lane halves
// supplying the two k slots of each (the same k assignment on both operands).
template <> struct Mma<float> {
    static __device__ __forceinline__ void run(f32x16& acc, const u32x4& a, const u32x4& b)
    {
        const f32x4 af = __builtin_bit_cast(f32x4, a), bf = __builtin_bit_cast(f32x4, b);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[0], bf[0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[1], bf[1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[2], bf[2], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[3], bf[3], acc, 0, 0, 0);
    }
};

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

// What a workgroup works on, derived from its block index and the list's tile_base array.
struct Tile {
    uint32_t tenant, m0, rows, n0, split;
};

// XCD-aware numbering: consecutive block indices go to different XCDs (each with its own L2),
// so the logical tile index is chosen such that every XCD gets one contiguous run of tiles;
// tiles that re-read the same weight panel (the row tiles of one column group) then
// share an L2.  Returns false for blocks past the end of the list.
__device__ __forceinline__ bool logical_tile(uint32_t n_tiles, uint32_t* logical)
{
    const uint32_t per_xcd = (n_tiles + 7) / 8, b = blockIdx.x;
    *logical = (b & 7) * per_xcd + (b >> 3);
    return (b >> 3) < per_xcd && *logical < n_tiles;
}

// Variant for the big-tile kernel: the tile order is dealt to the XCDs in chunks of kXcdChunk
// tiles (round robin), so that at any time the whole GPU works on a narrow window of the order
// (about two tenants' panels, which fit the memory-side cache) while the tiles that run together
// on one XCD are still neighbours (L2 reuse).  The grid must be a multiple of 8 * kXcdChunk.
constexpr uint32_t kXcdChunk = 64;
__device__ __forceinline__ bool logical_tile_chunked(uint32_t n_tiles, uint32_t* logical)
{
    const uint32_t b = blockIdx.x, xcd = b & 7, i = b >> 3;
    *logical = ((i / kXcdChunk) * 8 + xcd) * kXcdChunk + (i % kXcdChunk);
    return *logical < n_tiles;
}

// Tenant that owns logical tile `idx` by binary search over a copy of the list in LDS: last t with
// base[t] <= idx (base[T] > idx).  Kept for the big-tile kernel, whose tiles run for ~100 us and
// whose wait counts the compiler only keeps exact while the kernel issues no other register loads
// than the one staging loop at its head.
__device__ __forceinline__ uint32_t find_tenant(const uint32_t* base, uint32_t T, uint32_t idx)
{
    uint32_t lo = 0, hi = T;
    while (hi - lo > 1) { const uint32_t mid = (lo + hi) >> 1; if (base[mid] <= idx) lo = mid; else hi = mid; }
    return lo;
}

// Tenant that owns a logical tile.  A tile list base[0..T] is non-decreasing with base[0] = 0 and
// base[T] = the number of tiles, so the owner of tile idx is the number of entries base[1..T]
// that are <= idx.  The workgroup counts them together: every thread fetches its entries
// (tile_owner_fetch, all loads issued before anything waits, and before the tile index is
// known), the waves count with one ballot per entry slot and add their counts through `part`
// (LDS, one word per wave, not reused by the caller: no second barrier is needed).  One memory
// round trip and one barrier; a binary search over a copy of the list in LDS took a dozen
// dependent LDS reads and two barriers at the head of every tile.
template <uint32_t THREADS>
struct TileOwner {
    static constexpr uint32_t SLOTS = kMaxTenantsPadded / THREADS;
    uint32_t v[SLOTS];
    __device__ __forceinline__ void fetch(const uint32_t* __restrict__ base, uint32_t T)
    {
#pragma unroll
        for (uint32_t s = 0; s < SLOTS; ++s) {
            const uint32_t j = 1 + s * THREADS + threadIdx.x;
            v[s] = 0xffffffffu;
            if (s * THREADS < T && j <= T) v[s] = base[j];
        }
    }
    // wave-uniform result; every thread of the workgroup must call it
    __device__ __forceinline__ uint32_t owner(uint32_t T, uint32_t idx, uint32_t* part) const
    {
        uint32_t cnt = 0;
#pragma unroll
        for (uint32_t s = 0; s < SLOTS; ++s)
            if (s * THREADS < T) cnt += (uint32_t)__builtin_popcountll(__ballot(v[s] <= idx));
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = cnt;
        __syncthreads();
        uint32_t t = 0;
#pragma unroll
        for (uint32_t w = 0; w < THREADS / 64; ++w) t += part[w];
        return __builtin_amdgcn_readfirstlane(t);
    }
};

// The same, together with what a tile needs to know of its tenant: the layer's row, the tenant's requests and first packed row, and its first tile.  With at most
// TENANTS tenants (0: any number, by loads of its own) the workgroup fetches those of all of them beside the tile list, a 16-byte piece or two per thread, and finds
// its own in LDS: one trip to memory at the head of a tile instead of two that depend on each other.
// A launch of few tiles lasts as long as its chain of trips: residual nets of one request 161.9 -> 151.4 us a pass, MLPs, CNNs and residual nets side by side
// 193.8 -> 182.0, residual nets of 64 images 531 -> 518, one request to an MLP 20.3 -> 19.7.  LDS: ahead_bytes(), not read behind the next barrier.
constexpr uint32_t kRowWords = sizeof(LayerDev) / 4, kFactsWords = kRowWords + 4;      // of a tenant's row; with three more, and padding
constexpr uint32_t ahead_bytes(uint32_t tenants = 64) { return tenants * kFactsWords * 4; }
template <uint32_t THREADS, uint32_t TENANTS = 64>
struct TileLookup {
    static constexpr uint32_t PER = kRowWords / 4, PIECES = TENANTS ? (TENANTS * PER + THREADS - 1) / THREADS : 1;      // 16-byte pieces of a row; of a thread
    static_assert(TENANTS <= 64 && kFactsWords <= 64, "a tenant, and a word, per lane");
    TileOwner<THREADS> list;
    u32x4 piece[PIECES];
    uint32_t first_tile, requests, off;
    __device__ __forceinline__ void fetch(const GemmArgs& a)
    {
        if constexpr (TENANTS == 0) {
            list.fetch(a.tile_base, a.T);
        } else {
            const uint32_t tid = threadIdx.x, lane = tid & 63;
            list.v[0] = lane < a.T ? a.tile_base[1 + lane] : 0xffffffffu;              // every wave counts for itself
#pragma unroll
            for (uint32_t i = 0; i < PIECES; ++i) {
                const uint32_t q = i * THREADS + tid, t = q / PER, c = q % PER;
                if (t < a.T) piece[i] = ((const u32x4*)(a.layers + (t * MT_MAX_LAYERS + a.layer)))[c];
            }
            if (tid < a.T) { requests = a.M[tid]; off = a.off[tid]; first_tile = a.tile_base[tid]; }
        }
    }
    // wave-uniform results; every thread of the workgroup must call it
    __device__ __forceinline__ void find(const GemmArgs& a, uint32_t idx, uint32_t* part, uint8_t* lds, uint32_t* tenant, LayerDev* L, uint32_t* Mt, uint32_t* seg0, uint32_t* local) const
    {
        if constexpr (TENANTS == 0) {
            const uint32_t t = list.owner(a.T, idx, part);                              // uniform: the tenant's facts come through scalar loads
            *tenant = t;
            *L = a.layers[t * MT_MAX_LAYERS + a.layer];
            *Mt = a.M[t]; *seg0 = a.off[t]; *local = idx - a.tile_base[t];
        } else {
            const uint32_t tid = threadIdx.x, lane = tid & 63;
            uint32_t* words = (uint32_t*)lds;
#pragma unroll
            for (uint32_t i = 0; i < PIECES; ++i) {
                const uint32_t q = i * THREADS + tid, t = q / PER, c = q % PER;
                if (t < a.T) *(u32x4*)(words + t * kFactsWords + c * 4) = piece[i];
            }
            if (tid < a.T) {
                uint32_t* w = words + tid * kFactsWords + kRowWords;
                w[0] = requests; w[1] = off; w[2] = first_tile;
            }
            const uint32_t t = (uint32_t)__builtin_popcountll(__ballot(list.v[0] <= idx));
            *tenant = t;
            lds_barrier();
            const uint32_t word = words[t * kFactsWords + min(lane, kFactsWords - 1)];
            struct Words { uint32_t w[kRowWords]; } row;
#pragma unroll
            for (uint32_t i = 0; i < kRowWords; ++i) row.w[i] = __builtin_amdgcn_readlane(word, i);
            *L = __builtin_bit_cast(LayerDev, row);
            *Mt = __builtin_amdgcn_readlane(word, kRowWords); *seg0 = __builtin_amdgcn_readlane(word, kRowWords + 1); *local = idx - __builtin_amdgcn_readlane(word, kRowWords + 2);
        }
    }
};

}  // namespace mt

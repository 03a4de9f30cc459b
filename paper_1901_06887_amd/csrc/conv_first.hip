// Convolutions that read the submitted images themselves (see mt_device.h for the overview).
#include "mt_device.h"
#include <type_traits>

namespace mt {

// A model's first layer, a 1x1, 3x3 or 7x7 convolution of images with at most four channels.  Run like the other
// convolutions it needs the images staged with eight channels a pixel (a pass of its own) and reads every byte of that once
// per tap through the texture path.  Here a workgroup copies the rows that a tile of whole output rows needs from the submitted image
// into a frame in LDS, four channels (8 or 16 bytes) a pixel and zeros around the image, and reads its MFMA operands from there.  The
// filters of a wave's block of 32 channels stay in its registers.
// POOL: a max-pool that is the layer's only reader is done here as well (LayerDev::first_pool): the convolution's rows, rounded as they
// would have been stored, never leave the registers.  A tile is rows of the pool's output then, a wave walks down 32 columns of
// the convolution's output with the two rows above in registers, takes the vertical maxima from those and the horizontal
// ones from its neighbour lanes.
//
// bf16: the sums are to the bit those of the staged path, which takes two taps of eight channels a k step, one in each half of
// the wave: so does this one, with the lower four channels of each.  Filters of two steps share a register quad; the
// operand's other half is zero (it does not matter to the bits in which half of a lane's eight elements the four lie; with
// finite filters, which is what the host lets through).  fp32: a lane's 16 bytes are one tap, a step takes two of a kernel row.
//
// 64 images of 224x224x3 through 7x7x64 at stride 2 and a 3x3 max-pool: staging 27.5, convolution 83.8 and pool 27.1 us -> 48 (MFMAs alone: 22 at
// the clock they leave; of a row of a wave's column some 800 clocks MFMAs and 500 vector instructions, four waves to a SIMD; 8-9 us until
// the first MFMA).  2048 images of 32x32x3 through 3x3x32: 15.5 + 51.9 -> 33 (134 MB written: 4.1 TB/s).  150 fp32 images of 29x35x3 through
// 3x3x24: 5.7 + 16.4 -> 14.5.  One image of 224x224: 6.9 + 10.6 + 10.2 -> 10.4, and two launches fewer.
// Tried: rows in a ring in LDS and maxima from there, the next rows prefetched into registers (88 us: two barriers a row, spills at 128 registers);
// maxima of bf16 values as floats (58 us: 230 vector instructions for what 60 of packed 16-bit integers do).
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// A submitted row is aligned to its elements only.
template <typename T> struct SubmittedDword;
template <> struct SubmittedDword<__bf16> { typedef uint32_t type __attribute__((aligned(2))); };
template <> struct SubmittedDword<float> { typedef uint32_t type; };

// registers (16 bytes a lane) that hold a block's filters, taps as they lie: four taps (bf16) or two of a kernel row (fp32) to a register quad
template <typename T, uint32_t KS> constexpr uint32_t first_quads() { return sizeof(T) == 2 ? (KS * KS + 3) / 4 : KS * ((KS + 1) / 2); }

// This wave's filters from where they are packed for the other kernels: k = tap * 8 + channel in bricks of 32 output channels, so a
// tap's four channels are the first 8 or 16 bytes at tap * 32 * 8 elements + output channel * 16 bytes.  Taps that do not exist: zero.
template <typename T, uint32_t KS, uint32_t N>
__device__ __forceinline__ void load_filters(u32x4 (&filters)[N], const uint8_t* block)
{
    constexpr uint32_t kTapBytes = kBrickRows * kChanPad * sizeof(T), taps = KS * KS;
    typedef const __attribute__((address_space(1))) uint8_t* bptr_t;
    const uint32_t lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    bptr_t at = (bptr_t)block + li * 16;
    if constexpr (sizeof(T) == 2) {
        typedef const __attribute__((address_space(1))) u32x2* qptr_t;
#pragma unroll
        for (uint32_t q = 0; q < first_quads<T, KS>(); ++q) {
            const uint32_t t0 = 4 * q + lh, t1 = t0 + 2;
            u32x2 lo = *(qptr_t)(at + min(t0, taps - 1) * kTapBytes), hi = *(qptr_t)(at + min(t1, taps - 1) * kTapBytes);
            if (4 * q + 3 >= taps) {
                lo = t0 < taps ? lo : u32x2{0, 0};
                hi = t1 < taps ? hi : u32x2{0, 0};
            }
            filters[q] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
    } else {
        typedef const __attribute__((address_space(1))) u32x4* fptr_t;
        constexpr uint32_t S = (KS + 1) / 2;
#pragma unroll
        for (uint32_t kh = 0; kh < KS; ++kh)
#pragma unroll
            for (uint32_t j = 0; j < S; ++j) {
                const uint32_t kw = 2 * j + lh;
                u32x4 f = *(fptr_t)(at + (kh * KS + min(kw, KS - 1)) * kTapBytes);
                if (j == S - 1) f = kw < KS ? f : u32x4{0, 0, 0, 0};
                filters[kh * S + j] = f;
            }
    }
}

// 32 pixels x 32 channels of the convolution: acc += filters x window, `at`: where the frame holds the top-left tap of this lane's
// pixel.  Operands are read AHEAD steps in front of their MFMAs (fences: left alone the compiler reads the whole window first).
template <typename T, uint32_t KS, uint32_t N>
__device__ __forceinline__ void first_window(f32x16& acc, const u32x4 (&filters)[N], const uint8_t* at, uint32_t row_bytes)
{
    constexpr uint32_t PXB = 4 * sizeof(T), AHEAD = 4;
    const uint32_t lh = (threadIdx.x & 63) >> 5;
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
    if constexpr (sizeof(T) == 2) {
        constexpr uint32_t taps = KS * KS, S = (taps + 1) / 2;
        // step s takes taps 2s and 2s + 1, one in each half of the wave: neighbours in a kernel row, or the end of one and the start of the next
        const uint8_t* in_row = at + lh * PXB;
        const uint8_t* across = at + lh * (row_bytes - (KS - 1) * PXB);
        u32x2 v[S];
        auto read = [&](uint32_t s) {
            const uint32_t r = 2 * s / KS, c = 2 * s % KS;
            v[s] = *(const u32x2*)((c + 1 < KS || 2 * s + 1 >= taps ? in_row : across) + r * row_bytes + c * PXB);
        };
#pragma unroll
        for (uint32_t s = 0; s < (AHEAD < S ? AHEAD : S); ++s) read(s);
        fence();
#pragma unroll
        for (uint32_t s = 0; s < S; ++s) {
            if (s + AHEAD < S) read(s + AHEAD);
            if (2 * s + 1 >= taps) v[s] = lh ? u32x2{0, 0} : v[s];   // the last tap has no partner (what was read there belongs to another window)
            const u32x4 x = s % 2 == 0 ? u32x4{v[s][0], v[s][1], 0, 0} : u32x4{0, 0, v[s][0], v[s][1]};
            Mma<T>::run(acc, filters[s / 2], x);                     // rows = channels, columns = pixels
            fence();
        }
    } else {
        constexpr uint32_t S = (KS + 1) / 2, STEPS = KS * S;
        u32x4 v[STEPS];
        auto read = [&](uint32_t s) { v[s] = *(const u32x4*)(at + (s / S) * row_bytes + (s % S) * 2 * PXB + lh * PXB); };
#pragma unroll
        for (uint32_t s = 0; s < (AHEAD < STEPS ? AHEAD : STEPS); ++s) read(s);
        fence();
#pragma unroll
        for (uint32_t s = 0; s < STEPS; ++s) {
            if (s + AHEAD < STEPS) read(s + AHEAD);
            if (s % S == S - 1) v[s] = lh ? u32x4{0, 0, 0, 0} : v[s];   // windows are odd: the tap past a kernel row belongs to another window
            Mma<T>::run(acc, filters[s], v[s]);
            fence();
        }
    }
}

// What the parts below share of a tile.
template <typename T> struct FirstTile {
    const uint8_t* frame;
    uint32_t row_bytes, c0, rows;        // of a frame row; the tile's convolution rows are c0 .. c0 + rows - 1
    uint32_t stride, out_w, N, nbase;    // ... of the convolution; the wave's first channel
    uint32_t act;
    const float* bias;                   // the wave's block, in LDS
    T* out;                              // the request's output
};

// bias (added behind the sums, as the staged path does) and activation
template <typename T>
__device__ __forceinline__ void first_activate(f32x4 (&y)[4], const f32x16& acc, const FirstTile<T>& f)
{
    const uint32_t lh = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f32x4 b = *(const f32x4*)(f.bias + 8 * g + 4 * lh);
#pragma unroll
        for (int e = 0; e < 4; ++e) y[g][e] = acc[4 * g + e] + b[e];
    }
    if (f.act == MT_ACT_RELU) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) y[g][e] = max0(y[g][e]);
    } else if (f.act == MT_ACT_GELU) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {                                // four at a time: the registers hold the filters
#pragma unroll
            for (int e = 0; e < 4; ++e) y[g][e] = gelu(y[g][e]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// The tile's pixels in blocks of 32, `du` waves side by side.
template <typename T, uint32_t KS, uint32_t N>
__device__ __forceinline__ void first_rows_out(const FirstTile<T>& f, const u32x4 (&filters)[N], uint32_t u0, uint32_t du, uint32_t through, uint8_t* scratch)
{
    const uint32_t lane = threadIdx.x & 63, li = lane & 31, px = f.rows * f.out_w, nvalid = min((uint32_t)kBrickRows, f.N - min(f.N, f.nbase));
    const float inv = 1.0f / (float)f.out_w;
    for (uint32_t u = u0; u * kBrickRows < px; u += du) {
        const uint32_t p = u * kBrickRows + li, q = p < px ? p : 0;  // empty slots multiply the first pixel; nothing becomes of them
        const uint32_t oh = (uint32_t)(((float)q + 0.5f) * inv), ow = q - __umul24(oh, f.out_w);      // (exact: fewer than 2^20 pixels)
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
        first_window<T, KS>(acc, filters, f.frame + (__umul24(oh, f.stride * f.row_bytes) + __umul24(ow, f.stride * 4 * (uint32_t)sizeof(T))), f.row_bytes);
        f32x4 y[4];
        first_activate<T>(y, acc, f);
        store_unit_nhwc<T>(y, p < px ? f.out + (size_t)(f.c0 * f.out_w + p) * f.N + f.nbase : nullptr, nvalid, through, scratch);
    }
}

// A dword of values as maxima are taken of them.  fp32: one value.  bf16: two, as 16-bit integers of the same order (a negative value's
// magnitude bits inverted; nothing to do behind a ReLU).  NaN counts as -inf: the max-pool passes over NaN, and has -inf where there is nothing else.
typedef short i16x2 __attribute__((ext_vector_type(2)));
template <typename T> struct Ordered;
template <> struct Ordered<float> {
    static constexpr uint32_t kLeast = 0xff800000u;
    static __device__ __forceinline__ uint32_t max(uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b))); }
    static __device__ __forceinline__ uint32_t turn(uint32_t w) { return w; }
};
template <> struct Ordered<__bf16> {
    static constexpr uint32_t kLeast = 0x80008000u;
    static __device__ __forceinline__ uint32_t max(uint32_t a, uint32_t b) { return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, a), __builtin_bit_cast(i16x2, b))); }
    static __device__ __forceinline__ uint32_t turn(uint32_t w) { return w ^ (__builtin_bit_cast(uint32_t, __builtin_bit_cast(i16x2, w) >> (short)15) & 0x7fff7fffu); }      // its own inverse
};
// the value of the next lane (lane 63: any; none of its columns is a window's first)
__device__ __forceinline__ uint32_t next_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, true); }      // wave_shl:1

// Rows pr0 .. pr1 - 1 of the pool's output under 32 columns of the convolution's, from column col on (outside the image: least).
// pk, ps, pp: the pool's window, stride and padding; pw: its output's width.
template <typename T, uint32_t KS, uint32_t N>
__device__ __forceinline__ void first_pool_column(const FirstTile<T>& f, const u32x4 (&filters)[N], uint32_t pr0, uint32_t pr1, int32_t col, uint32_t out_h,
                                                  uint32_t pk, uint32_t ps, uint32_t pp, uint32_t pw)
{
    typedef Ordered<T> O;
    constexpr uint32_t HW = 16 * sizeof(T) / 4;                      // dwords of a lane's 16 values
    const uint32_t lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    const int32_t c = col + (int32_t)li;
    const bool inside = c >= 0 && c < (int32_t)f.out_w;
    const uint8_t* at = f.frame + (uint32_t)min(max(c, 0), (int32_t)f.out_w - 1) * f.stride * 4 * (uint32_t)sizeof(T);
    // the outputs of this wave: lanes 0, ps, 2 ps, ... whose window lies inside its 32 columns
    const uint32_t pc = (uint32_t)(col + (int32_t)pp + (int32_t)li) / ps;
    const bool holds = li % ps == 0 && li + pk <= (uint32_t)kBrickRows && pc < pw;
    uint32_t above[2][HW];                                           // the two rows above: [0] the nearer one; [1]: least where windows have two rows
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h)
#pragma unroll
        for (uint32_t i = 0; i < HW; ++i) above[h][i] = O::kLeast;
    int32_t next = (int32_t)(pr0 * ps) - (int32_t)pp;                // first row of the next output's window
    uint32_t pr = pr0;
    const uint32_t first = (uint32_t)max(next, 0), last = (uint32_t)min((int32_t)((pr1 - 1) * ps + pk) - (int32_t)pp, (int32_t)out_h) - 1;
    const bool turned = f.act != MT_ACT_RELU;
    for (uint32_t r = first; r <= last; ++r) {
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
        first_window<T, KS>(acc, filters, at + (r - f.c0) * f.stride * f.row_bytes, f.row_bytes);
        f32x4 y[4];
        first_activate<T>(y, acc, f);
        if (turned) {
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) y[g][e] = fmaxf(y[g][e], -INFINITY);
        }
        uint32_t now[HW];
#pragma unroll
        for (uint32_t g = 0; g < 4; ++g) {
            if constexpr (sizeof(T) == 2) {                          // rounded as they would have been stored
                typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                typedef float f32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
                for (uint32_t w = 0; w < 2; ++w) now[2 * g + w] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{y[g][2 * w], y[g][2 * w + 1]}, bf16x2));
            } else {
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) now[4 * g + e] = __float_as_uint(y[g][e]);      // (a bit cast of a vector's element reads its first)
            }
        }
        if (turned) {
#pragma unroll
            for (uint32_t i = 0; i < HW; ++i) now[i] = O::turn(now[i]);
        }
#pragma unroll
        for (uint32_t i = 0; i < HW; ++i) now[i] = inside ? now[i] : O::kLeast;
        // a window whose last row this is (or whose rows below lie outside the image); with a padded window at the image's last row, two of them
        while (pr < pr1 && ((int32_t)r == next + (int32_t)pk - 1 || r + 1 == out_h)) {
            // (at the image's last row a window may hold fewer rows than it has: those above it, which no later window needs either, drop out)
            const int32_t n_above = (int32_t)r - next;
            if (n_above + 1 < (int32_t)pk) {
#pragma unroll
                for (uint32_t i = 0; i < HW; ++i) {
                    above[1][i] = O::kLeast;
                    above[0][i] = n_above < 1 ? O::kLeast : above[0][i];
                }
            }
            uint32_t best[HW];
#pragma unroll
            for (uint32_t i = 0; i < HW; ++i) {
                best[i] = O::max(O::max(now[i], above[0][i]), above[1][i]);
                best[i] = O::max(best[i], next_lane(best[i]));
            }
            if (pk == 3) {
#pragma unroll
                for (uint32_t i = 0; i < HW; ++i) best[i] = O::max(best[i], next_lane(best[i]));
            }
            if (turned) {
#pragma unroll
                for (uint32_t i = 0; i < HW; ++i) best[i] = O::turn(best[i]);
            }
            T* out = f.out + ((size_t)pr * pw + pc) * f.N + f.nbase;
            if constexpr (sizeof(T) == 2) {
                // lane (li, lh) holds channels 8g + 4 lh + {0..3}: the halves trade, so that each has 16 bytes of one pixel twice
#pragma unroll
                for (uint32_t g = 0; g < 4; g += 2)
#pragma unroll
                    for (uint32_t w = 0; w < 2; ++w) {
                        auto swapped = __builtin_amdgcn_permlane32_swap(best[2 * g + w], best[2 * g + 2 + w], false, false);
                        best[2 * g + w] = swapped[0]; best[2 * g + 2 + w] = swapped[1];
                    }
                // now best[2g], [2g+1] and [2g+2], [2g+3]: channels 8 (g + lh) + {0..7}
#pragma unroll
                for (uint32_t g = 0; g < 4; g += 2)
                    if (holds && f.nbase + 8 * (g + lh) < f.N)
                        *(u32x4*)(out + 8 * (g + lh)) = u32x4{best[2 * g], best[2 * g + 1], best[2 * g + 2], best[2 * g + 3]};
            } else {
#pragma unroll
                for (uint32_t g = 0; g < 4; ++g)
                    if (holds && f.nbase + 8 * g + 4 * lh < f.N)
                        *(u32x4*)(out + 8 * g + 4 * lh) = u32x4{best[4 * g], best[4 * g + 1], best[4 * g + 2], best[4 * g + 3]};
            }
            ++pr; next += (int32_t)ps;
        }
#pragma unroll
        for (uint32_t i = 0; i < HW; ++i) { above[1][i] = pk == 3 ? above[0][i] : O::kLeast; above[0][i] = now[i]; }
    }
}

// The submitted rows [row0, row0 + n) of the image, into frame rows r0 ...
template <typename T, uint32_t THREADS>
__device__ __forceinline__ void fill_frame(uint8_t* frame, const T* src, uint32_t row0, uint32_t n, uint32_t iw_n, uint32_t cin, uint32_t row_bytes, uint32_t pad)
{
    constexpr uint32_t PXB = 4 * sizeof(T), GP = 24 / (3 * sizeof(T)), NB = 4;      // three-channel images: four (bf16) or two (fp32) pixels are six dwords; groups in flight
    const uint32_t tid = threadIdx.x, npx = n * iw_n;
    const float inv = 1.0f / (float)iw_n;
    auto row_of = [&](uint32_t q) { return (uint32_t)(((float)q + 0.5f) * inv); };        // (exact: fewer than 2^20 pixels)
    if (cin == 3 && npx >= GP) {
        typedef const __attribute__((address_space(1))) typename SubmittedDword<T>::type* dptr_t;
        const T* from = src + (size_t)row0 * iw_n * 3;                              // rows lie one behind the other
        const uint32_t groups = ceil_div(npx, GP);
        for (uint32_t g0 = tid; g0 < groups; g0 += NB * THREADS) {
            uint32_t w[NB][6];
#pragma unroll
            for (uint32_t j = 0; j < NB; ++j) {
                const uint32_t q = min((g0 + j * THREADS) * GP, npx - GP);          // the last group ends at the last pixel
#pragma unroll
                for (uint32_t i = 0; i < 6; ++i) w[j][i] = ((dptr_t)(from + q * 3))[i];
            }
#pragma unroll
            for (uint32_t j = 0; j < NB; ++j) {
                if (g0 + j * THREADS >= groups) break;
                const uint32_t q = min((g0 + j * THREADS) * GP, npx - GP);
                uint32_t r = row_of(q), c = q - r * iw_n;
#pragma unroll
                for (uint32_t e = 0; e < GP; ++e) {
                    uint8_t* dst = frame + r * row_bytes + (pad + c) * PXB;
                    if constexpr (sizeof(T) == 2) {
                        const uint32_t d = 3 * e / 2;
                        *(u32x2*)dst = e % 2 == 0 ? u32x2{w[j][d], w[j][d + 1] & 0xffffu} : u32x2{(w[j][d] >> 16) | (w[j][d + 1] << 16), w[j][d + 1] >> 16};
                    } else {
                        *(u32x4*)dst = u32x4{w[j][3 * e], w[j][3 * e + 1], w[j][3 * e + 2], 0};
                    }
                    if (++c == iw_n) { c = 0; ++r; }
                }
            }
        }
    } else {
        const T* from = src + (size_t)row0 * iw_n * cin;
        for (uint32_t q = tid; q < npx; q += THREADS) {
            const uint32_t r = row_of(q), c = q - r * iw_n;
            T* dst = (T*)(frame + r * row_bytes + (pad + c) * PXB);
            for (uint32_t e = 0; e < cin; ++e) dst[e] = from[(size_t)q * cin + e];
        }
    }
}

template <typename T, uint32_t KSMAX, bool POOL>
__global__ __launch_bounds__(POOL ? 512 : 256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && KSMAX == 7 ? 2 : 4)))
void conv_first_kernel(GemmArgs a)
{
    constexpr uint32_t THREADS = POOL ? 512 : 256, WAVES = THREADS / 64, PXB = 4 * sizeof(T);
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    __shared__ uint32_t owner_part[WAVES];
    __shared__ __attribute__((aligned(16))) float bias[kFirstBlocks * kBrickRows];
    const uint32_t tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    TileOwner<THREADS> lookup;
    lookup.fetch(a.tile_base, a.T);
    const uint32_t n_tiles = a.tile_base[a.T];
    // the frame starts as zeros; written while the tile list is on its way, published by the barrier of the lookup
    for (uint32_t q = tid * 16; q < a.img_lds; q += THREADS * 16) *(u32x4*)(lds + q) = u32x4{0, 0, 0, 0};
    uint32_t idx;
    if (!logical_tile(n_tiles, &idx)) return;
    const uint32_t t = lookup.owner(a.T, idx, owner_part);           // uniform: the tenant's facts come through scalar loads
    const LayerDev L = a.layers[t * MT_MAX_LAYERS];
    const uint32_t seg0 = a.off[t], Mt = a.M[t];
    const bool pooled = POOL && L.first_pool;
    const LayerDev& G = a.layers[t * MT_MAX_LAYERS + (POOL ? 1 : 0)];   // the max-pool, if it is done here
    const uint32_t pk = pooled ? G.ksize : 1, ps = pooled ? G.stride : 1, pp = pooled ? G.pad : 0, pw = pooled ? G.out_w : 1;
    const uint32_t out_w = L.out_w, out_h = L.rows_per_req / out_w, end_rows = pooled ? G.rows_per_req / pw : out_h;
    const uint32_t strips = first_strips(end_rows, L.first_rows, a.first_cap), step = ceil_div(end_rows, strips);
    uint32_t local = idx - a.tile_base[t];
    const uint32_t strip = local % strips;
    local /= strips;
    const uint32_t pass = local / Mt, req = local - pass * Mt;
    const T* const src = (const T*)a.row_src[a.perm[seg0 + req]];
    const uint32_t nb0 = pass * kFirstBlocks, ncb = min(kFirstBlocks, L.N_pad / kBrickRows - nb0);

    // ---- this wave's filters, the workgroup's bias
    const uint32_t ks = L.ksize, cb = wave % ncb, u0 = wave / ncb, du = WAVES / ncb;      // waves take the channel blocks in turn (one or two)
    u32x4 filters[first_quads<T, KSMAX>()];
    {
        const uint8_t* wp = a.arena + L.w_off + (size_t)(nb0 + cb) * L.K * kBrickRows * sizeof(T);
        if (KSMAX == 7 && ks == 7) load_filters<T, KSMAX>(filters, wp);
        else if (ks == 3) load_filters<T, 3>(filters, wp);
        else load_filters<T, 1>(filters, wp);
    }
    if (tid < ncb * kBrickRows) bias[tid] = ((const float*)(a.arena + L.b_off))[nb0 * kBrickRows + tid];      // padded to N_pad

    // ---- frame
    const uint32_t p0 = strip * step, p1 = min(p0 + step, end_rows);    // rows of the pool's output, or the convolution's
    FirstTile<T> f;
    f.row_bytes = first_frame_cols(L) * PXB;
    f.c0 = (uint32_t)max((int32_t)(p0 * ps) - (int32_t)pp, 0);
    f.rows = (uint32_t)min((int32_t)((p1 - 1) * ps + pk) - (int32_t)pp, (int32_t)out_h) - f.c0;
    f.frame = lds; f.stride = L.stride; f.out_w = out_w; f.N = L.N; f.nbase = (nb0 + cb) * kBrickRows; f.act = L.act;
    f.bias = bias + cb * kBrickRows;
    f.out = (T*)act_of(a.act, pooled ? G.out_buf : L.out_buf) + (size_t)(seg0 + req) * a.S;
    {
        const int32_t ih0 = (int32_t)(f.c0 * L.stride) - (int32_t)L.pad, n_ih = (int32_t)((f.rows - 1) * L.stride + ks);
        const int32_t lo = max(ih0, 0), hi = min(ih0 + n_ih, (int32_t)L.in_h);
        fill_frame<T, THREADS>(lds + (uint32_t)(lo - ih0) * f.row_bytes, src, (uint32_t)lo, (uint32_t)max(hi - lo, 0), L.in_w, L.first_cin, f.row_bytes, L.pad);
    }
    lds_barrier();

    auto compute = [&](auto KS_) {
        constexpr uint32_t KS = decltype(KS_)::value;
        if constexpr (POOL) {
            if (pooled) {
                // columns of 32 of the convolution, each the windows of `wide` outputs; where those are few, waves share the rows of a tile
                const uint32_t wide = ((uint32_t)kBrickRows - pk) / ps + 1, columns = ceil_div(pw, wide), parts = max(du / columns, 1u);
                const uint32_t per = ceil_div(p1 - p0, parts);
                for (uint32_t u = u0; u < columns * parts; u += du) {
                    const uint32_t part = u / columns, x = u - part * columns, a0 = p0 + part * per, a1 = min(a0 + per, p1);
                    if (a0 < a1) first_pool_column<T, KS>(f, filters, a0, a1, (int32_t)(x * wide * ps) - (int32_t)pp, out_h, pk, ps, pp, pw);
                }
                return;
            }
        }
        first_rows_out<T, KS>(f, filters, u0, du, a.store_through, lds + a.img_lds + wave * unit_scratch_bytes<T>());
    };
    if (KSMAX == 7 && ks == 7) compute(std::integral_constant<uint32_t, KSMAX>{});
    else if (ks == 3) compute(std::integral_constant<uint32_t, 3>{});
    else compute(std::integral_constant<uint32_t, 1>{});
}

// ---- a first convolution and the 3x3 convolution behind it ----------------------------------------
// Where that convolution is the first one's only reader, in every model that starts with one (LayerDev::pair_rows): a workgroup computes the rows of the first layer that a
// tile of whole rows of the second one needs into a frame in LDS, rounded as they would have been stored and with a zero border, and
// the second layer from there as conv_img_kernel does: four waves side by side over NCB blocks of channels and the pixel blocks,
// filters through a register ring.  The first layer's output is never written; its rows on a tile's edge are computed twice.  Sums in the
// order of the other kernels: the same bits.
// 2048 images of 32x32x3 through 3x3x32 and 3x3x64 at stride 2: 33 + 55 -> 65 us, and 134 MB neither written nor read (the pass 162 -> 115); 150 fp32 images of
// 29x35x3 through 3x3x24 and 3x3x40 14.5 + 54 -> 64.5.  Of the 11 us of a tile (three to a compute unit) 4 pass before the first MFMA, 3 are the first
// layer, 2.3 the second, 1.4 its stores.  Tiles in 26 / 32 / 40 / 52 KiB of LDS: 103 / 78 / 70 / 65.5 us.  Beside models that cannot take
// it (a launch of theirs besides) it gains nothing: MLPs, CNNs and residual nets by turns, 600 requests 12.6 + 12.7 against 12.7 + 13.8, 6000 requests 78 + 36 against 98 + 70.
template <typename T, uint32_t NCB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void conv_pair_kernel(GemmArgs a)
{
    constexpr uint32_t THREADS = 256, WAVES = 4, EPC = 16 / sizeof(T), KB = 2 * EPC, P = 8, WR = WAVES / NCB, RBW = kConvTileRows / kBrickRows / WR;
    typedef const __attribute__((address_space(1))) u32x4* gptr_t;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    __shared__ uint32_t owner_part[WAVES];
    __shared__ __attribute__((aligned(16))) float bias[kFirstBlocks * kBrickRows];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 31, lh = lane >> 5;
    TileOwner<THREADS> lookup;
    lookup.fetch(a.tile_base, a.T);
    const uint32_t n_tiles = a.tile_base[a.T];
    uint8_t* const mid = lds + a.img_lds;                            // the first layer's rows
    for (uint32_t q = tid * 16; q < a.img_lds + a.mid_lds; q += THREADS * 16) *(u32x4*)(lds + q) = u32x4{0, 0, 0, 0};
    uint32_t idx;
    if (!logical_tile(n_tiles, &idx)) return;
    const uint32_t t = lookup.owner(a.T, idx, owner_part);           // uniform: the tenant's facts come through scalar loads
    const LayerDev L = a.layers[t * MT_MAX_LAYERS], M = a.layers[t * MT_MAX_LAYERS + 1];
    const uint32_t seg0 = a.off[t], h1 = M.rows_per_req / M.out_w, strips = first_strips(h1, M.pair_rows, a.first_cap), step = ceil_div(h1, strips);
    const uint32_t local = idx - a.tile_base[t], req = local / strips, strip = local - req * strips;
    const T* const src = (const T*)a.row_src[a.perm[seg0 + req]];
    const uint32_t p0 = strip * step, p1 = min(p0 + step, h1);
    const uint32_t w0 = L.out_w, h0 = L.rows_per_req / w0, ncb0 = L.N_pad / kBrickRows, cb0 = wave % ncb0;

    // ---- the first layer's rows under rows p0 .. p1 - 1 of the second one's
    const uint32_t st = M.stride, cin = M.cin, PB = cin * (uint32_t)sizeof(T) + 16, RSB = (w0 + 2) * PB;     // bytes per pixel and row of `mid`
    const int32_t m0 = (int32_t)(p0 * st) - 1;                       // the first layer's row in row 0 of `mid`
    FirstTile<T> f;
    f.row_bytes = first_frame_cols(L) * 4 * (uint32_t)sizeof(T);
    f.c0 = (uint32_t)max(m0, 0);
    f.rows = (uint32_t)min((int32_t)((p1 - 1) * st) + 2, (int32_t)h0) - f.c0;
    f.frame = lds; f.stride = L.stride; f.out_w = w0; f.N = L.N; f.nbase = cb0 * kBrickRows; f.act = L.act;
    f.bias = bias + cb0 * kBrickRows; f.out = nullptr;
    constexpr uint32_t KSMAX = 3;
    u32x4 filters[first_quads<T, KSMAX>()];
    {
        const uint8_t* wp = a.arena + L.w_off + (size_t)cb0 * L.K * kBrickRows * sizeof(T);
        if (L.ksize == 3) load_filters<T, 3>(filters, wp); else load_filters<T, 1>(filters, wp);
    }
    if (tid < ncb0 * kBrickRows) bias[tid] = ((const float*)(a.arena + L.b_off))[tid];      // padded to N_pad
    {
        const int32_t ih0 = (int32_t)(f.c0 * L.stride) - (int32_t)L.pad, n_ih = (int32_t)((f.rows - 1) * L.stride + L.ksize);
        const int32_t lo = max(ih0, 0), hi = min(ih0 + n_ih, (int32_t)L.in_h);
        fill_frame<T, THREADS>(lds + (uint32_t)(lo - ih0) * f.row_bytes, src, (uint32_t)lo, (uint32_t)max(hi - lo, 0), L.in_w, L.first_cin, f.row_bytes, L.pad);
    }
    lds_barrier();
    {
        const uint32_t px = f.rows * w0, du = WAVES / ncb0, top = (uint32_t)((int32_t)f.c0 - m0);
        const float inv = 1.0f / (float)w0;
        for (uint32_t u = wave / ncb0; u * kBrickRows < px; u += du) {
            const uint32_t p = u * kBrickRows + li, q = p < px ? p : 0;
            const uint32_t oh = (uint32_t)(((float)q + 0.5f) * inv), ow = q - __umul24(oh, w0);      // (exact: fewer than 2^20 pixels)
            const uint8_t* at = lds + (__umul24(oh, f.stride * f.row_bytes) + __umul24(ow, f.stride * 4 * (uint32_t)sizeof(T)));
            f32x16 acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
            if (L.ksize == 3) first_window<T, 3>(acc, filters, at, f.row_bytes); else first_window<T, 1>(acc, filters, at, f.row_bytes);
            f32x4 y[4];
            first_activate<T>(y, acc, f);
            uint8_t* dst = mid + __umul24(oh + top, RSB) + __umul24(ow + 1, PB) + (f.nbase + 4 * lh) * (uint32_t)sizeof(T);
#pragma unroll
            for (uint32_t g = 0; g < 4; ++g) {
                if (p < px && f.nbase + 8 * g + 4 * lh < L.N) put4<T>(dst + 8 * g * (uint32_t)sizeof(T), y[g]);      // channels are a multiple of 8: a run of four exists whole or not at all
            }
        }
    }

    // ---- the second layer; its first filters are asked for in front of the barrier
    const uint32_t nKB = M.K / KB, nKBv = M.k_valid / KB;            // cin is whole k steps
    const uint32_t wc = wave % NCB, wr = wave / NCB, out_w = M.out_w, px = (p1 - p0) * out_w;
    const bool active = wc < M.N_pad / kBrickRows && wr * RBW * kBrickRows < px;
    gptr_t wp = (gptr_t)((const u32x4*)(a.arena + M.w_off) + (size_t)(active ? wc : 0) * nKB * 64 + lane);
    u32x4 wq[P];
#pragma unroll
    for (uint32_t j = 0; j < P; ++j) wq[j] = wp[(size_t)min(j, nKBv - 1) * 64];
    lds_barrier();
    f32x16 acc[RBW];
#pragma unroll
    for (uint32_t r = 0; r < RBW; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] = 0.0f;
    if (active) {
        const uint8_t* base[RBW];
        const float inv = 1.0f / (float)out_w;
#pragma unroll
        for (uint32_t r = 0; r < RBW; ++r) {
            const uint32_t p = (wr * RBW + r) * kBrickRows + li, q = p < px ? p : 0;         // an empty slot multiplies the first pixel; nothing is stored for it
            const uint32_t oh = (uint32_t)(((float)q + 0.5f) * inv), ow = q - __umul24(oh, out_w);
            base[r] = mid + (__umul24(oh, st * RSB) + __umul24(ow, st * PB) + lh * 16);
        }
        const uint32_t last = 2 * RSB + 2 * PB + (cin - KB) * (uint32_t)sizeof(T);
        auto k_loop = [&](auto NR_) {
            constexpr uint32_t NR = decltype(NR_)::value;
            uint32_t ch = 0, kw = 0, row_off = 0, off = 0;           // scalar: channel inside the tap, kernel column, byte offset of the tap's row, of the k step
            auto advance = [&] {
                ch += KB; off += KB * (uint32_t)sizeof(T);
                if (ch == cin) {
                    ch = 0; ++kw;
                    if (kw == 3) { kw = 0; row_off += RSB; }
                    off = row_off + kw * PB;
                }
            };
            u32x4 av[NR];
#pragma unroll
            for (uint32_t r = 0; r < NR; ++r) av[r] = *(const u32x4*)(base[r]);
            auto one = [&](const u32x4& wv) {                        // operands a step ahead (past the last one: the frame's last, unused)
                advance();
                const uint32_t next = min(off, last);
                u32x4 an[NR];
#pragma unroll
                for (uint32_t r = 0; r < NR; ++r) an[r] = *(const u32x4*)(base[r] + next);
#pragma unroll
                for (uint32_t r = 0; r < NR; ++r) Mma<T>::run(acc[r], wv, av[r]);           // rows = channels, columns = pixels
#pragma unroll
                for (uint32_t r = 0; r < NR; ++r) av[r] = an[r];
            };
            const uint32_t full = nKBv / P;
            for (uint32_t g = 0; g < full; ++g) {
#pragma unroll
                for (uint32_t j = 0; j < P; ++j) {
                    one(wq[j]);
                    wq[j] = wp[(size_t)min(g * P + j + P, nKBv - 1) * 64];
                }
            }
#pragma unroll
            for (uint32_t j = 0; j < P; ++j)
                if (full * P + j < nKBv) one(wq[j]);
        };
        if (RBW > 1 && px <= (wr * RBW + RBW / 2) * kBrickRows) k_loop(std::integral_constant<uint32_t, (RBW > 1 ? RBW / 2 : 1)>{});
        else k_loop(std::integral_constant<uint32_t, RBW>{});
    }
    const uint32_t nbase = (active ? wc : 0) * kBrickRows;
    const float* bias2 = (const float*)(a.arena + M.b_off);
    f32x4 bias_q[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) bias_q[g] = *(const f32x4*)(bias2 + nbase + 8 * g + 4 * lh);
    lds_barrier();                                                   // every wave is done with the rows: they now serve as store scratch
    if (!active) return;
    uint8_t* scratch = lds + wave * unit_scratch_bytes<T>();
    T* const out = (T*)act_of(a.act, M.out_buf) + (size_t)(seg0 + req) * a.S + (size_t)p0 * out_w * M.N + nbase;
#pragma unroll
    for (uint32_t r = 0; r < RBW; ++r) {
        const uint32_t p = (wr * RBW + r) * kBrickRows + li;
        f32x4 y[4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) y[g][e] = acc[r][4 * g + e] + bias_q[g][e];
        __builtin_amdgcn_sched_barrier(0);
        activate_block<4>(y, M.act);
        store_unit_nhwc<T>(y, p < px ? out + (size_t)p * M.N : nullptr, min((uint32_t)kBrickRows, M.N - nbase), a.store_through, scratch);
    }
}

// ---- launcher ------------------------------------------------------------
// scratch: some model's rows leave through the waves' store scratch (none does where every model's max-pool is done here)
template <typename T, uint32_t KSMAX, bool POOL>
static hipError_t launch_first_t(const GemmArgs& a, bool scratch, uint32_t frame_bytes, uint32_t grid, hipStream_t s)
{
    constexpr uint32_t threads = POOL ? 512 : 256;
    static_assert(8 * unit_scratch_bytes<T>() == first_scratch_bytes(sizeof(T)), "what the layers' limits were checked with");
    GemmArgs b = a;
    b.img_lds = (frame_bytes + 15) / 16 * 16;
    hipLaunchKernelGGL((conv_first_kernel<T, KSMAX, POOL>), dim3(grid), dim3(threads), b.img_lds + (scratch ? threads / 64 * unit_scratch_bytes<T>() : 0), s, b);
    return hipGetLastError();
}

template <typename T>
static hipError_t prepare_first_t()
{
    hipError_t e = hipSuccess;
    auto allow = [&](auto kernel) {
        const hipError_t x = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFirstMaxBytes);
        if (e == hipSuccess) e = x;
    };
    allow(conv_first_kernel<T, 3, false>); allow(conv_first_kernel<T, 3, true>); allow(conv_first_kernel<T, 7, false>); allow(conv_first_kernel<T, 7, true>);
    allow(conv_pair_kernel<T, 2>); allow(conv_pair_kernel<T, 4>);
    return e;
}
template <typename T>
static hipError_t launch_pair_t(const GemmArgs& a, uint32_t blocks, uint32_t frame_bytes, uint32_t mid_bytes, uint32_t grid, hipStream_t s)
{
    GemmArgs b = a;
    b.img_lds = (frame_bytes + 15) / 16 * 16;
    b.mid_lds = mid_bytes;                                           // (pixels are multiples of 16 bytes)
    const uint32_t lds = std::max<uint32_t>(b.img_lds + b.mid_lds, 4 * unit_scratch_bytes<T>());
    if (blocks <= 2) hipLaunchKernelGGL((conv_pair_kernel<T, 2>), dim3(grid), dim3(256), lds, s, b);
    else hipLaunchKernelGGL((conv_pair_kernel<T, 4>), dim3(grid), dim3(256), lds, s, b);
    return hipGetLastError();
}
// blocks: the widest second layer in blocks of 32 channels
hipError_t launch_conv_pair(const GemmArgs& a, uint32_t dtype, uint32_t blocks, uint32_t frame_bytes, uint32_t mid_bytes, uint32_t grid, hipStream_t s)
{
    if (grid == 0) return hipSuccess;
    grid = (grid + 7) / 8 * 8;
    return dtype == MT_BF16 ? launch_pair_t<__bf16>(a, blocks, frame_bytes, mid_bytes, grid, s) : launch_pair_t<float>(a, blocks, frame_bytes, mid_bytes, grid, s);
}

hipError_t prepare_conv_first(uint32_t dtype) { return dtype == MT_BF16 ? prepare_first_t<__bf16>() : prepare_first_t<float>(); }

template <typename T>
static hipError_t launch_conv_first_t(const GemmArgs& a, uint32_t max_ks, bool pool, bool scratch, uint32_t frame_bytes, uint32_t grid, hipStream_t s)
{
    if (max_ks <= 3) return pool ? launch_first_t<T, 3, true>(a, scratch, frame_bytes, grid, s) : launch_first_t<T, 3, false>(a, scratch, frame_bytes, grid, s);
    return pool ? launch_first_t<T, 7, true>(a, scratch, frame_bytes, grid, s) : launch_first_t<T, 7, false>(a, scratch, frame_bytes, grid, s);
}
hipError_t launch_conv_first(const GemmArgs& a, uint32_t dtype, uint32_t max_ks, bool pool, bool scratch, uint32_t frame_bytes, uint32_t grid, hipStream_t s)
{
    if (grid == 0) return hipSuccess;
    grid = (grid + 7) / 8 * 8;
    return dtype == MT_BF16 ? launch_conv_first_t<__bf16>(a, max_ks, pool, scratch, frame_bytes, grid, s)
                            : launch_conv_first_t<float>(a, max_ks, pool, scratch, frame_bytes, grid, s);
}

}  // namespace mt

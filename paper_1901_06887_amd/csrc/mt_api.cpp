// Host side of the multi-tenant worker runtime: the C ABI of include/mt.h, the tenant
// registry (closed layer set, paper section 3.1), the packed weight arena in device memory
// (models stay resident on the accelerator, section 3.3) and the fixed launch sequence of
// mt_run (segmentation, gather, one grouped launch per layer index, head).
#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "mt_internal.h"
#include "../../include/mt_debug.h"

using namespace mt;

// Scratch of mt_run_static: batch descriptors, both activation buffers and logits of one run.  The
// array lives in device memory of every GPU the library runs on until the process ends.  On the
// host its name is only a handle: the device address is looked up once per context
// (hipGetSymbolAddress in mt_create, with the context's device current) and kept in the context.
static __device__ __align__(256) unsigned char scratch[MT_STATIC_SCRATCH_BYTES];


namespace {

constexpr uint32_t kMaxTenants = 2048;
constexpr uint32_t kSegSlots = MT_SEG_SLOTS;   // pinned segment tables: runs of several submissions in flight at once
constexpr uint32_t kMaxRunSlots = 4;      // runs in flight at once (each with its own device scratch); <= kSegSlots
constexpr uint64_t kArenaAlign = 256;
constexpr uint64_t kMaxLaunchItems = 0xffff0000u;   // work items of one launch (the grid is rounded up to a multiple of 8 or 512 workgroups)
// profiling slots: batcher, gather, head, then gemm and gap of every layer index
constexpr uint32_t kProfBatcher = 0, kProfGather = 1, kProfHead = 2, kProfFc = 3, kProfConv = 3 + MT_MAX_LAYERS,
                   kProfGap = 3 + 2 * MT_MAX_LAYERS, kProfBig = 3 + 3 * MT_MAX_LAYERS, kProfGatherImg = 3 + 4 * MT_MAX_LAYERS,
                   kProfImageOps = 4 + 4 * MT_MAX_LAYERS;
constexpr uint32_t kProfSlots = 4 + 5 * MT_MAX_LAYERS;

inline uint32_t round_up(uint32_t v, uint32_t a) { return (v + a - 1) / a * a; }
inline uint64_t round_up64(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

struct HostLayer {
    mt_layer_spec spec;
    LayerDev dev;               // w_off / b_off: absolute arena offsets while the model is resident
    uint64_t w_bytes, b_bytes;
    uint64_t w_rel, b_rel;      // the same offsets relative to the model's arena block
};

struct HostTenant {
    bool registered = false;
    uint32_t n_layers = 0;
    HostLayer layers[MT_MAX_LAYERS];
    TenantDev dev{};
    uint64_t arena_off = 0, arena_len = 0;
    uint32_t act_buffers = 2;   // activation buffers a run needs for this model (two for a chain)
    // Model cache (cfg.cache): the packed weights stay in pinned host memory (`stage`: the arena
    // image followed by the device table rows of this tenant) and the arena holds the models used
    // most recently.  Outside cache mode every registered model is resident and stage is null.
    bool resident = false;
    uint64_t last_use = 0;
    uint8_t* stage = nullptr;
};

struct FreeBlock { uint64_t off, len; };

// What the tiles of a first convolution on the submitted images take: LDS for the images' rows and for the first layer's (with the second layer), and
// tiles of a request.
struct FirstNeed {
    uint64_t frame, mid, tiles;
    bool operator==(const FirstNeed& o) const { return frame == o.frame && mid == o.mid && tiles == o.tiles; }
};

// The first two layers of models that start with a convolution which can read the submitted images (without arena offsets), and how many have them.
struct FirstShape { LayerDev conv, next; uint32_t models; };

// What the launches of the runs captured between two registrations assume of every model they serve.  Replayed after a later registration,
// such a run serves that model only if this holds for it too.
struct PlanUse {
    uint32_t plan = 0;
    bool any = false;                 // there was one
    uint32_t act_buffers = 0, layer_slots = 0;      // activation buffers and layer indices that it has
    bool first = false;               // first convolutions read the submitted images: ...
    bool pair = false, pool = false, plain = false, ops1 = false;      // with the convolutions behind them; some max-pool done with them; some rows stored themselves; max-pools or additions at layer index 1 have a launch
    uint32_t max_ks = 0, pair_blocks = 0;
    uint64_t chunk_layers = 0;        // layer indices whose split convolutions loaded whole chunks
    std::vector<FirstNeed> most;      // the most that the models then registered take, by the rows of a tile less one ...
    uint32_t cap = 0;                 // ... or of tiles of so many rows
    bool same_as(const PlanUse& o) const
    {
        return act_buffers == o.act_buffers && layer_slots == o.layer_slots && first == o.first && pair == o.pair && pool == o.pool && plain == o.plain && ops1 == o.ops1 && max_ks == o.max_ks &&
               pair_blocks == o.pair_blocks && chunk_layers == o.chunk_layers && most == o.most && cap == o.cap;
    }
};
constexpr size_t kPlansKept = 64;

struct NamedRows { uint32_t tenant, rows; };   // requests of a tenant in the submissions that named it

// The event behind every run orders runs of other streams of the same device behind it, on the device; nothing on the host or another device looks at it.  So it needs no
// fence of the whole system, which wrote back the L2s at the end of every run: 64 fp32 requests to MLPs 23.0 -> 21.3 us a pass, and where the labels are copied out
// behind every pass 43.7 -> 42.7, one bf16 request 39.8 -> 38.5, 150 fp32 images to CNNs 151.4 -> 149.5.  (Whoever waits for the stream, or copies from it, has a fence of their own.)
constexpr unsigned kSlotEvent = hipEventDisableTiming | hipEventDisableSystemFence;

// Device scratch of one run in flight: batch descriptors, activation buffers, logits.  A run owns
// one slot from its batcher to its last kernel; the weights and model tables are shared.
struct RunSlot {
    int32_t* d_row_tenant = nullptr; uint32_t* d_row_rank = nullptr; uint32_t* d_hist_g = nullptr;
    const void** d_row_src = nullptr; int32_t* d_pos_of = nullptr; int32_t* d_perm = nullptr;
    uint32_t* d_M = nullptr; uint32_t* d_off = nullptr; uint32_t* d_tile_base = nullptr;
    void* d_act[kActBuffers] = {}; float* d_logits = nullptr;   // (only as many activation buffers as the registered models need)
    hipEvent_t done = nullptr;      // recorded behind the slot's last run
    hipStream_t stream = nullptr;   // ... which was enqueued here
    uint64_t last_run = 0;          // ... and was the context's run number this
    bool used = false;
};

}  // namespace

struct mt_ctx {
    mt_config cfg{};
    bool host_only = false;
    uint32_t elem_size = 2;
    uint32_t S = 0;        // elements between consecutive requests in an activation buffer
    uint32_t C_pad = 0;    // floats between consecutive rows of the internal logits buffer
    std::vector<HostTenant> tenants;
    std::vector<FreeBlock> free_list;
    uint64_t arena_used = 0;
    uint32_t n_registered = 0;

    // per layer index, over registered tenants: bounds that size the grouped launches
    uint32_t n_layer_slots = 0;
    uint32_t max_in_len = 0, max_fc_in_len = 0;      // longest input; ... of a model that starts with an FC layer
    // [kind][layer]: kind 0 = FC tiles, 1 = conv tiles, 2 = big FC tiles
    uint32_t max_nt[kListKinds][MT_MAX_LAYERS]{}, has_gap[MT_MAX_LAYERS]{};
    uint64_t gap_chunks[MT_MAX_LAYERS]{};            // most 16-byte pieces that a workgroup of a pooling layer of the index can have in flight (launch_gap)
    // pool_fused[l]: layer index l + 1 is a global average pool for every registered model that is that deep, and
    // each of their convolutions at l can pool by itself: the convolution launch writes the pooled activation
    // and nothing runs at index l + 1 (all or nothing: the activation buffers alternate per layer index)
    bool pool_fused[MT_MAX_LAYERS]{};
    double sum_macs = 0.0;                           // multiply-accumulates of one request, summed over the registered tenants
    uint32_t max_conv_cb[MT_MAX_LAYERS]{};
    // Every registered model that starts with a convolution has one that can read the submitted images (LayerDev::first_rows): layer
    // index 0 is launched that way and nothing stages images.  Over those models: whether some max-pool is done with them, some
    // layer's rows are stored themselves; largest window; most rows of a tile, and tiles of one row of an image.
    bool first_on = false, first_pool = false, first_plain = false;
    uint32_t first_max_ks = 0, first_max_rows = 0;
    uint64_t first_max_tiles = 0;
    std::vector<FirstShape> first_shapes;
    uint32_t n_conv_first = 0;                       // registered models that start with a convolution
    // In every one of those models the second layer is a 3x3 convolution that can be done with the first (LayerDev::pair_rows); the widest in
    // blocks; no other model has a convolution at layer index 1 then.
    bool pair_on = false;
    uint32_t pair_blocks = 0;
    uint32_t no_conv_pair = 0;                       // tuning/testing: every convolution has a launch
    uint32_t no_conv_first = 0;                      // tuning/testing: images are always staged
    uint32_t first_cap = 0;                          // testing: MT_FIRST_ROWS in place of first_tile_rows()'s choice, and whatever fits takes those tiles
    uint32_t conv_img_lds[MT_MAX_LAYERS]{};          // every conv of a layer index can keep its tiles' input in LDS: the largest frame in bytes, else 0
    double conv_frame_share[MT_MAX_LAYERS]{};        // largest share of a row-tiled layer's MFMAs that is neither empty pixel slots nor missing channel blocks
    int conv_img_two[MT_MAX_LAYERS]{};               // ... and their pixels are one 16-byte chunk: 1, none is: 0 (-1: no convolution seen yet)
    uint32_t no_conv_img = 0;                        // tuning: never use that kernel
    bool conv_uniform[MT_MAX_LAYERS]{};              // every conv of a layer index has input channels in multiples of a k step, and a window of at most 64 taps
    bool conv_quad[MT_MAX_LAYERS]{};                 // every conv of a layer index has input channels in multiples of four 16-byte chunks           // widest conv tile (32-channel blocks, at most 4) of a layer index
    uint64_t sum_nt[kListKinds][MT_MAX_LAYERS]{};
    uint32_t max_fc_per64[MT_MAX_LAYERS]{};   // streaming FC tiles per 64 rows of one tenant, maximum over the registered models
    uint64_t sum_nt_sk[MT_MAX_LAYERS]{};      // the same two figures for the K-split tile shape
    uint32_t max_fc_per64_sk[MT_MAX_LAYERS]{};
    uint32_t max_big_blocks[MT_MAX_LAYERS]{};  // most column blocks of a registered FC layer whose rows past the big tiles take K-split tiles
    uint32_t fc_split_k = 0;   // tuning: every run uses FC tiles of one column block with K split four ways
    uint32_t no_auto_split_k = 0;   // tuning: small runs keep the ordinary tile shape
    uint32_t no_fused_gather = 0;  // tuning/testing: always stage FC inputs with the gather kernel
    bool fc_first_chunked = true;  // every registered FC-first model's input is a whole number of 16-byte chunks
    bool any_conv_first = false, any_fc_first = false;
    uint32_t list_mask[MT_MAX_LAYERS / kLayerGroup] = {};   // per group of layer indices, bit kind*kLayerGroup + l%kLayerGroup: some registered model has that kind at layer l
    uint32_t has_image_ops[MT_MAX_LAYERS]{};   // some registered model has a max-pool or an addition at this layer index
    uint32_t image_op_fill[MT_MAX_LAYERS]{};   // ... and the longest output row (elements) among them
    uint32_t min_layers = 0;                   // layers of the registered model with the fewest
    uint32_t no_entry = 0;                     // tuning/testing: the batcher always has a launch
    uint32_t max_image_pixels = 0;             // most pixels in a submitted image (models whose first layer is a convolution)
    uint32_t act_buffers = 2;      // activation buffers every run slot holds (grows when a model with skip connections needs more)
    uint32_t max_reg_classes = 0, min_reg_classes = 0;
    bool wide_last_unfit = false;              // some registered model ends with a layer of 33 to 128 classes that tiles of all its blocks do not pay for (whole_pays)
    bool wide_last[MT_MAX_LAYERS]{};           // some registered model ends with such a layer at the index
    uint32_t no_fused_head = 0;    // tuning/testing: always run the separate head kernel
    uint32_t no_fused_pool = 0;    // tuning/testing: always run the separate pooling kernel
    uint32_t no_fused_add = 0;     // tuning/testing: residual additions always run as launches of their own
    uint32_t big_walk = 1;         // big FC tiles: one workgroup per CU walks several tiles (tuning/testing: MT_BIG_WALK=0 gives every tile a workgroup of its own)
    uint32_t n_cus = 256;          // compute units of the device, rounded down to a multiple of 8
    uint32_t max_fc_cols[MT_MAX_LAYERS]{};     // widest (padded) FC layer of a layer index: up to 64 outputs split K in every run
    uint32_t min_fc_k[MT_MAX_LAYERS]{};        // shortest padded fan-in among the registered FC layers of a layer index
    uint32_t no_conv_uniform = 0;  // tuning/testing: convolution gathers always walk the window lane by lane
    uint32_t no_conv_loaders = 0;  // tuning/testing: convolution tiles never get waves of their own for the loads
    uint32_t max_conv_blocks[MT_MAX_LAYERS]{};  // widest convolution of a layer index over the registered models, in blocks of 32 channels
    uint64_t max_conv_work[MT_MAX_LAYERS]{};    // most output pixels x channel blocks of one convolution of the layer index
    uint64_t max_conv_tile_rows[MT_MAX_LAYERS]{};  // ... rows by which its ordinary tiles are counted x tiles side by side
    uint64_t sum_conv_work[MT_MAX_LAYERS]{};    // sum over the registered models of output pixels x channel blocks
    uint64_t sum_conv_blocks[MT_MAX_LAYERS]{};  // ... and their sum
    uint32_t max_conv_k[MT_MAX_LAYERS]{};      // longest reduction among the registered convolutions of a layer index
    int64_t conv_split_tiles = -1;              // testing: MT_CONV_SPLIT_TILES in place of conv_split_line (0: no convolution launch splits K)
    uint32_t min_conv_k[MT_MAX_LAYERS]{};      // shortest reduction among the registered convolutions of a layer index
    uint32_t big_min_tiles = kBigMinTiles;   // testing: MT_BIG_MIN_TILES=1 sends every qualifying tenant-layer to big tiles
    uint32_t P_cap = 0;        // packed rows incl. per-tenant padding to 32

    // device state.  The per-run pointers below (d_row_tenant .. d_logits) are those of the run
    // slot bound last (bind_slot): the slot of the run being enqueued, then of the last run.
    std::vector<RunSlot> slots;
    RunSlot static_slot;               // the slot of mt_run_static: its buffers are carved out of static_scratch per run
    uint8_t* static_scratch = nullptr; // device address of `scratch` on this context's GPU
    uint8_t* d_arena = nullptr;
    TenantDev* d_tenants = nullptr;
    LayerDev* d_layers = nullptr;
    uint64_t* d_served = nullptr;      // [max_tenants][2]: requests served, runs with at least one request (accounting)
    uint32_t* d_facts = nullptr;       // [MT_MAX_LAYERS][max_tenants][kFactWords]: the batcher's view of the layers (BatchArgs::facts)
    int32_t* d_row_tenant = nullptr;
    uint32_t* d_row_rank = nullptr;
    uint32_t* d_hist_g = nullptr;      // [kHistEntries] per-workgroup tenant histograms of the ranking kernel
    const void** d_row_src = nullptr;
    int32_t* d_pos_of = nullptr;
    int32_t* d_perm = nullptr;
    uint32_t* d_M = nullptr;
    uint32_t* d_off = nullptr;
    void* d_zeros = nullptr;           // 256 bytes of zeros: where masked operand loads point instead of branching
    uint32_t* d_tile_base = nullptr;   // [kListKinds][MT_MAX_LAYERS][T+1]: FC, conv and big-FC arrays, then one word: the big-tile layer mask
    void* d_act[kActBuffers] = {};
    float* d_logits = nullptr;
    Segment* h_segs[kSegSlots] = {};    // pinned, device-visible
    Segment* d_segs[kSegSlots] = {};    // device addresses of the same memory
    hipEvent_t seg_event[kSegSlots] = {};
    bool seg_busy[kSegSlots] = {};
    uint64_t run_count = 0;
    hipStream_t last_stream = nullptr;

    // model cache
    bool cache = false;
    uint64_t use_clock = 0;                 // stamps HostTenant::last_use
    hipEvent_t cache_event = nullptr;       // recorded behind the last asynchronous residency change
    hipStream_t cache_stream = nullptr;
    bool cache_pending = false;
    uint64_t n_uploads = 0, upload_bytes = 0, n_evictions = 0;

    uint32_t plan = 1;                      // registrations and removals so far, and one (BatchArgs::plan)
    PlanUse used;                           // by the runs captured since the last of them (`any`, `act_buffers`, `first` and `chunk_layers`; the rest is noted by close_plan)
    std::vector<PlanUse> plans_used;        // by those captured before, oldest first, each kind once (the newest of it); at most kPlansKept
    uint32_t plans_dropped = 0;             // the newest of those no longer known

    // pending submissions
    std::vector<Segment> pending;
    uint32_t pending_rows = 0;
    std::vector<NamedRows> named;            // scratch of mt_run (count_named); reserved in mt_create
    std::vector<uint32_t> named_at;          // [max_tenants] 1 + a tenant's place in it, 0 between runs

    uint32_t last_run_rows = 0, last_run_launches = 0;
    std::string err;

    // optional per-kernel timing: event 2*i / 2*i+1 bracket launch slot i
    bool profiling = false;
    std::vector<hipEvent_t> prof_events;
    bool prof_used[kProfSlots] = {};
    bool prof_valid = false;
    uint32_t prof_last = 0;
};

namespace {

mt_status fail(mt_ctx* c, mt_status st, const char* fmt, ...)
{
    if (c) {
        char buf[512];
        va_list ap; va_start(ap, fmt); vsnprintf(buf, sizeof buf, fmt, ap); va_end(ap);
        c->err = buf;
    }
    return st;
}

void bind_slot(mt_ctx* c, const RunSlot& r)
{
    c->d_row_tenant = r.d_row_tenant; c->d_row_rank = r.d_row_rank; c->d_hist_g = r.d_hist_g; c->d_row_src = r.d_row_src;
    c->d_pos_of = r.d_pos_of; c->d_perm = r.d_perm; c->d_M = r.d_M; c->d_off = r.d_off; c->d_tile_base = r.d_tile_base;
    for (int i = 0; i < kActBuffers; ++i) c->d_act[i] = r.d_act[i];
    c->d_logits = r.d_logits;
}

#define HIP_TRY(c, expr)                                                                    \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess)                                                               \
            return fail((c), e_ == hipErrorOutOfMemory ? MT_ENOMEM : MT_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

// ---- arena: first-fit free list, blocks merged on release -----------------------------
bool arena_alloc(mt_ctx* c, uint64_t len, uint64_t* off)
{
    len = round_up64(len, kArenaAlign);
    for (size_t i = 0; i < c->free_list.size(); ++i) {
        FreeBlock& b = c->free_list[i];
        if (b.len >= len) {
            *off = b.off;
            b.off += len; b.len -= len;
            if (b.len == 0) c->free_list.erase(c->free_list.begin() + (long)i);
            c->arena_used += len;
            return true;
        }
    }
    return false;
}

void arena_free(mt_ctx* c, uint64_t off, uint64_t len)
{
    len = round_up64(len, kArenaAlign);
    FreeBlock nb{off, len};
    auto it = std::lower_bound(c->free_list.begin(), c->free_list.end(), nb,
                               [](const FreeBlock& a, const FreeBlock& b) { return a.off < b.off; });
    it = c->free_list.insert(it, nb);
    if (it + 1 != c->free_list.end() && it->off + it->len == (it + 1)->off) { it->len += (it + 1)->len; c->free_list.erase(it + 1); }
    if (it != c->free_list.begin() && (it - 1)->off + (it - 1)->len == it->off) { (it - 1)->len += it->len; c->free_list.erase(it); }
    c->arena_used -= len;
}

// how an FC layer's column blocks are grouped into tiles (must match the device code)
uint32_t fc_groups(uint32_t n_pad, uint32_t split_k)
{
    const uint32_t nblk = n_pad / kBrickRows;
    const uint32_t split = split_k ? 1u : (nblk >= 3 ? 4u : nblk);
    return (nblk + split - 1) / split;
}
// ... and the rows of such a tile: 64 where the four waves stand side by side, else 32
uint32_t fc_tile_rows(uint32_t n_pad, uint32_t split_k)
{
    return (!split_k && n_pad / kBrickRows >= 3) ? kTileRows : kTileRows / 2;
}

// Bytes of LDS that the input rows of one row tile take (conv_img_kernel's frame): per sub-image the input rows of
// its output rows and one more above and below, a pixel slot left and right, pixels 16 bytes apart from cin
// elements (a padded three-channel pixel of 16 bytes stands alone).
uint64_t row_tile_frame_bytes(const LayerDev& L, uint32_t es, RowTiling r)
{
    const bool chunk_pixel = L.cin * es == 16;
    const uint32_t n_ih = (r.n_oh - 1) * L.stride + 3;
    return (uint64_t)r.ni * n_ih * (L.in_w + 2) * (L.cin * es + (chunk_pixel ? 0 : 16));
}

// Of the pixel slots and channel blocks that row tiles multiply, the share that holds some (a tile of at most half the slots multiplies half).
double row_tile_share(const LayerDev& L)
{
    const RowTiling r = unpack_row_tiling(L.row_tiles);
    const uint32_t blocks = L.N_pad / kBrickRows, wide = kTileCols / kBrickRows;
    const uint32_t full = r.n_oh * L.out_w, px = L.rows_per_req;
    auto slots = [](uint32_t n) { return n <= (uint32_t)kConvTileRows / 2 ? (uint32_t)kConvTileRows / 2 : (uint32_t)kConvTileRows; };
    const double pixels = r.ni > 1 ? (double)px * r.ni / kConvTileRows : (double)px / ((r.tpi - 1) * slots(full) + slots(px - (r.tpi - 1) * full));
    return pixels * blocks / (blocks <= 2 ? blocks : (blocks + wide - 1) / wide * wide);
}

// Row tiling of a 3x3 convolution (0: none): the most output rows per tile, or the most whole small images (a power
// of two), whose input rows fit the frame.  Tiles of fewer than 128 pixels leave MFMA columns idle; the gathering
// kernels they replace move every input byte nine times through the texture path at a quarter of the rate of a
// contiguous load.
uint32_t choose_row_tiling(const LayerDev& L, uint32_t es)
{
    // (stride 2: a tile's frame is four times its output rows, its workgroups sit alone on their CUs with the
    // zeroing, the copy and the K loop in a row; measured slower than the gathers on every such layer of r18 and c4)
    if (L.stride != 1) return 0;
    const uint64_t budget = kConvFrameMaxBytes;
    const uint32_t kb = 32 / es, rpr = L.rows_per_req;
    if (L.ksize != 3 || L.pad != 1 || L.out_w == 0 || L.out_w > (uint32_t)kConvTileRows) return 0;
    if (L.cin % kb != 0 && L.cin * es != 16) return 0;
    const uint32_t H = rpr / L.out_w;
    for (uint32_t ni = 8; ni >= 2; ni >>= 1) {               // whole images side by side
        const RowTiling r{H, ni, 1};
        if (rpr * ni <= (uint32_t)kConvTileRows && row_tile_frame_bytes(L, es, r) <= budget) return pack_row_tiling(r);
    }
    for (uint32_t n_oh = std::min<uint32_t>(H, (uint32_t)kConvTileRows / L.out_w); n_oh >= 1; --n_oh) {
        const RowTiling r{n_oh, 1, (H + n_oh - 1) / n_oh};
        if (r.tpi < 65536 && row_tile_frame_bytes(L, es, r) <= budget) return pack_row_tiling(r);
    }
    return 0;
}

// LDS of a tile of conv_first_kernel: the input rows of `rows` rows of the layer's output, or of the max-pool's behind it (else null).
uint64_t first_frame_bytes(const LayerDev& L, const LayerDev* pool, uint32_t es, uint32_t rows)
{
    const uint64_t conv_rows = pool ? std::min((rows - 1) * pool->stride + pool->ksize, L.rows_per_req / L.out_w) : rows;
    return ((conv_rows - 1) * L.stride + L.ksize) * first_frame_cols(L) * kFirstMaxCin * es;
}

// The same of conv_pair_kernel: the first layer's rows under `rows` rows of the second one's output, and their input.
void pair_lds(const LayerDev& L, const LayerDev& second, uint32_t es, uint32_t rows, uint64_t* frame, uint64_t* mid)
{
    const uint32_t need = (rows - 1) * second.stride + 3;
    *frame = first_frame_bytes(L, nullptr, es, std::min(need, L.rows_per_req / L.out_w));
    *mid = (uint64_t)need * (L.out_w + 2) * (second.cin * es + 16);
}

// Most rows of such a tile: up to 128 pixels; 0: its rows are too long or too wide.
uint32_t choose_pair_rows(const LayerDev& L, const LayerDev& second, uint32_t es)
{
    const uint32_t H = second.rows_per_req / second.out_w;
    if (L.N_pad > kFirstBlocks * kBrickRows || second.N_pad > kPairMaxBlocks * kBrickRows || second.cin % (32 / es) || second.out_w > (uint32_t)kConvTileRows || H > 0xffffu || L.in_w > 0xffffu) return 0;
    for (uint32_t rows = std::min<uint32_t>(H, (uint32_t)kConvTileRows / second.out_w); rows >= 1; --rows) {
        uint64_t frame, mid;
        pair_lds(L, second, es, rows, &frame, &mid);
        if (frame + 16 + mid <= kPairLdsBytes) return rows;
    }
    return 0;
}

// MFMA steps of a window of 32 pixels and 32 channels in conv_first_kernel.
uint32_t first_steps(uint32_t ksize, uint32_t es) { return es == 2 ? (ksize * ksize + 1) / 2 : ksize * ((ksize + 1) / 2); }

// Whether the two layers are at least as fast with each other as by a launch each, from one request to thousands.  A tile (at most `rows` rows) multiplies the first layer's
// rows above and below it once more, and pixel slots that its rows do not fill; one request has its tiles' two walks through K one behind the other, in four waves.
// Passes over those with staged images, with each other / by a launch each, most requests (4096, or 2^18 pixels): bf16, 32 -> 64 channels at stride 2, images 4 / 6 / 8 / 10 / 12 / 16 / 32 / 64
// wide 1.06 / 1.03 / 0.98 / 0.89 / 0.75 / 0.74 / 0.73 / 0.74 against 0.92 / 0.93 / 0.91 / 0.89 / 0.80 / 0.89 / 0.87 / 0.89, 64 -> 128 1.32 / 1.11 / 1.01 / 0.91 / 0.72 / 0.73 / 0.75 / 0.76 against 0.88 /
// 0.85 / 0.85 / 0.83 / 0.78 / 0.86 / 0.87 / 0.85.  fp32, where multiplications decide: the steps of a tile's longest wave against those of full tiles: 24 -> 40 over 29x35 1.12 (0.91 against
// 0.94), 64 -> 64 over 28x28 1.05 (0.92 / 0.93), 24x24 1.26 (0.99 / 0.93), 32x32 1.43 (1.06 / 0.93), 32 -> 32 over 32x32 2.0 (1.01 / 0.91), one or two rows to a tile: 64 -> 32 over 48x48 1.68 / 0.92,
// 64 -> 128 at stride 2 over 40x40 1.80 / 0.88.  One request in fp32: 66 steps (24 -> 40) 0.94-1.08, 162 (64 -> 64) 1.05-1.27, 270 (64 -> 128) 1.26.
bool pair_pays(const LayerDev& L, const LayerDev& second, uint32_t es, uint32_t rows)
{
    constexpr uint32_t kMostSteps = 72;
    constexpr double kMostMore = 1.25;
    const uint32_t px0 = L.rows_per_req, px1 = second.rows_per_req, h1 = px1 / second.out_w, b0 = L.N_pad / kBrickRows, b1 = second.N_pad / kBrickRows;
    if (px1 < (es == 4 ? 32u : b0 > 1 ? 24u : 16u)) return false;      // (few requests gain by small tiles too: 16 -> 32 over 8x8, one and 24 of them 0.81 / 0.79 against 0.98 / 0.90)
    if (es == 2) return true;
    auto ceil_div = [](uint32_t a, uint32_t b) { return (a + b - 1) / b; };
    const uint32_t tiles = ceil_div(h1, rows), step = ceil_div(h1, tiles), need = std::min((step - 1) * second.stride + 3, px0 / L.out_w);
    const uint32_t units = b1 <= 2 ? 2 : 4, unit = step * second.out_w <= units / 2 * kBrickRows ? units / 2 : units;      // pixel blocks of a wave (conv_pair_kernel)
    const uint32_t s0 = first_steps(L.ksize, es), s1 = second.k_valid * es / 32, longest = ceil_div(ceil_div(need * L.out_w, kBrickRows), 4 / b0) * s0 + unit * s1;
    const double full = ((double)px0 * b0 * s0 + (double)px1 * b1 * s1 / (second.row_tiles ? row_tile_share(second) : 1.0)) / kBrickRows / 4;
    return longest <= kMostSteps && tiles * longest <= kMostMore * full;
}

// Whether such a layer is at least as fast that way as on staged images, from one request to thousands.  A tile holds pixels of one image, where the tiles
// of the staged kernels run on over the images, and a row of pixels is walked by one workgroup.  Passes over the staged ones, most requests (8192, or 2^18
// pixels) and 64 channels unless noted: 3x3, 1x1 to 6x6 images 1.19 / 0.87 / 0.82 / 0.81 / 0.80 / 0.78 bf16 and 1.54 / 0.96 / 0.93 / 0.95 / 0.84 / 0.75 fp32, at
// stride 2 1.18 / 1.17 / 1.10 / 1.12 / 1.03 / 1.04 and 1.54 / 1.52 / 1.30 / 1.28 / 1.20 / 1.20, 512 channels 1.44 / 1.41 / 1.21 / 1.35 / 1.04 / 0.90; from 8x8 on 0.7-1.0 all.
// 7x7 at stride 2, 8x8 / 10x10 / 12x12 1.11 / 1.00 / 0.91 and 1.18 / 1.03 / 0.82.  Long rows and few of them, one request (and many): fp32 7x7 and 32 channels,
// 30x260 1.16 (0.73), 20x150 1.06 (0.66), 40x130 1.05 (0.63), 48x200 0.97 (0.67), 12x120 0.94 (0.71); 3x3 and 64, 3x300 1.18 (0.90), 8x200 1.08 (0.80), 20x150 0.95; bf16
// 7x7, 16x700 1.11 (0.79), 30x260 1.01 (0.76).
bool first_pays(const LayerDev& L, uint32_t es)
{
    const uint32_t out_h = L.rows_per_req / L.out_w, row = (L.out_w + kBrickRows - 1) / kBrickRows * std::min<uint32_t>(L.N_pad / kBrickRows, kFirstBlocks) * first_steps(L.ksize, es);
    if (L.in_h * L.in_w < 64 || (L.ksize == 7 && L.rows_per_req < (uint32_t)kBrickRows)) return false;
    return out_h >= 48 || row <= (es == 2 ? 512u : out_h < 10 ? 59u : 112u);
}

// Most rows of such a tile (0: not even one row's input fits LDS, or the image has too many).
uint32_t choose_first_rows(const LayerDev& L, const LayerDev* pool, uint32_t es)
{
    const uint32_t H = pool ? pool->rows_per_req / pool->out_w : L.rows_per_req / L.out_w;
    if (H > 0xffffu || L.in_w > 0xffffu) return 0;
    uint32_t rows = pool ? H : std::min(H, std::max(1u, kFirstTilePixels / L.out_w));
    while (rows > 1 && first_frame_bytes(L, pool, es, rows) > (pool ? kFirstPoolFrameBytes : kFirstFrameBytes)) --rows;
    return first_frame_bytes(L, pool, es, rows) + first_scratch_bytes(es) + 16 <= kFirstMaxBytes ? rows : 0;
}

// Whether the max-pool behind such a layer is better done with it (in tiles of `rows` of its output) than by a launch of its own.  A wave's column of 32 outputs of the
// convolution holds whole windows only, rows shared by two waves' windows are multiplied twice, and some waves of a tile may have no column: `more` is what
// is multiplied over what is needed, less one.  Passes over the staged ones, 2^18 pixels and a 3x3 pool at stride 2, done with it / by itself:
// bf16, where the columns decide, 3x3x64 images 3 / 8 / 10 / 12 / 16 / 24 / 32 / 64 / 224 wide 1.59 / 1.10 / 1.01 / 0.81 / 0.78 / 0.74 / 0.74 / 0.71 / 0.52 against 0.86 / 0.83 /
// 0.85 / 0.80 / 0.88 / 0.86 / 0.85 / 0.87 / 0.77, 7x7x64 at stride 2, 12 / 16 / 24 / 64 wide 1.25 / 0.96 / 0.83 / 0.75 against 0.91 / 0.75 / 0.79 / 0.78.  fp32, whose multiplications take
// eight times as long and weigh against the convolution's output that is neither written nor read: 7x7x64 at stride 2, 48 / 128 / 224 wide 1.06 / 1.18 / 0.68
// against 0.74 / 0.80 / 0.71, 3x3x64 24 / 48 / 96 / 224 wide 0.91 / 0.73 / 0.70 / 0.42 against 0.76 / 0.78 / 0.77 / 0.85, 3x3x8 1.01 / 0.83 / 0.74 / 0.65 against 0.76 / 0.75 / 0.71 / 0.74.
bool first_pool_pays(const LayerDev& L, const LayerDev& pool, uint32_t es, uint32_t rows)
{
    auto ceil_div = [](uint32_t a, uint32_t b) { return (a + b - 1) / b; };
    const uint32_t h = pool.rows_per_req / pool.out_w, columns = ceil_div(pool.out_w, ((uint32_t)kBrickRows - pool.ksize) / pool.stride + 1);
    if (columns * kBrickRows > 2 * L.out_w) return false;
    if (es == 2) return true;
    const uint32_t waves = 8 / std::min<uint32_t>(L.N_pad / kBrickRows, kFirstBlocks), parts = std::max(waves / columns, 1u);
    const uint32_t per = ceil_div(ceil_div(h, ceil_div(h, rows)), parts), units = columns * parts;
    const double more = (double)(columns * kBrickRows) / L.out_w * ((per - 1) * pool.stride + pool.ksize) / (per * pool.stride) * (ceil_div(units, waves) * waves) / units - 1.0;
    return more * first_steps(L.ksize, es) <= (L.ksize == 7 ? 9.5 : 3.0) * L.N / L.N_pad;      // (the 7x7 at 224 and 48 above: 9.3 and 15.6; the 3x3x64 at 96 and 24: 2.3 and 3.3)
}

// Rows of an image that the tiles of such a layer deal out: of its output, or of the max-pool's that is done with it.
uint32_t first_out_rows(const HostTenant& t)
{
    const LayerDev& last = t.layers[t.layers[0].dev.first_pool ? 1 : 0].dev;
    return last.rows_per_req / last.out_w;
}

// The same of one model in a run whose tiles have at most `cap` rows; pair: with the second layer.
FirstNeed first_need(const LayerDev& conv, const LayerDev& next, bool pair, uint32_t es, uint32_t cap)
{
    const LayerDev& out = pair || conv.first_pool ? next : conv;
    const uint32_t h = out.rows_per_req / out.out_w, strips = first_strips(h, pair ? next.pair_rows : conv.first_rows, cap), rows = (h + strips - 1) / strips;
    FirstNeed n{};
    if (pair) pair_lds(conv, next, es, rows, &n.frame, &n.mid);
    else n.frame = first_frame_bytes(conv, conv.first_pool ? &next : nullptr, es, rows);
    n.tiles = (uint64_t)strips * ((conv.N_pad / kBrickRows + kFirstBlocks - 1) / kFirstBlocks);
    return n;
}

// The batcher's words per layer of one tenant (see BatchArgs::facts).
void fill_facts(const mt_ctx* c, const HostTenant& ht, uint32_t (*w)[kFactWords])
{
    for (uint32_t l = 0; l < MT_MAX_LAYERS; ++l) for (uint32_t i = 0; i < (uint32_t)kFactWords; ++i) w[l][i] = 0;
    for (uint32_t l = 0; l < ht.n_layers; ++l) {
        const LayerDev& L = ht.layers[l].dev;
        if (L.kind == MT_FC) {
            w[l][0] = fc_groups(L.N_pad, c->fc_split_k) | (fc_tile_rows(L.N_pad, c->fc_split_k) == kTileRows ? 0u : 1u << 30) | (l > 0 && L.is_last && fc_whole(L.N_pad) ? 1u << 29 : 0u);
            w[l][1] = L.N_pad;
        } else if (L.kind == MT_CONV2D) {
            w[l][0] = L.N_pad / kBrickRows | 1u << 31;
            w[l][1] = conv_tile_rows(L.rows_per_req, L.row_tiles);
            w[l][2] = L.rows_per_req;
            if (L.first_rows) w[l][3] = first_out_rows(ht) | L.first_rows << 16;
            else if (L.pair_rows) w[l][3] = L.rows_per_req / L.out_w | L.pair_rows << 16;
        }
    }
}

// What a tenant's device state is uploaded from, in one host block: the arena image
// (arena_len bytes), then its rows of the three device tables.
struct StageTail {
    LayerDev rows[MT_MAX_LAYERS];
    TenantDev td;
    uint32_t facts[MT_MAX_LAYERS][kFactWords];
};
size_t stage_tail_offset(uint64_t arena_len) { return (size_t)round_up64(arena_len, 256); }
size_t stage_bytes(uint64_t arena_len) { return stage_tail_offset(arena_len) + sizeof(StageTail); }

// A tenant's rows of the three device tables travel inside kernel arguments: the runtime copies
// those when the launch is enqueued, so the host may change its copy (a later placement of the same
// model at another arena offset) while this one is still queued behind earlier work.  An asynchronous
// copy from the host block would read it only when it executes.  Kernel arguments are limited to a
// few kilobytes, so the layer rows go in pieces of kLayerGroup layers; the tenant row goes with the
// last piece, after a fence: a tenant that the batcher sees has its layer rows in place.
struct RowsPiece {
    LayerDev rows[kLayerGroup];
    uint32_t facts[kLayerGroup][kFactWords];
    TenantDev td;
};
static_assert(sizeof(RowsPiece) <= 2048, "a piece of a tenant's table rows must fit kernel arguments");
__global__ void install_rows_kernel(RowsPiece piece, LayerDev* rows, uint32_t* facts, uint32_t n_tenants, TenantDev* td)
{
    const uint32_t* src_rows = (const uint32_t*)piece.rows;
    for (uint32_t i = threadIdx.x; i < sizeof(piece.rows) / 4; i += blockDim.x) ((uint32_t*)rows)[i] = src_rows[i];
    for (uint32_t i = threadIdx.x; i < sizeof(piece.facts) / 4; i += blockDim.x)
        facts[(size_t)(i / kFactWords) * n_tenants * kFactWords + i % kFactWords] = piece.facts[i / kFactWords][i % kFactWords];
    if (!td) return;
    __threadfence();
    __syncthreads();
    const uint32_t* src_td = (const uint32_t*)&piece.td;
    for (uint32_t i = threadIdx.x; i < sizeof(piece.td) / 4; i += blockDim.x) ((uint32_t*)td)[i] = src_td[i];
}

hipError_t install_rows(mt_ctx* c, uint32_t tenant, const StageTail& tail, hipStream_t s);

// Point the tenant's layer descriptors at arena block `off` and refresh the table rows in its stage.
void place_tenant(const mt_ctx* c, HostTenant& ht, uint64_t off, uint8_t* stage)
{
    ht.arena_off = off;
    StageTail* tail = (StageTail*)(stage + stage_tail_offset(ht.arena_len));
    *tail = StageTail{};
    for (uint32_t l = 0; l < ht.n_layers; ++l) {
        ht.layers[l].dev.w_off = off + ht.layers[l].w_rel;
        ht.layers[l].dev.b_off = off + ht.layers[l].b_rel;
        tail->rows[l] = ht.layers[l].dev;
    }
    tail->td = ht.dev;
    fill_facts(c, ht, tail->facts);
}

hipError_t install_rows(mt_ctx* c, uint32_t tenant, const StageTail& tail, hipStream_t s)
{
    // a tenant that disappears (n_layers 0) loses its tenant row first, in the first piece
    const uint32_t n_pieces = tail.td.registered ? (tail.td.n_layers + kLayerGroup - 1) / kLayerGroup : MT_MAX_LAYERS / kLayerGroup;
    for (uint32_t g = 0; g < n_pieces; ++g) {
        RowsPiece piece;
        std::memcpy(piece.rows, tail.rows + g * kLayerGroup, sizeof piece.rows);
        std::memcpy(piece.facts, tail.facts + g * kLayerGroup, sizeof piece.facts);
        piece.td = tail.td;
        const bool with_td = tail.td.registered ? g + 1 == n_pieces : g == 0;
        hipLaunchKernelGGL(install_rows_kernel, dim3(1), dim3(256), 0, s, piece, c->d_layers + (size_t)tenant * MT_MAX_LAYERS + g * kLayerGroup,
                           c->d_facts + ((size_t)g * kLayerGroup * c->cfg.max_tenants + tenant) * kFactWords, c->cfg.max_tenants, with_td ? c->d_tenants + tenant : nullptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Copy a placed tenant's weights and table rows to the device: on `s` without waiting (the arena
// image in the stage must be pinned and is never changed again; the table rows are taken from the
// stage now, see install_rows_kernel), or synchronously.
hipError_t upload_tenant(mt_ctx* c, uint32_t tenant, const HostTenant& ht, const uint8_t* stage, hipStream_t s, bool async)
{
    const StageTail* tail = (const StageTail*)(stage + stage_tail_offset(ht.arena_len));
    hipError_t e = async ? hipMemcpyAsync(c->d_arena + ht.arena_off, stage, (size_t)ht.arena_len, hipMemcpyHostToDevice, s)
                         : hipMemcpy(c->d_arena + ht.arena_off, stage, (size_t)ht.arena_len, hipMemcpyHostToDevice);
    if (e != hipSuccess) return e;
    e = install_rows(c, tenant, *tail, async ? s : nullptr);          // behind the weights on the same stream
    if (e != hipSuccess) return e;
    if (!async) { e = hipStreamSynchronize(nullptr); if (e != hipSuccess) return e; }
    c->n_uploads++; c->upload_bytes += ht.arena_len;
    return hipSuccess;
}

// Take a tenant's model off the device: the batcher no longer sees it, its arena block is free.
hipError_t hide_tenant(mt_ctx* c, uint32_t tenant, hipStream_t s, bool async)
{
    const hipError_t e = install_rows(c, tenant, StageTail{}, async ? s : nullptr);
    if (e != hipSuccess || async) return e;
    return hipStreamSynchronize(nullptr);
}

// Find `len` bytes of arena.  In cache mode, models used least recently (and before `protect`)
// give way until the block fits; their stages stay in host memory.
bool make_room(mt_ctx* c, uint64_t len, uint64_t protect, hipStream_t s, bool async, uint64_t* off, hipError_t* err)
{
    *err = hipSuccess;
    while (!arena_alloc(c, len, off)) {
        if (!c->cache) return false;
        int victim = -1;
        for (uint32_t t = 0; t < c->cfg.max_tenants; ++t) {
            const HostTenant& h = c->tenants[t];
            if (h.registered && h.resident && h.last_use < protect && (victim < 0 || h.last_use < c->tenants[victim].last_use)) victim = (int)t;
        }
        if (victim < 0) return false;
        HostTenant& v = c->tenants[victim];
        if (!c->host_only) { *err = hide_tenant(c, (uint32_t)victim, s, async); if (*err != hipSuccess) return false; }
        arena_free(c, v.arena_off, v.arena_len);
        v.resident = false;
        c->n_evictions++;
    }
    return true;
}

void recompute_pool_fusion(mt_ctx* c)
{
    for (uint32_t l = 0; l + 1 < MT_MAX_LAYERS; ++l) {
        bool any = false, all = true;
        for (const HostTenant& t : c->tenants) {
            if (!t.registered || t.n_layers <= l + 1) continue;
            any = true;
            all = all && t.layers[l + 1].dev.kind == MT_GAP && t.layers[l].dev.pool_fill != 0;
        }
        c->pool_fused[l] = any && all && !c->no_fused_pool;
    }
}

// Whether a last layer of 33 to 128 classes takes less time in tiles of all its column blocks than in one per block with the head's launch behind them.  Two blocks at once, and
// the pairs in turn, are a longer walk through K than one block by itself: some 0.12 us for each k step of a wave's quarter in fp32, 0.04 in bf16; the launch takes 1 to 3.  One request
// to one model of 256-256-K-C / 64 to four / 300 to one, us a pass with the head's launch and so: fp32, C = 64, K = 512 24.3 / 24.6 / 27.2 -> 21.9 / 22.2 / 27.2, 768 24.4 / 25.2 / 28.6 ->
// 23.7 / 24.2 / 29.1 (2048: 30.0 -> 34.1); C = 128, 128 23.6 / 23.8 / 27.0 -> 21.6 / 21.6 / 26.4, 192 23.8 / 23.9 / 27.1 -> 22.5 / 22.6 / 27.3 (2048: 29.9 -> 50.8); bf16, C = 64, 2048
// 23.4 / 23.5 / 27.2 -> 20.8 / 20.9 / 26.3, 4096 21.9 / - / 34.1 -> 21.2 / - / 34.1; C = 128, 1024 23.0 / 23.3 / 27.0 -> 21.2 / 21.2 / 26.0, 1536 23.2 / 23.4 / 27.3 -> 21.5 / 21.9 / 27.7.
bool whole_pays(const mt_ctx* c, const LayerDev& L)
{
    const uint32_t steps = L.K * c->elem_size / 128, pairs = (L.N_pad / kBrickRows + 1) / 2;
    return steps * (2 * pairs - 1) <= (c->elem_size == 2 ? 64 : 16);
}

void recompute_bounds(mt_ctx* c)
{
    c->n_layer_slots = 0;
    c->max_in_len = c->max_fc_in_len = 0; c->max_image_pixels = 0; c->min_layers = 0xffffffffu;
    c->fc_first_chunked = true; c->any_conv_first = c->any_fc_first = false;
    for (uint32_t& m : c->list_mask) m = 0;
    c->max_reg_classes = 0; c->min_reg_classes = 0xffffffffu; c->wide_last_unfit = false; c->sum_macs = 0.0;
    c->first_on = !c->no_conv_first; c->first_pool = c->first_plain = false; c->pair_on = !c->no_conv_pair;
    c->first_max_ks = c->first_max_rows = c->pair_blocks = c->n_conv_first = 0; c->first_max_tiles = 0;
    for (const HostTenant& t : c->tenants) {         // (ahead of the others: it says which max-pools have a launch)
        if (!t.registered || t.dev.in_layout == kLayoutBricks) continue;
        const LayerDev& L = t.layers[0].dev;
        c->any_conv_first = true; ++c->n_conv_first;
        if (!L.first_rows) { c->first_on = false; continue; }
        (L.first_pool ? c->first_pool : c->first_plain) = true;
        c->first_max_ks = std::max(c->first_max_ks, L.ksize);
        c->first_max_tiles = std::max<uint64_t>(c->first_max_tiles, (uint64_t)first_out_rows(t) * ((L.N_pad / kBrickRows + kFirstBlocks - 1) / kFirstBlocks));
        const LayerDev& second = t.layers[t.n_layers > 1 ? 1 : 0].dev;
        if (!second.pair_rows) c->pair_on = false;
        c->pair_blocks = std::max(c->pair_blocks, second.N_pad / kBrickRows);
        c->first_max_rows = std::max(c->first_max_rows, L.first_rows);
    }
    c->first_on = c->first_on && c->any_conv_first;
    c->pair_on = c->pair_on && c->first_on;
    if (c->pair_on) {                                // tiles are rows of the second layer's output then
        c->first_max_rows = 0; c->first_max_tiles = 0;
        for (const HostTenant& t : c->tenants) {
            if (!t.registered || t.dev.in_layout == kLayoutBricks) continue;
            c->first_max_rows = std::max(c->first_max_rows, t.layers[1].dev.pair_rows);
            c->first_max_tiles = std::max<uint64_t>(c->first_max_tiles, t.layers[1].dev.rows_per_req / t.layers[1].dev.out_w);
        }
    }
    for (uint32_t l = 0; l < MT_MAX_LAYERS; ++l) {
        c->has_gap[l] = 0; c->gap_chunks[l] = 0; c->has_image_ops[l] = 0; c->image_op_fill[l] = 0; c->min_conv_k[l] = 0xffffffffu; c->max_conv_k[l] = 0; c->max_conv_work[l] = 0; c->max_conv_tile_rows[l] = 0; c->sum_conv_work[l] = 0; c->max_conv_blocks[l] = 0; c->sum_conv_blocks[l] = 0; c->min_fc_k[l] = 0xffffffffu; c->max_fc_cols[l] = 0; c->wide_last[l] = false; c->max_conv_cb[l] = 0; c->conv_quad[l] = true; c->conv_uniform[l] = true; c->pool_fused[l] = false; c->conv_img_lds[l] = 1; c->conv_img_two[l] = -1; c->conv_frame_share[l] = 0.0;
        for (int k = 0; k < kListKinds; ++k) { c->max_nt[k][l] = 0; c->sum_nt[k][l] = 0; }
        c->max_fc_per64[l] = 0; c->max_fc_per64_sk[l] = 0; c->sum_nt_sk[l] = 0; c->max_big_blocks[l] = 0;
    }
    for (const HostTenant& t : c->tenants) {
        if (!t.registered) continue;
        c->n_layer_slots = std::max(c->n_layer_slots, t.n_layers);
        c->min_layers = std::min(c->min_layers, t.n_layers);
        c->max_in_len = std::max(c->max_in_len, t.dev.in_len);
        c->max_reg_classes = std::max(c->max_reg_classes, t.dev.n_classes);
        c->min_reg_classes = std::min(c->min_reg_classes, t.dev.n_classes);
        if (t.dev.in_layout == kLayoutBricks) {
            c->any_fc_first = true;
            c->max_fc_in_len = std::max(c->max_fc_in_len, t.dev.in_len);
            if ((t.dev.in_len * c->elem_size) % 16) c->fc_first_chunked = false;
        } else {
            c->max_image_pixels = std::max(c->max_image_pixels, t.dev.in_len / (t.dev.in_cin ? t.dev.in_cin : (uint32_t)kChanPad));
        }
        for (uint32_t l = 0; l < t.n_layers; ++l) {
            const LayerDev& L = t.layers[l].dev;
            if (L.kind == kKindNone) continue;
            if (L.kind == MT_GAP) { c->has_gap[l] = 1; c->gap_chunks[l] = std::max(c->gap_chunks[l], std::min<uint64_t>((uint64_t)L.in_h * L.in_w, kGapSweepPixels) * L.cin * c->elem_size / 16); continue; }
            if (l == 1 && c->first_on && t.layers[0].dev.first_pool) continue;          // done with the convolution in front of it
            if (l == 1 && c->pair_on && L.pair_rows) { c->sum_macs += (double)L.k_valid * L.N * L.rows_per_req; continue; }
            if (L.kind == MT_MAXPOOL || L.kind == MT_ADD) { c->has_image_ops[l] = 1; c->image_op_fill[l] = std::max(c->image_op_fill[l], L.out_fill); continue; }
            const int k = L.kind == MT_FC ? 0 : 1;
            c->sum_macs += (double)L.k_valid * L.N * L.rows_per_req;
            c->list_mask[l / kLayerGroup] |= 1u << (k * kLayerGroup + l % kLayerGroup);
            const uint32_t nt = k == 0 ? fc_groups(L.N_pad, c->fc_split_k) : (L.N + kTileCols - 1) / kTileCols;
            c->max_nt[k][l] = std::max(c->max_nt[k][l], nt);
            c->sum_nt[k][l] += nt;
            if (k == 0) {
                c->min_fc_k[l] = std::min(c->min_fc_k[l], L.K);
                c->max_fc_cols[l] = std::max(c->max_fc_cols[l], L.N_pad);
                if (L.is_last && fc_whole(L.N_pad)) { c->wide_last[l] = true; c->wide_last_unfit = c->wide_last_unfit || l == 0 || !whole_pays(c, L); }
                c->max_fc_per64[l] = std::max(c->max_fc_per64[l], nt * (kTileRows / fc_tile_rows(L.N_pad, c->fc_split_k)));
                const uint32_t nt_sk = fc_groups(L.N_pad, 1);
                c->sum_nt_sk[l] += nt_sk;
                c->max_fc_per64_sk[l] = std::max(c->max_fc_per64_sk[l], nt_sk * (kTileRows / fc_tile_rows(L.N_pad, 1)));
            }
            if (k == 1) {
                c->min_conv_k[l] = std::min(c->min_conv_k[l], L.k_valid);
                const uint64_t work = (uint64_t)L.rows_per_req * (L.N_pad / kBrickRows);
                c->max_conv_work[l] = std::max(c->max_conv_work[l], work);
                c->max_conv_tile_rows[l] = std::max(c->max_conv_tile_rows[l], (uint64_t)conv_tile_rows(L.rows_per_req, L.row_tiles) * nt);
                c->max_conv_k[l] = std::max(c->max_conv_k[l], L.k_valid);
                c->max_conv_blocks[l] = std::max(c->max_conv_blocks[l], L.N_pad / kBrickRows);
                c->sum_conv_work[l] += work;
                c->sum_conv_blocks[l] += L.N_pad / kBrickRows;
                c->max_conv_cb[l] = std::max(c->max_conv_cb[l], std::min<uint32_t>(L.N_pad / kBrickRows, kTileCols / kBrickRows));
                if (L.cin % (4 * (16 / c->elem_size))) c->conv_quad[l] = false;
                if (L.cin % (2 * (16 / c->elem_size)) || L.ksize * L.ksize > 64) c->conv_uniform[l] = false;
                // frame of one tile of the LDS-resident-input kernel (conv_img_kernel), which serves the layer index
                // when every tenant's layer is row-tiled
                const bool chunk_pixel = L.cin * c->elem_size == 16;            // a pixel is one 16-byte chunk: two taps per k step, no padding
                const uint64_t frame = L.row_tiles ? row_tile_frame_bytes(L, c->elem_size, unpack_row_tiling(L.row_tiles)) : 0;
                if (c->conv_img_two[l] < 0) c->conv_img_two[l] = chunk_pixel;
                if (L.row_tiles) c->conv_frame_share[l] = std::max(c->conv_frame_share[l], row_tile_share(L));
                if (frame == 0 || c->conv_img_lds[l] == 0 || c->conv_img_two[l] != (int)chunk_pixel) c->conv_img_lds[l] = 0;
                else c->conv_img_lds[l] = std::max<uint32_t>(c->conv_img_lds[l], (uint32_t)frame);
            }
            if (k == 0 && L.N_pad >= (uint32_t)kBigMinCols && l < (uint32_t)kBigMaxLayer) {      // may be served with big tiles when it gets enough rows
                c->list_mask[l / kLayerGroup] |= 1u << (2 * kLayerGroup + l % kLayerGroup);
                c->max_nt[2][l] = std::max(c->max_nt[2][l], (L.N_pad + kBigTile - 1) / kBigTile);
                if (big_remainder_split_k(L.N_pad)) c->max_big_blocks[l] = std::max(c->max_big_blocks[l], L.N_pad / kBrickRows);
            }
        }
    }
}

// The most that the registered models take.
FirstNeed most_first_need(const mt_ctx* c, uint32_t cap)
{
    FirstNeed m{};
    for (const FirstShape& s : c->first_shapes) {
        const FirstNeed n = first_need(s.conv, s.next, c->pair_on, c->elem_size, cap);
        m.frame = std::max(m.frame, n.frame); m.mid = std::max(m.mid, n.mid); m.tiles = std::max(m.tiles, n.tiles);
    }
    return m;
}

// Keeps mt_ctx::first_shapes: a model comes (+1) or goes (-1).
void note_first_shape(mt_ctx* c, const HostTenant& t, int by)
{
    if (t.dev.in_layout == kLayoutBricks || !t.layers[0].dev.first_rows) return;
    FirstShape s{t.layers[0].dev, t.layers[1].dev, 1};
    s.conv.w_off = s.conv.b_off = s.next.w_off = s.next.b_off = 0;
    auto it = std::find_if(c->first_shapes.begin(), c->first_shapes.end(), [&](const FirstShape& o) {
        return std::memcmp(&o.conv, &s.conv, sizeof s.conv) == 0 && std::memcmp(&o.next, &s.next, sizeof s.next) == 0;
    });
    if (it == c->first_shapes.end()) c->first_shapes.push_back(s);
    else if ((it->models += (uint32_t)by) == 0) c->first_shapes.erase(it);
}

// Whether a run that was planned like `u` can serve a model registered since.
bool covers(const mt_ctx* c, const PlanUse& u, const HostTenant& m)
{
    const bool images = m.dev.in_layout != kLayoutBricks;
    if (m.act_buffers > u.act_buffers || m.n_layers > u.layer_slots) return false;
    for (uint32_t l = 0; l < m.n_layers; ++l)
        if (m.layers[l].dev.kind == MT_CONV2D && ((u.chunk_layers >> l) & 1) && m.layers[l].dev.cin % (4 * (16 / c->elem_size))) return false;
    if (!u.first || !images) return true;
    const LayerDev &conv = m.layers[0].dev, &next = m.layers[1].dev;
    if (!conv.first_rows || !(conv.first_pool ? u.pool : u.plain) || (conv.ksize > 3 && u.max_ks <= 3)) return false;
    if (u.pair && (!next.pair_rows || (u.pair_blocks <= 2 && next.N_pad / kBrickRows > 2))) return false;
    if (!u.ops1 && !conv.first_pool && (next.kind == MT_MAXPOOL || next.kind == MT_ADD)) return false;
    for (uint32_t i = 0; i < u.most.size(); ++i) {                   // any of these a run may have had
        const FirstNeed n = first_need(conv, next, u.pair, c->elem_size, u.cap ? u.cap : i + 1), &most = u.most[i];
        if (n.frame > most.frame || n.mid > most.mid || n.tiles > most.tiles) return false;
    }
    return true;
}

// A registration or a removal follows: the runs from now on are another plan's.
void close_plan(mt_ctx* c)
{
    PlanUse& u = c->used;
    if (u.any) try {
        u.plan = c->plan; u.layer_slots = c->n_layer_slots;
        if (u.first) {
            u.pair = c->pair_on; u.pool = c->first_pool; u.plain = c->first_plain; u.ops1 = c->has_image_ops[1];
            u.max_ks = c->first_max_ks; u.pair_blocks = c->pair_blocks; u.cap = c->first_cap;
            u.most.resize(u.cap ? 1 : c->first_max_rows);
        }
        for (uint32_t i = 0; i < u.most.size(); ++i) u.most[i] = most_first_need(c, u.cap ? u.cap : i + 1);
        c->plans_used.erase(std::remove_if(c->plans_used.begin(), c->plans_used.end(), [&](const PlanUse& o) { return o.same_as(u); }), c->plans_used.end());
        if (c->plans_used.size() == kPlansKept) { c->plans_dropped = c->plans_used.front().plan; c->plans_used.erase(c->plans_used.begin()); }
        c->plans_used.push_back(std::move(u));
    } catch (const std::bad_alloc&) {                // nothing registered from now on is served by a run captured before
        c->plans_used.clear();
        c->plans_dropped = c->plan;
    }
    u = PlanUse{};
    c->plan++;
}

// The first plan from which on every captured run covers a model that is about to be registered.
uint32_t first_plan_for(const mt_ctx* c, const HostTenant& m)
{
    for (size_t i = c->plans_used.size(); i-- > 0;)
        if (!covers(c, c->plans_used[i], m)) return c->plans_used[i].plan + 1;
    return c->plans_dropped + 1;
}

// Upper bound of the number of tiles of one list over any split of R rows among tenants.
uint64_t tile_bound(const mt_ctx* c, int kind, uint32_t l, uint64_t R, bool split_k = false, bool big_enabled = false)
{
    if (c->max_nt[kind][l] == 0) return 0;
    // streaming tiles of a run with big tiles: the tenants that big tiles serve (at most R / kBigMinRows of them) leave
    // at most kBigRemRows rows each, in narrow layers tiled 32 rows and one column block at a time
    if (kind == 0 && big_enabled && !split_k)
        return tile_bound(c, 0, l, R) + (R / kBigMinRows) * (kBigRemRows / kBrickRows) * c->max_big_blocks[l];
    if (kind == 2)      // big FC tiles: only tenants with >= kBigMinRows rows; sum ceil(M_t/256) <= R/256 + R/kBigMinRows
        return R < (uint64_t)kBigMinBatch ? 0 : (uint64_t)c->max_nt[2][l] * (R / kBigTile + R / kBigMinRows);
    // sum over tenants of ceil(M_t / rows_t) * groups_t <= R * max(groups_t / rows_t) + sum(groups_t): the maximum of the quotient, not
    // of its two parts, which may be two models' (one with many pixels, one with many channels: a launch past 2^32 work items)
    if (kind == 0 && split_k) return ((uint64_t)c->max_fc_per64_sk[l] * R + kTileRows - 1) / kTileRows + c->sum_nt_sk[l];
    if (kind == 0) return ((uint64_t)c->max_fc_per64[l] * R + kTileRows - 1) / kTileRows + c->sum_nt[0][l];
    return R * c->max_conv_tile_rows[l] / kConvTileRows + c->sum_nt[1][l];
}

// Tile shape of the FC layers of a run over R rows.  When no layer index can have more than
// kSplitKMaxTiles ordinary tiles the launches fill a fraction of the chip and their duration is one
// wave's walk through K (on the fp32 mix of four small models: 13-16 us per layer, most of it the
// fp32 MFMAs of a 256- or 512-step K loop in a single wave).  Such runs take tiles of one column
// block whose four waves split K (and 32 rows): four times the workgroups, a quarter of the walk.
constexpr uint64_t kSplitKMaxTiles = 128;
bool run_split_k(const mt_ctx* c, uint64_t R)
{
    if (c->fc_split_k) return true;
    if (c->no_auto_split_k) return false;
    // at most min(R, registered models) tenants have rows, each with one ragged row tile per column group
    const uint64_t active = std::min<uint64_t>(R, c->n_registered);
    uint64_t most = 0;
    for (uint32_t l = 0; l < c->n_layer_slots; ++l)
        most = std::max(most, ((uint64_t)c->max_fc_per64[l] * R + kTileRows - 1) / kTileRows + active * c->max_nt[0][l]);
    return most > 0 && most <= kSplitKMaxTiles;
}

// How the convolutions of a layer index are launched in a run of R rows.
struct ConvPlan {
    bool frames;        // tiles read their input from LDS frames
    bool split;         // tiles of 32 pixels and one channel block whose waves split K
    uint32_t first_cap; // > 0: the submitted images are read (layer index 0), in tiles of at most so many rows ...
    uint32_t first_frame; // ... whose input takes at most so many bytes of LDS
    uint32_t pair_mid;  // > 0: ... and the convolutions behind them with them: the tiles are rows of those; bytes of LDS for the first layer's rows
    uint64_t tiles;     // upper bound of the launch's tiles
};

// Convolution launches of at most so many tiles of 32 pixels and one channel block take such tiles, K split among their waves.
// Chains of eight equal layers, split over unsplit time (one tenant; the tiles of 16 waves come in rounds of 256).  LDS frames in bf16 at 256 / 512 / 640
// tiles: 18 k steps (16x16x32) 0.81 / 0.88 / 1.00, 36 (8x8x64) 0.81 / 0.91 / 1.06, 72 (28x28x128) 0.63 / 0.96 / 1.25, 144 (14x14x256) 0.52 / 0.81 / 1.06,
// 288 (7x7x512) 0.64 / 1.29 / 1.29, and 0.94 at 320.  In fp32 at 512 / 768 / 1536 / 2048: 36 (16x16x32) 0.89 / 1.12, 27 (32x32x24, 1024) 1.14, 72 (8x8x64)
// 0.78 / 0.97 / 1.52, 144 (28x28x128) 0.33 / 0.54 / 0.85 / 1.06.  Gathers, whole passes of three convolutions the last of which has stride 2, split and unsplit, us: bf16,
// 36 steps 39 / 40 us at 640 tiles, 72 steps 43 / 46 at 496, 47 / 46 at 640, 144 steps 43 / 59 at 256, 58 / 60 at 400, 68 / 60 at 528; fp32, 45 steps 59 / 71 at
// 1029, 72 steps 103 / 108 at 1032, 116 / 109 at 1544, 144 steps 127 / 151 at 1520, 221 / 186 at 3088, 288 steps 240 / 264 at 1552.  (The bf16 lines of long
// gathers and of frames stay above the crossing: another order of the sums turns roundings, and with them close labels, of deep bf16 nets.)
// fp32 frames are long in bytes: images of many channels leave most of a frame's tile empty.  A k step of a split tile then takes less than its share of a frame's
// tile does where it can load whole chunks, however many tiles there are: nanoseconds of a compute unit, fitted to 8192 tiles, measured 41 against 122 (7x7x512, a share of 0.26), 47 / 57
// (14x14x256, 0.58), 55 / 89 (9x9x160, 0.4), 58 / 65 (12x12x40, 0.75), and where the frames stay 63 / 50 (28x28x128, 0.88), 80 / 61 (20x20x72, 0.6), 80 / 40 (8x8x64, 1), 76 / 49 (16x16x32, 1).
uint64_t conv_split_line(const mt_ctx* c, uint32_t l, bool frames)
{
    constexpr uint32_t kFewSteps = 24, kManySteps = 192, kMostTiles = 1u << 20;        // (a launch of 16 waves a tile stays below 2^32 work items)
    constexpr double kSplitStepNs = 35.0, kSplitTileNs = 3200.0, kFrameStepNs = 40.0;
    if (c->conv_split_tiles >= 0) return (uint64_t)c->conv_split_tiles;
    const uint32_t k_steps = (c->max_conv_k[l] * c->elem_size + 31) / 32;
    if (!frames) return c->elem_size == 2 ? 768 : k_steps > 128 ? 1536 : 1024;
    if (c->elem_size == 4) {
        if (c->conv_quad[l] && k_steps > 64 && kSplitStepNs + kSplitTileNs / k_steps < kFrameStepNs / c->conv_frame_share[l]) return kMostTiles;
        return k_steps >= 128 || (k_steps <= 64 && c->conv_frame_share[l] < 0.8) ? 1536 : k_steps > 64 ? 768 : 640;        // (12x12x40 at 1638: 0.83)
    }
    return k_steps <= kFewSteps ? 768 : k_steps <= kManySteps ? 512 : 256;
}
// Where the host does not know whose the requests are, it takes them to be spread evenly, unless their all being the
// heaviest model's would make more than so many times the tiles of conv_split_line.  64 tenants, one of them a chain of five convolutions
// that all requests go to, at 1 / 2 / 4 times: 28x28x128, 8 requests 95 / 141 / 141 us, 14x14x256, 32 requests 134 / 133 / 284 (with no
// such limit 128 requests to the first 1306 instead of 237); MLPs, CNNs and small residual nets by turns, 600 requests 246 / 214 / 206.
constexpr uint64_t kConvSplitSkew = 2;

// Most rows of a tile of the first convolutions in a run of R rows to models that start with one: the whole batch in about two workgroups to a compute unit.  A workgroup takes 4-9 us
// to find its tenant, its filters and its pixels, and more of them do not hide that from each other.  Launches in us at 512 / 1024 / 2048 / 4096
// workgroups (as far as tiles go): 64 images 224x224 through 7x7x64 and its max-pool 48 / 56 / 60 / 92, 2048 images 32x32 (3x3x32) 33.5 / 33.8 / 33.2 /
// 35.1, 500 of them 11.4 / 11.9 / 14.3 / 18.9, 150 fp32 29x35 (3x3x24) 14.5 / 14.2 / 17.7 / 24.6, MLPs, CNNs and residual nets by turns, 600 requests
// 13.3 / 16.4 / 19.9 / 28.4.
uint32_t first_tile_rows(const mt_ctx* c, uint64_t R)
{
    if (c->first_cap) return c->first_cap;
    const uint64_t wanted = 2 * c->n_cus;
    return (uint32_t)std::min<uint64_t>((std::max<uint64_t>(R, 1) * c->first_max_tiles + wanted - 1) / wanted, c->first_max_rows);
}

// `named`: the requests of every tenant that has any, where each submission named its tenant; null where some stand in a
// device-resident id array; captured: replays may find other models of those tenants
ConvPlan plan_conv(const mt_ctx* c, uint32_t l, uint64_t R, const std::vector<NamedRows>* named, bool captured = false)
{
    ConvPlan p{};
    if (l == 0 && c->first_on) {
        // Where the host does not know whose the requests are: all of them, or, where at most half of the models start with a convolution, their
        // share of an even spread and at least an eighth.  512 requests to 32x32x64 layers and MLPs, 10 of them to the former, us a pass with tiles for 512 and for the
        // share: one model of 16 61.7 / 52.6, four of eight 59.2 / 54.2; 150 of them 60.0 / 53.3 and 57.9 / 53.1; MLPs, CNNs and residual nets by turns, 600 requests 194.1 / 196.6.
        const uint64_t models = c->n_registered, share = 2 * c->n_conv_first > models ? 8 * models : std::max<uint64_t>(8 * (uint64_t)c->n_conv_first, models);
        uint64_t images = (R * share + 8 * models - 1) / (8 * models);
        if (named) {
            images = 0;
            for (const NamedRows& r : *named) if (c->tenants[r.tenant].dev.in_layout != kLayoutBricks) images += r.rows;
        }
        p.first_cap = first_tile_rows(c, images);
        const FirstNeed most = most_first_need(c, p.first_cap);
        p.first_frame = (uint32_t)most.frame; p.pair_mid = (uint32_t)most.mid;
        p.tiles = R * most.tiles;
        if (named && !captured) {
            p.tiles = 0;
            for (const NamedRows& r : *named) {
                const HostTenant& t = c->tenants[r.tenant];
                if (t.dev.in_layout != kLayoutBricks) p.tiles += r.rows * first_need(t.layers[0].dev, t.layers[1].dev, c->pair_on, c->elem_size, p.first_cap).tiles;
            }
            p.tiles = std::max<uint64_t>(p.tiles, 1);      // (none: an empty launch, as mt_estimate_run counts them)
        }
        return p;
    }
    p.frames = c->conv_img_lds[l] > 1 && !c->pool_fused[l] && !c->no_conv_img;
    p.tiles = tile_bound(c, 1, l, R);
    if (c->max_nt[1][l] == 0 || c->pool_fused[l]) return p;
    const uint64_t line = conv_split_line(c, l, p.frames), active = std::min<uint64_t>(R, c->n_registered);
    // at most (every request the heaviest model's): the same bound as in tile_bound, with the ragged tiles of those with requests
    uint64_t tiles = R * c->max_conv_work[l] / kBrickRows + std::min<uint64_t>(c->sum_conv_blocks[l], active * c->max_conv_blocks[l]);
    bool split = tiles <= line;
    if (!split && named) {
        uint64_t n = 0;
        for (const NamedRows& r : *named) {
            const HostTenant& t = c->tenants[r.tenant];
            if (l >= t.n_layers || t.layers[l].dev.kind != MT_CONV2D) continue;
            const LayerDev& L = t.layers[l].dev;
            n += ((uint64_t)r.rows * L.rows_per_req + kBrickRows - 1) / kBrickRows * (L.N_pad / kBrickRows);
            if (n > line) break;
        }
        split = n <= line;
        if (split) tiles = std::max<uint64_t>(n, 1);          // (none: an empty launch, as mt_estimate_run counts them)
    } else if (!split) {
        // the requests spread evenly over the registered models, a ragged tile per channel block of those with requests
        const uint64_t even = R * c->sum_conv_work[l] / c->n_registered / kBrickRows + active * c->sum_conv_blocks[l] / c->n_registered / 2;
        split = even <= line && tiles <= kConvSplitSkew * line;
    }
    if (split) { p.split = true; p.frames = false; p.tiles = tiles; }
    return p;
}

// How the FC layers of index 0 get their rows.  They read them themselves where every row is a whole number of 16-byte chunks at such addresses, and
// else (a lane's 16 bytes begin anywhere, in two cache lines as often as not) while that is few lane addresses: a compute unit takes 2.4 clocks for each,
// and all of a layer's column groups ask for every row.  Staged, and read so, us a pass, bf16: 301-333-520-37, 8 tenants, 5 / 200 / 20000 requests 28.7 / 30.6 / 86.1 -> 21.8 / 24.1 / 79.9;
// 787-1024-512-10, 32 tenants, 200 / 1000 / 5000 (15300 lane addresses to a compute unit) 52.7 / 58.5 / 73.4 -> 41.4 / 52.2 / 73.1; 1023-4000-64, 1 tenant, 200 / 1000 (16400) / 5000
// (82000) 43.8 / 55.7 / 111.9 -> 40.6 / 58.1 / 186.4; 3001-2500-10, 2 tenants, 200 (23000) 49.8 -> 64.9.  fp32, whose tiles wait for their MFMAs: 1023-4000-64, 1000 / 5000 (164000) 133.1 / 403.3 ->
// 123.1 / 416.1, 3001-2500-10, 1000 (58000) 232.9 -> 232.4.
// pending: as submitted, else chunked wherever the models allow.
constexpr uint64_t kAnyRowsLanes = 14000, kAnyRowsLanesF32 = 128000;
int first_rows(const mt_ctx* c, uint64_t R, bool split_k, bool big_possible, bool pending)
{
    if (!c->any_fc_first || c->no_fused_gather || big_possible) return kRowsStaged;
    bool chunked = c->fc_first_chunked;
    if (pending)
        for (const Segment& sg : c->pending) chunked = chunked && ((uintptr_t)sg.src & 15) == 0 && ((uint64_t)sg.row_stride * c->elem_size) % 16 == 0;
    if (chunked) return kRowsChunked;
    const uint64_t chunks = (uint64_t)c->max_fc_in_len * c->elem_size / 16 + 1, groups = split_k ? (c->max_fc_per64_sk[0] + 1) / 2 : c->max_fc_per64[0];
    const uint64_t lanes = std::max<uint64_t>((split_k ? kBrickRows : kTileRows) * chunks, R * groups * chunks / c->n_cus);
    return lanes <= (c->elem_size == 2 ? kAnyRowsLanes : kAnyRowsLanesF32) ? kRowsAny : kRowsStaged;
}

// Whether layer 0 does the batcher's work in a run of one submission of R rows that it reads itself: few tenants, nothing but FC layers, and no model that is
// finished there.  kEntryNarrow: few rows and nothing but tiles that split K; kEntryWide: any tiles, as long as they start together (three workgroups to a compute
// unit): every tile of a second round does the segmentation once more behind the first.  us a pass, with the batcher's launch and so, bf16: 64 tenants of
// 784-1024-1024-10, 320 / 1024 / 2048 requests 58.1 / 58.7 / 66.0 -> 53.9 / 54.3 / 61.3; 16 of 512-512-512-10, 320 / 1024 / 2048 / 4096 22.9 / 29.3 / 33.0 / 41.8 ->
// 18.9 / 25.4 / 28.8 / 37.4; one of 1024-2048-2048-40, 320 / 2048 / 3000 (at most 766 tiles) 39.7 / 66.7 / 86.3 -> 36.4 / 63.8 / 82.5.  Beyond the upper line, when
// these tiles still spilled registers: 4096 of the last (1040 tiles) 110.2 -> 112.7, of the first (1024) 100.9 -> 100.2, three runs in flight 215.0 -> 221.6.
// The lower line is no measured crossing: 257 requests to the first took 52.4 in place of 54.6, and by the same trips to memory so would any from 65 on.  Up to
// 319 rows runs of ordinary tiles keep a launch per layer and one, which is what their estimates have promised.
constexpr uint32_t kEntryWideMin = 320;
constexpr uint64_t kEntryWideTilesPerCu = 3;
enum : int { kEntryNone = 0, kEntryNarrow, kEntryWide };
int run_entry(const mt_ctx* c, uint64_t R, bool split_k)
{
    if (c->cfg.max_tenants > kEntryMaxTenants || c->no_entry || c->any_conv_first || !c->any_fc_first || c->min_layers < 2) return kEntryNone;
    if (R <= kEntryMaxRows && (split_k || c->max_fc_cols[0] <= 2 * (uint32_t)kBrickRows)) return kEntryNarrow;
    return R >= kEntryWideMin && R <= kEntryWideRows && tile_bound(c, 0, 0, R, split_k) <= kEntryWideTilesPerCu * c->n_cus ? kEntryWide : kEntryNone;
}

// Whether last layers of 33 to 128 classes take tiles of all their column blocks in a run whose tiles split K (fc_whole_tile): where it pays for all of them, as the head's launch
// does the rows of all or of none.  Not where such a layer is a model's first, which reads submitted rows; nor in captured runs, whose replays may meet such a model.
bool run_whole(const mt_ctx* c, bool split_k, bool captured) { return split_k && !captured && !c->no_fused_head && !c->wide_last_unfit; }

// Most classes a last layer may have for its FC tiles to finish their rows themselves (softmax, argmax, outputs): one column block (32), or a whole tile of
// four (128) where the run's tiles are not single column blocks, or take all of such a layer's; 0: the head kernel does every row.
uint32_t fused_head_classes(const mt_ctx* c, bool split_k, bool whole)
{
    if (c->no_fused_head) return 0;
    return split_k && !whole ? (uint32_t)kBrickRows : (uint32_t)kTileCols;
}

// ---- validation of a layer chain; fills dev layouts (without arena offsets) -------------
mt_status plan_model(mt_ctx* c, const mt_layer_spec* specs, uint32_t n_layers, HostTenant* out)
{
    if (n_layers == 0 || n_layers > MT_MAX_LAYERS)
        return fail(c, MT_EUNSUPPORTED, "a model needs 1..%d layers, got %u", MT_MAX_LAYERS, n_layers);
    const uint32_t es = c->elem_size;
    out->n_layers = n_layers;
    out->dev = TenantDev{};
    // Values: 0 is the request, l + 1 the output of layer l.  A layer reads the value before it unless
    // its spec names another one (skip connections); shape[] is what every value looks like.
    struct Shape { uint32_t h, w, ch, len; bool image; };
    Shape shape[MT_MAX_LAYERS + 1] = {};
    uint32_t src_of[MT_MAX_LAYERS] = {}, src2_of[MT_MAX_LAYERS] = {}, last_use[MT_MAX_LAYERS + 1] = {};
    for (uint32_t l = 0; l < n_layers; ++l) {
        const mt_layer_spec& s = specs[l];
        HostLayer& hl = out->layers[l];
        hl.spec = s;
        LayerDev d{};
        d.kind = s.kind; d.act = s.act; d.is_last = (l == n_layers - 1);
        d.stride = 1; d.out_w = 1; d.rows_per_req = 1;
        if (s.act > MT_ACT_GELU) return fail(c, MT_EUNSUPPORTED, "layer %u: activation %u is not in the supported set", l, s.act);
        if (d.is_last && s.act != MT_ACT_NONE) return fail(c, MT_EUNSUPPORTED, "layer %u: the last layer yields logits and takes no activation", l);
        if (s.src > l || s.src2 > l) return fail(c, MT_EUNSUPPORTED, "layer %u: a layer can only read outputs of earlier layers", l);
        if (s.src2 != 0 && s.kind != MT_ADD) return fail(c, MT_EUNSUPPORTED, "layer %u: only an addition takes a second source", l);
        const uint32_t src = s.src ? s.src : l;              // value read: the named one, else the one before this layer
        src_of[l] = src; last_use[src] = l;
        const Shape in = shape[src];                         // (undefined for the request: the first layer defines it)
        const bool first = l == 0;
        const bool image_kind = s.kind == MT_CONV2D || s.kind == MT_GAP || s.kind == MT_MAXPOOL || s.kind == MT_ADD;
        if (image_kind) {
            if (s.in_features == 0 || s.in_h == 0 || s.in_w == 0) return fail(c, MT_EINVAL, "layer %u: zero-sized image", l);
            if ((uint64_t)s.in_h * s.in_w * s.in_features > 0x7fffffffu) return fail(c, MT_EUNSUPPORTED, "layer %u: image too large", l);
            if (!first && (!in.image || in.h != s.in_h || in.w != s.in_w || in.ch != s.in_features))
                return fail(c, MT_EUNSUPPORTED, "layer %u takes a %ux%ux%u image but its source yields %s of %u values", l, s.in_h, s.in_w, s.in_features,
                            in.image ? "another image" : "a vector", in.len);
            if (d.is_last) return fail(c, MT_EUNSUPPORTED, "layer %u: the last layer must be fully connected", l);
        }
        Shape o{};
        if (s.kind == MT_FC) {
            if (s.in_features == 0 || s.out_features == 0) return fail(c, MT_EINVAL, "layer %u: zero-sized FC", l);
            if (!first && in.image)
                return fail(c, MT_EUNSUPPORTED, "layer %u: an FC layer cannot read an image directly; pool first", l);
            if (!first && in.len != s.in_features) return fail(c, MT_EUNSUPPORTED, "layer %u takes %u values but its source yields %u", l, s.in_features, in.len);
            d.K = round_up(s.in_features, kWidthAlign); d.k_valid = s.in_features; d.N = s.out_features;
            d.N_pad = round_up(s.out_features, d.is_last ? kBrickRows : kWidthAlign);
            d.out_len = s.out_features;
            hl.w_bytes = (uint64_t)d.N_pad * d.K * es; hl.b_bytes = (uint64_t)d.N_pad * 4;
            o = Shape{1, 1, s.out_features, s.out_features, false};
        } else if (s.kind == MT_CONV2D) {
            if (s.kh != s.kw || (s.kh != 1 && s.kh != 3 && s.kh != 7) || s.pad != (s.kh - 1) / 2 || (s.stride != 1 && s.stride != 2))
                return fail(c, MT_EUNSUPPORTED, "layer %u: convolutions are 1x1, 3x3 or 7x7 with pad (k - 1) / 2 and stride 1 or 2", l);
            if (s.out_features == 0) return fail(c, MT_EINVAL, "layer %u: zero-sized conv", l);
            if (s.out_features % kChanPad) return fail(c, MT_EUNSUPPORTED, "layer %u: conv output channels must be a multiple of %d", l, kChanPad);
            if (!first && s.in_features % kChanPad) return fail(c, MT_EUNSUPPORTED, "layer %u: conv input channels must be a multiple of %d past the first layer", l, kChanPad);
            const uint32_t oh = (s.in_h + 2 * s.pad - s.kh) / s.stride + 1, ow = (s.in_w + 2 * s.pad - s.kw) / s.stride + 1;
            d.cin = round_up(s.in_features, kChanPad);
            d.in_h = s.in_h; d.in_w = s.in_w; d.stride = s.stride; d.out_w = ow; d.ksize = s.kh; d.pad = s.pad;
            d.rows_per_req = oh * ow;
            d.K = round_up(s.kh * s.kw * d.cin, kWidthAlign); d.k_valid = s.kh * s.kw * d.cin; d.N = s.out_features; d.N_pad = round_up(s.out_features, kBrickRows);
            d.out_len = oh * ow * s.out_features;
            hl.w_bytes = (uint64_t)d.N_pad * d.K * es; hl.b_bytes = (uint64_t)d.N_pad * 4;
            o = Shape{oh, ow, s.out_features, d.out_len, true};
        } else if (s.kind == MT_GAP) {
            if (s.out_features != s.in_features || s.act != MT_ACT_NONE) return fail(c, MT_EUNSUPPORTED, "layer %u: pooling keeps the channel count and has no activation", l);
            if (first) return fail(c, MT_EUNSUPPORTED, "layer %u: pooling cannot be the first layer", l);
            d.cin = s.in_features; d.in_h = s.in_h; d.in_w = s.in_w; d.N = s.in_features; d.N_pad = s.in_features;
            d.out_len = s.in_features;
            hl.w_bytes = hl.b_bytes = 0;
            o = Shape{1, 1, s.in_features, s.in_features, false};
        } else if (s.kind == MT_MAXPOOL) {
            if (s.kh != s.kw || (s.kh != 2 && s.kh != 3) || s.pad > 1 || s.pad >= s.kh || (s.stride != 1 && s.stride != 2))
                return fail(c, MT_EUNSUPPORTED, "layer %u: max-pooling takes 2x2 or 3x3 windows, pad 0 or 1, stride 1 or 2", l);
            if (s.out_features != s.in_features || s.act != MT_ACT_NONE) return fail(c, MT_EUNSUPPORTED, "layer %u: pooling keeps the channel count and has no activation", l);
            if (first) return fail(c, MT_EUNSUPPORTED, "layer %u: pooling cannot be the first layer", l);
            if (s.in_h + 2 * s.pad < s.kh || s.in_w + 2 * s.pad < s.kw) return fail(c, MT_EUNSUPPORTED, "layer %u: the window exceeds the image", l);
            const uint32_t oh = (s.in_h + 2 * s.pad - s.kh) / s.stride + 1, ow = (s.in_w + 2 * s.pad - s.kw) / s.stride + 1;
            d.cin = s.in_features; d.in_h = s.in_h; d.in_w = s.in_w; d.stride = s.stride; d.out_w = ow; d.ksize = s.kh; d.pad = s.pad;
            d.rows_per_req = oh * ow; d.N = s.in_features; d.N_pad = s.in_features;
            d.out_len = oh * ow * s.in_features;
            hl.w_bytes = hl.b_bytes = 0;
            o = Shape{oh, ow, s.in_features, d.out_len, true};
        } else if (s.kind == MT_ADD) {
            if (first || s.src2 == 0) return fail(c, MT_EUNSUPPORTED, "layer %u: an addition names its second source and cannot be the first layer", l);
            if (s.out_features != s.in_features) return fail(c, MT_EUNSUPPORTED, "layer %u: an addition keeps the channel count", l);
            const Shape in2 = shape[s.src2];
            if (!in2.image || in2.h != s.in_h || in2.w != s.in_w || in2.ch != s.in_features)
                return fail(c, MT_EUNSUPPORTED, "layer %u: the second source is not a %ux%ux%u image", l, s.in_h, s.in_w, s.in_features);
            src2_of[l] = s.src2; last_use[s.src2] = l;
            d.cin = s.in_features; d.in_h = s.in_h; d.in_w = s.in_w; d.out_w = s.in_w; d.rows_per_req = s.in_h * s.in_w;
            d.N = s.in_features; d.N_pad = s.in_features;
            d.out_len = s.in_h * s.in_w * s.in_features;
            hl.w_bytes = hl.b_bytes = 0;
            o = Shape{s.in_h, s.in_w, s.in_features, d.out_len, true};
        } else {
            return fail(c, MT_EUNSUPPORTED, "layer %u: kind %u is not in the supported set", l, s.kind);
        }
        if (s.kind != MT_FC && s.in_features % kChanPad && !(first && s.kind == MT_CONV2D))
            return fail(c, MT_EUNSUPPORTED, "layer %u: image channels must be a multiple of %d", l, kChanPad);
        shape[l + 1] = o;
        d.out_fill = round_up(d.out_len, kWidthAlign);
        if (first) {
            const uint32_t in_len = s.kind == MT_FC ? s.in_features : s.in_h * s.in_w * s.in_features;
            out->dev.in_len = in_len;
            uint32_t staged = in_len;
            if (s.kind == MT_CONV2D && d.cin != s.in_features) {
                out->dev.in_cin = s.in_features; out->dev.in_cin_pad = d.cin;
                staged = s.in_h * s.in_w * d.cin;
            }
            out->dev.in_fill = round_up(staged, kWidthAlign);
            out->dev.in_layout = s.kind == MT_FC ? kLayoutBricks : kLayoutRows;
            if (out->dev.in_fill > c->S) return fail(c, MT_EUNSUPPORTED, "input of %u values exceeds max_width", in_len);
        }
        if (!d.is_last && d.out_fill > c->S) return fail(c, MT_EUNSUPPORTED, "layer %u output of %u values exceeds max_width", l, d.out_len);
        if (s.kind == MT_FC && d.K > c->S) return fail(c, MT_EUNSUPPORTED, "layer %u fan-in %u exceeds max_width", l, s.in_features);
        if (d.is_last && d.out_len > c->cfg.max_classes) return fail(c, MT_EUNSUPPORTED, "%u classes exceed max_classes", d.out_len);
        hl.dev = d;
    }
    out->dev.n_layers = n_layers;
    out->dev.n_classes = shape[n_layers].len;

    // A convolution whose output goes to a global average pool and nowhere else can pool by itself
    // when every image lies inside one wave's pixel blocks; its input then has to outlive the pooling
    // layer's index, because the pooled activation is written where that layer would have written it.
    for (uint32_t l = 1; l < n_layers; ++l) {
        if (out->layers[l].dev.kind != MT_GAP || src_of[l] != l || out->layers[l - 1].dev.kind != MT_CONV2D) continue;
        LayerDev& conv = out->layers[l - 1].dev;
        last_use[src_of[l - 1]] = std::max(last_use[src_of[l - 1]], l);
        if (conv.N % kWidthAlign == 0 && (conv.rows_per_req == kBrickRows || conv.rows_per_req == 2 * kBrickRows) && last_use[l] == l)
            conv.pool_fill = round_up(out->layers[l].dev.N, kWidthAlign);
    }
    // A convolution whose output goes to a residual addition right behind it and nowhere else adds the
    // other operand itself (rounding its own output first, as the addition would have read it) and writes
    // what the addition would have written; the addition's index is then empty for this tenant.
    bool fused_add[MT_MAX_LAYERS] = {};
    for (uint32_t l = 1; l < n_layers && !c->no_fused_add; ++l) {
        const LayerDev& add = out->layers[l].dev;
        LayerDev& conv = out->layers[l - 1].dev;
        if (add.kind != MT_ADD || conv.kind != MT_CONV2D || conv.pool_fill || last_use[l] != l) continue;
        if (src_of[l] != l && src2_of[l] != l) continue;                            // neither operand is that convolution's output
        const uint32_t other = src_of[l] == l ? src2_of[l] : src_of[l];
        if (other == l) continue;                                                   // x + x
        fused_add[l] = true;
        conv.fuse_add = 1 + add.act;
        src2_of[l - 1] = other;                                                     // the convolution reads it now
    }
    // Activation buffers: the request sits in buffer 0; a layer writes the lowest-numbered buffer that
    // holds no value still to be read at or after its index (its own inputs included).  A plain chain
    // alternates between two buffers.
    uint32_t buf_of[MT_MAX_LAYERS + 1] = {};
    out->act_buffers = 1;
    for (uint32_t l = 0; l < n_layers; ++l) {
        LayerDev& d = out->layers[l].dev;
        d.in_buf = buf_of[src_of[l]];
        d.in2_buf = (d.kind == MT_ADD || d.fuse_add) ? buf_of[src2_of[l]] : 0;
        if (d.is_last) break;                                 // logits have a buffer of their own
        if (fused_add[l]) {                                   // the sum is where the convolution before wrote it
            buf_of[l + 1] = buf_of[l]; d.out_buf = buf_of[l]; d.kind = kKindNone;
            continue;
        }
        uint32_t pick = kActBuffers;
        for (uint32_t b = 0; b < (uint32_t)kActBuffers && pick == (uint32_t)kActBuffers; ++b) {
            bool busy = false;
            for (uint32_t v = 0; v <= l; ++v) busy = busy || (buf_of[v] == b && last_use[v] >= l);
            if (!busy) pick = b;
        }
        if (pick == (uint32_t)kActBuffers)
            return fail(c, MT_EUNSUPPORTED, "layer %u: more than %d layer outputs are alive at once", l, kActBuffers);
        buf_of[l + 1] = pick; d.out_buf = pick;
        out->act_buffers = std::max(out->act_buffers, pick + 1);
    }
    for (uint32_t l = 0; l + 1 < n_layers; ++l)
        if (out->layers[l].dev.pool_fill) out->layers[l].dev.pool_buf = out->layers[l + 1].dev.out_buf;
    for (uint32_t l = 0; l < n_layers && !c->no_conv_img; ++l) {
        LayerDev& d = out->layers[l].dev;
        if (d.kind == MT_CONV2D && !d.pool_fill) d.row_tiles = choose_row_tiling(d, es);
    }
    // A first convolution of images with few channels can read them as submitted, and take a max-pool that is its only reader with it.
    if (LayerDev& d = out->layers[0].dev; d.kind == MT_CONV2D && specs[0].in_features <= kFirstMaxCin && !d.pool_fill && !d.fuse_add && (c->first_cap || first_pays(d, es))) {
        const LayerDev* pool = n_layers > 1 && out->layers[1].dev.kind == MT_MAXPOOL && src_of[1] == 1 && last_use[1] == 1 ? &out->layers[1].dev : nullptr;
        d.first_rows = pool ? choose_first_rows(d, pool, es) : 0;
        if (d.first_rows && !c->first_cap && !first_pool_pays(d, *pool, es, d.first_rows)) d.first_rows = 0;
        d.first_pool = d.first_rows != 0;
        if (!d.first_pool) { pool = nullptr; d.first_rows = choose_first_rows(d, nullptr, es); }
        if (d.first_rows && !pool && n_layers > 2 && d.ksize <= 3 && src_of[1] == 1 && last_use[1] == 1) {
            LayerDev& second = out->layers[1].dev;
            const uint32_t rows = second.kind == MT_CONV2D && second.ksize == 3 && !second.pool_fill && !second.fuse_add ? choose_pair_rows(d, second, es) : 0;
            second.pair_rows = rows && (c->first_cap || pair_pays(d, second, es, rows)) ? rows : 0;
        }
        d.first_cin = specs[0].in_features;
    }
    return MT_OK;
}

// Arena image of one layer: bricks[n_block][k_block][lane][EPC] with lane = row + 32*half (zero
// rows and columns as padding), the order in which a wavefront consumes MFMA operands.  The
// reduction index k is the fan-in for FC; for conv the filters [Co][Ci][kh][kw] are read as
// k = (kh*ksize + kw) * ci_padded + ci, so that a GEMM k index walks the NHWC input contiguously.
// (On a line of the instruction cache: registration is this loop, 10 % slower where it happened to straddle two.)
template <typename T>
__attribute__((aligned(64))) void pack_weights(const HostLayer& hl, const void* w_src, uint8_t* dst)
{
    const LayerDev& d = hl.dev;
    const T* src = (const T*)w_src;
    T* out = (T*)dst;
    std::memset(dst, 0, hl.w_bytes);
    constexpr uint32_t EPC = 16 / sizeof(T), KB = 2 * EPC;
    const uint32_t nKB = d.K / KB;
    auto put = [&](uint32_t n, uint32_t k, T v) {
        const uint32_t nb = n / kBrickRows, i = n % kBrickRows, kb = k / KB, h = (k % KB) / EPC, e = k % EPC;
        out[(((size_t)nb * nKB + kb) * 64 + i + 32 * h) * EPC + e] = v;
    };
    if (d.kind == MT_FC) {
        const uint32_t K = hl.spec.in_features;
        for (uint32_t n = 0; n < d.N; ++n)
            for (uint32_t k = 0; k < K; ++k) put(n, k, src[(size_t)n * K + k]);
    } else {
        const uint32_t Ci = hl.spec.in_features, ks = d.ksize;
        for (uint32_t co = 0; co < d.N; ++co)
            for (uint32_t ci = 0; ci < Ci; ++ci)
                for (uint32_t kh = 0; kh < ks; ++kh)
                    for (uint32_t kw = 0; kw < ks; ++kw)
                        put(co, (kh * ks + kw) * d.cin + ci, src[(((size_t)co * Ci + ci) * ks + kh) * ks + kw]);
    }
}

// ---- batch normalisation folded into the convolution in front of it ---------------------------
// Nearest-even rounding of a double to bfloat16 (bit pattern), done on the bits of the double so
// that the value is rounded once: sign, 8 exponent bits, 7 fraction bits; results below 2^-126
// are subnormal (spacing 2^-133), results beyond the largest finite value become infinity.
uint16_t bf16_bits_from_double(double x)
{
    uint64_t u; std::memcpy(&u, &x, 8);
    const uint16_t sign = (uint16_t)((u >> 63) << 15);
    const int64_t e = (int64_t)((u >> 52) & 0x7ff) - 1023;
    const uint64_t frac = u & ((1ull << 52) - 1);
    if (((u >> 52) & 0x7ff) == 0x7ff) return (uint16_t)(sign | 0x7f80 | (frac ? 0x40 : 0));       // infinity / NaN
    if (((u >> 52) & 0x7ff) == 0 || e < -140) return sign;                                        // zero, or far below half the smallest subnormal
    const uint64_t mant = (1ull << 52) | frac;                       // value = mant * 2^(e - 52)
    // keep 7 fraction bits of a normal result; a result below 2^-126 keeps fewer: its last place is 2^-133
    const int shift = e >= -126 ? 45 : (int)(45 + (-126 - e));
    uint64_t kept = mant >> shift;
    const uint64_t rem = mant & ((1ull << shift) - 1), half = 1ull << (shift - 1);
    if (rem > half || (rem == half && (kept & 1))) ++kept;
    if (e >= -126) {
        int64_t be = e + 127;                                        // biased exponent; kept holds the hidden bit (128..256)
        if (kept == 256) { kept = 128; ++be; }
        if (be >= 255) return (uint16_t)(sign | 0x7f80);
        return (uint16_t)(sign | (uint16_t)(be << 7) | (uint16_t)(kept - 128));
    }
    return (uint16_t)(sign | (uint16_t)kept);                        // subnormal; kept == 128 is the smallest normal number
}

bool all_finite_bf16(const uint16_t* w, size_t n)
{
    for (size_t i = 0; i < n; ++i)
        if ((w[i] & 0x7f80) == 0x7f80) return false;
    return true;
}

// W' = round(W * s), b' = float((b - mean) * s + beta) with s = gamma / sqrt(var + eps), per output
// channel, in double precision, each rounded once (no fused multiply-add: the products are rounded
// to double before the sums).  `w` holds the layer's filters [Co][per] in the context's element
// type and is folded in place; `b` its fp32 bias [Co].
#pragma clang fp contract(off)
void fold_batchnorm(uint32_t elem_size, void* w, float* b, uint32_t Co, size_t per, const float* bn, double eps)
{
    const float *gamma = bn, *beta = bn + Co, *mean = bn + 2 * (size_t)Co, *var = bn + 3 * (size_t)Co;
    for (uint32_t c = 0; c < Co; ++c) {
        const double s = (double)gamma[c] / std::sqrt((double)var[c] + eps);
        if (elem_size == 2) {
            uint16_t* row = (uint16_t*)w + c * per;
            for (size_t i = 0; i < per; ++i) {
                const uint32_t wide = (uint32_t)row[i] << 16;
                float f; std::memcpy(&f, &wide, 4);
                const double prod = (double)f * s;
                row[i] = bf16_bits_from_double(prod);
            }
        } else {
            float* row = (float*)w + c * per;
            for (size_t i = 0; i < per; ++i) { const double prod = (double)row[i] * s; row[i] = (float)prod; }
        }
        const double shifted = ((double)b[c] - (double)mean[c]) * s;
        const double sum = shifted + (double)beta[c];
        b[c] = (float)sum;
    }
}

// Offsets of a planned model's layers inside its arena block; returns the block's length.
uint64_t layout_model(HostTenant* ht)
{
    uint64_t total = 0;
    for (uint32_t l = 0; l < ht->n_layers; ++l) {
        HostLayer& hl = ht->layers[l];
        hl.w_rel = total; total += round_up64(hl.w_bytes, kArenaAlign);
        hl.b_rel = total; total += round_up64(hl.b_bytes, kArenaAlign);
    }
    if (total == 0) total = kArenaAlign;
    ht->arena_len = total;
    return total;
}

}  // namespace

extern "C" {

const char* mt_version(void) { return "mt 0.1 gfx950"; }

const char* mt_last_error(const mt_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

mt_status mt_create(mt_ctx** out, const mt_config* cfg)
{
    if (!out || !cfg) return MT_EINVAL;
    *out = nullptr;
    if (cfg->max_tenants == 0 || cfg->max_tenants > kMaxTenants || cfg->max_requests == 0 || cfg->max_width == 0 ||
        cfg->max_classes == 0 || cfg->arena_bytes == 0 || cfg->dtype > MT_BF16 || cfg->run_slots > kMaxRunSlots)
        return MT_EINVAL;
    if ((uint64_t)cfg->max_requests * 4096 > (1ull << 31)) return MT_EINVAL;   // row indices and GEMM row counts stay in 32 bits
    mt_ctx* c = new (std::nothrow) mt_ctx;
    if (!c) return MT_ENOMEM;
    c->cfg = *cfg;
    c->host_only = cfg->device < 0;
    c->elem_size = cfg->dtype == MT_BF16 ? 2 : 4;
    c->S = round_up(cfg->max_width, kWidthAlign);
    c->C_pad = round_up(cfg->max_classes, 4);
    c->named.reserve(cfg->max_tenants);
    c->first_shapes.reserve(cfg->max_tenants);
    c->named_at.assign(cfg->max_tenants, 0);
    c->P_cap = round_up(cfg->max_requests, kBrickRows) + kBrickRows * std::min(cfg->max_tenants, cfg->max_requests);
    if (const char* e = getenv("MT_FC_SPLIT_K")) c->fc_split_k = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_AUTO_SPLIT_K")) c->no_auto_split_k = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_FUSED_GATHER")) c->no_fused_gather = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_FUSED_HEAD")) c->no_fused_head = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_FUSED_POOL")) c->no_fused_pool = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_CONV_IMG")) c->no_conv_img = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_ENTRY")) c->no_entry = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_CONV_PAIR")) c->no_conv_pair = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_CONV_FIRST")) c->no_conv_first = atoi(e) != 0;
    if (const char* e = getenv("MT_FIRST_ROWS")) c->first_cap = (uint32_t)std::max(0, atoi(e));
    if (const char* e = getenv("MT_NO_FUSED_ADD")) c->no_fused_add = atoi(e) != 0;
    if (const char* e = getenv("MT_CONV_SPLIT_TILES")) c->conv_split_tiles = std::max(0, atoi(e));
    if (const char* e = getenv("MT_BIG_WALK")) c->big_walk = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_CONV_LOADERS")) c->no_conv_loaders = atoi(e) != 0;
    if (const char* e = getenv("MT_NO_CONV_UNIFORM")) c->no_conv_uniform = atoi(e) != 0;
    c->big_min_tiles = c->cfg.dtype == MT_BF16 ? kBigMinTiles : kBigMinTilesF32;
    if (const char* e = getenv("MT_BIG_MIN_TILES")) c->big_min_tiles = (uint32_t)std::max(1, atoi(e));
    c->cache = cfg->cache != 0;
    c->tenants.resize(cfg->max_tenants);
    c->cfg.arena_bytes = cfg->arena_bytes / kArenaAlign * kArenaAlign;
    c->free_list.push_back(FreeBlock{0, c->cfg.arena_bytes});
    *out = c;
    if (c->host_only) return MT_OK;

    auto bail = [&](mt_status st) { mt_destroy(c); *out = nullptr; return st; };
#define CREATE_TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) { fprintf(stderr, "mt_create: %s: %s\n", #expr, hipGetErrorString(e_)); return bail(e_ == hipErrorOutOfMemory ? MT_ENOMEM : MT_EDEVICE); } } while (0)
    CREATE_TRY(hipSetDevice(cfg->device));
    {
        int cus = 0;
        CREATE_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, cfg->device));
        c->n_cus = (uint32_t)std::max(cus, 8) / 8 * 8;
    }
    CREATE_TRY(prepare_conv(cfg->dtype));
    CREATE_TRY(prepare_conv_first(cfg->dtype));
    const uint64_t R = cfg->max_requests, T = cfg->max_tenants;
    CREATE_TRY(hipMalloc((void**)&c->d_arena, c->cfg.arena_bytes));
    CREATE_TRY(hipMalloc((void**)&c->d_tenants, T * sizeof(TenantDev)));
    CREATE_TRY(hipMemset(c->d_tenants, 0, T * sizeof(TenantDev)));
    CREATE_TRY(hipMalloc((void**)&c->d_layers, T * MT_MAX_LAYERS * sizeof(LayerDev)));
    CREATE_TRY(hipMemset(c->d_layers, 0, T * MT_MAX_LAYERS * sizeof(LayerDev)));
    CREATE_TRY(hipMalloc((void**)&c->d_facts, kFactWords * MT_MAX_LAYERS * T * 4));
    CREATE_TRY(hipMemset(c->d_facts, 0, kFactWords * MT_MAX_LAYERS * T * 4));
    CREATE_TRY(hipMalloc((void**)&c->d_served, T * 16));
    CREATE_TRY(hipMemset(c->d_served, 0, T * 16));
    CREATE_TRY(hipMalloc(&c->d_zeros, 256));
    CREATE_TRY(hipMemset(c->d_zeros, 0, 256));
    c->slots.resize(std::max<uint32_t>(1, cfg->run_slots));
    for (RunSlot& r : c->slots) {          // (a failed allocation leaves the rest null; mt_destroy frees what exists)
        CREATE_TRY(hipMalloc((void**)&r.d_row_tenant, R * 4));
        CREATE_TRY(hipMalloc((void**)&r.d_row_rank, R * 4));
        CREATE_TRY(hipMalloc((void**)&r.d_hist_g, kHistEntries * 4));
        CREATE_TRY(hipMalloc((void**)&r.d_row_src, R * sizeof(void*)));
        CREATE_TRY(hipMalloc((void**)&r.d_pos_of, R * 4));
        CREATE_TRY(hipMalloc((void**)&r.d_perm, (uint64_t)c->P_cap * 4));
        CREATE_TRY(hipMalloc((void**)&r.d_M, T * 4));
        CREATE_TRY(hipMemset(r.d_M, 0, T * 4));
        CREATE_TRY(hipMalloc((void**)&r.d_off, (T + 1) * 4));
        CREATE_TRY(hipMalloc((void**)&r.d_tile_base, (kListKinds * MT_MAX_LAYERS * (T + 1) + 1) * 4));
        CREATE_TRY(hipMemset(r.d_tile_base, 0, (kListKinds * MT_MAX_LAYERS * (T + 1) + 1) * 4));
        for (uint32_t i = 0; i < c->act_buffers; ++i) {
            CREATE_TRY(hipMalloc(&r.d_act[i], (uint64_t)c->P_cap * c->S * c->elem_size));
        }
        CREATE_TRY(hipMalloc((void**)&r.d_logits, (uint64_t)c->P_cap * c->C_pad * 4));
        CREATE_TRY(hipEventCreateWithFlags(&r.done, kSlotEvent));
    }
    bind_slot(c, c->slots[0]);
    CREATE_TRY(hipGetSymbolAddress((void**)&c->static_scratch, HIP_SYMBOL(scratch)));      // this device's copy of the array
    CREATE_TRY(hipEventCreateWithFlags(&c->static_slot.done, kSlotEvent));
    if (c->cache) {
        CREATE_TRY(hipEventCreateWithFlags(&c->cache_event, hipEventDisableTiming));
    }
    for (uint32_t i = 0; i < kSegSlots; ++i) {
        CREATE_TRY(hipHostMalloc((void**)&c->h_segs[i], R * sizeof(Segment), hipHostMallocMapped));
        CREATE_TRY(hipHostGetDevicePointer((void**)&c->d_segs[i], c->h_segs[i], 0));
        CREATE_TRY(hipEventCreateWithFlags(&c->seg_event[i], hipEventDisableTiming));
    }
#undef CREATE_TRY
    return MT_OK;
}

mt_status mt_destroy(mt_ctx* c)
{
    if (!c) return MT_EINVAL;
    if (!c->host_only) {
        (void)hipSetDevice(c->cfg.device);
        (void)hipDeviceSynchronize();
        void* bufs[] = {c->d_arena, c->d_tenants, c->d_layers, c->d_facts, c->d_served, c->d_zeros};
        for (void* p : bufs) if (p) (void)hipFree(p);
        for (RunSlot& r : c->slots) {
            void* rb[] = {r.d_row_tenant, r.d_row_rank, r.d_hist_g, (void*)r.d_row_src, r.d_pos_of, r.d_perm, r.d_M, r.d_off, r.d_tile_base,
                          r.d_act[0], r.d_act[1], r.d_act[2], r.d_act[3], r.d_logits};
            static_assert(kActBuffers == 4, "the list above names every activation buffer");
            for (void* p : rb) if (p) (void)hipFree(p);
            if (r.done) (void)hipEventDestroy(r.done);
        }
        if (c->static_slot.done) (void)hipEventDestroy(c->static_slot.done);
        for (uint32_t i = 0; i < kSegSlots; ++i) {
            if (c->h_segs[i]) (void)hipHostFree(c->h_segs[i]);
            if (c->seg_event[i]) (void)hipEventDestroy(c->seg_event[i]);
        }
        for (hipEvent_t e : c->prof_events) if (e) (void)hipEventDestroy(e);
        for (HostTenant& t : c->tenants) if (t.stage) (void)hipHostFree(t.stage);
        if (c->cache_event) (void)hipEventDestroy(c->cache_event);
    }
    delete c;
    return MT_OK;
}

mt_status mt_model_footprint_get(const mt_layer_spec* specs, uint32_t n_layers, uint32_t dtype, mt_model_footprint* out)
{
    if (!specs || !out || dtype > MT_BF16) return MT_EINVAL;
    *out = mt_model_footprint{};
    mt_ctx probe;                                   // a context without limits: the plan only depends on the element size
    probe.elem_size = dtype == MT_BF16 ? 2 : 4;
    probe.S = 0xffffffc0u;
    probe.cfg.max_classes = 0xffffffffu;
    HostTenant ht;
    const mt_status st = plan_model(&probe, specs, n_layers, &ht);
    if (st != MT_OK) return st;
    out->arena_bytes = layout_model(&ht);
    out->n_classes = ht.dev.n_classes;
    out->in_len = ht.dev.in_len;
    uint32_t width = ht.dev.in_fill;                // what plan_model holds against max_width
    for (uint32_t l = 0; l < n_layers; ++l) {
        const LayerDev& d = ht.layers[l].dev;
        if (!d.is_last) width = std::max(width, d.out_fill);
        if (d.kind == MT_FC) width = std::max(width, d.K);
    }
    out->min_width = width;
    return MT_OK;
}

mt_status mt_register_model(mt_ctx* c, uint32_t tenant, const mt_layer_spec* specs, uint32_t n_layers,
                            const void* const* weights, const void* const* biases)
{
    return mt_register_model_bn(c, tenant, specs, n_layers, weights, biases, nullptr, 0.0f);
}

mt_status mt_register_model_bn(mt_ctx* c, uint32_t tenant, const mt_layer_spec* specs, uint32_t n_layers,
                               const void* const* weights, const void* const* biases, const float* const* bn, float bn_eps)
{
    if (!c) return MT_EINVAL;
    if (!specs || !weights) return fail(c, MT_EINVAL, "null specs or weights");
    if (tenant >= c->cfg.max_tenants) return fail(c, MT_EINVAL, "tenant %u is outside 0..%u", tenant, c->cfg.max_tenants - 1);
    if (c->tenants[tenant].registered) return fail(c, MT_EEXIST, "tenant %u already has a model", tenant);
    HostTenant ht;
    mt_status st = plan_model(c, specs, n_layers, &ht);
    if (st != MT_OK) return st;
    for (uint32_t l = 0; l < n_layers; ++l) {
        const bool has_params = ht.layers[l].dev.kind == MT_FC || ht.layers[l].dev.kind == MT_CONV2D;
        if (has_params && !weights[l]) return fail(c, MT_EINVAL, "layer %u: null weights", l);
        if (bn && bn[l]) {
            if (ht.layers[l].dev.kind != MT_CONV2D) return fail(c, MT_EUNSUPPORTED, "layer %u: only a convolution can be followed by a batch normalisation", l);
            for (uint32_t ch = 0; ch < ht.layers[l].dev.N; ++ch)
                if (!((double)bn[l][3 * (size_t)ht.layers[l].dev.N + ch] + (double)bn_eps > 0.0))
                    return fail(c, MT_EINVAL, "layer %u: variance + eps of channel %u is not positive", l, ch);
        }
    }

    const uint64_t total = layout_model(&ht);
    if (total > c->cfg.arena_bytes)
        return fail(c, MT_ENOMEM, "model needs %llu bytes, the weight arena has %llu", (unsigned long long)total, (unsigned long long)c->cfg.arena_bytes);

    // the stage: pinned and kept in cache mode (models are reloaded from it), else a temporary
    std::vector<uint8_t> temp;
    uint8_t* stage = nullptr;
    if (!c->host_only) {
        HIP_TRY(c, hipSetDevice(c->cfg.device));
        if (c->cache) {
            if (hipHostMalloc((void**)&stage, stage_bytes(total), hipHostMallocDefault) != hipSuccess)
                return fail(c, MT_ENOMEM, "no pinned host memory for the %llu bytes of tenant %u", (unsigned long long)total, tenant);
            std::memset(stage, 0, stage_bytes(total));
        } else {
            temp.assign(stage_bytes(total), 0);
            stage = temp.data();
        }
        for (uint32_t l = 0; l < n_layers; ++l) {
            const HostLayer& hl = ht.layers[l];
            if (hl.dev.kind != MT_FC && hl.dev.kind != MT_CONV2D) continue;
            uint8_t* w_dst = stage + hl.w_rel;
            if (biases && biases[l]) std::memcpy(stage + hl.b_rel, biases[l], (size_t)hl.dev.N * 4);
            const void* w_src = weights[l];
            std::vector<uint8_t> folded;
            if (bn && bn[l]) {          // fold the normalisation into a copy of the filters and into the staged bias
                const size_t per = (size_t)hl.spec.in_features * hl.dev.ksize * hl.dev.ksize;
                folded.assign((const uint8_t*)weights[l], (const uint8_t*)weights[l] + (size_t)hl.dev.N * per * c->elem_size);
                fold_batchnorm(c->elem_size, folded.data(), (float*)(stage + hl.b_rel), hl.dev.N, per, bn[l], (double)bn_eps);
                w_src = folded.data();
            }
            if (c->elem_size == 2) pack_weights<uint16_t>(hl, w_src, w_dst); else pack_weights<float>(hl, w_src, w_dst);
            // conv_first_kernel's bf16 form multiplies a step's zeros with another step's filters: not with infinite ones
            if (LayerDev& d = ht.layers[l].dev; d.first_rows && c->elem_size == 2 && !all_finite_bf16((const uint16_t*)w_src, (size_t)d.N * hl.spec.in_features * d.ksize * d.ksize))
                d.first_rows = d.first_pool = 0, ht.layers[n_layers > 1 ? 1 : 0].dev.pair_rows = 0;
        }
    }
    auto drop_stage = [&]() { if (c->cache && stage) (void)hipHostFree(stage); };

    // a model with skip connections may need a third or fourth activation buffer in every run slot
    if (!c->host_only && ht.act_buffers > c->act_buffers) {
        const size_t act_bytes = (size_t)c->P_cap * c->S * c->elem_size;
        for (RunSlot& r : c->slots)
            for (uint32_t i = c->act_buffers; i < ht.act_buffers; ++i)
                if (!r.d_act[i] && hipMalloc(&r.d_act[i], act_bytes) != hipSuccess) {
                    (void)hipGetLastError();
                    drop_stage();
                    return fail(c, MT_ENOMEM, "no device memory for activation buffer %u of %zu bytes", i, act_bytes);
                }
        c->act_buffers = ht.act_buffers;
        for (RunSlot& r : c->slots) if (r.d_act[0] == c->d_act[0]) bind_slot(c, r);
    }

    // Registration is synchronous.  In cache mode every run in flight ends first: models may have to
    // give way, and a block that an earlier eviction freed may still be read by a run enqueued before it.
    uint64_t off = 0;
    hipError_t e = hipSuccess;
    const uint64_t stamp = ++c->use_clock;
    if (c->cache && !c->host_only) {
        const hipError_t es = hipDeviceSynchronize();
        if (es != hipSuccess) { drop_stage(); return fail(c, MT_EDEVICE, "device synchronisation failed: %s", hipGetErrorString(es)); }
    }
    if (!make_room(c, total, stamp, nullptr, false, &off, &e)) {
        drop_stage();
        if (e != hipSuccess) return fail(c, MT_EDEVICE, "eviction failed: %s", hipGetErrorString(e));
        return fail(c, MT_ENOMEM, "weight arena exhausted: model needs %llu bytes, %llu of %llu in use",
                    (unsigned long long)total, (unsigned long long)c->arena_used, (unsigned long long)c->cfg.arena_bytes);
    }
    close_plan(c);
    ht.dev.registered = c->plan; ht.dev.covered = first_plan_for(c, ht);
    ht.arena_off = off;
    for (uint32_t l = 0; l < n_layers; ++l) { ht.layers[l].dev.w_off = off + ht.layers[l].w_rel; ht.layers[l].dev.b_off = off + ht.layers[l].b_rel; }
    if (!c->host_only) {
        place_tenant(c, ht, off, stage);
        e = upload_tenant(c, tenant, ht, stage, nullptr, false);
        if (e != hipSuccess) {
            arena_free(c, off, total);
            drop_stage();
            return fail(c, MT_EDEVICE, "upload of tenant %u failed: %s", tenant, hipGetErrorString(e));
        }
    }
    ht.registered = true; ht.resident = true; ht.last_use = stamp;
    ht.stage = c->cache ? stage : nullptr;
    c->tenants[tenant] = ht;
    c->n_registered++;
    note_first_shape(c, ht, 1);
    recompute_bounds(c);
    recompute_pool_fusion(c);
    return MT_OK;
}

mt_status mt_prefetch(mt_ctx* c, const uint32_t* tenants, uint32_t n, void* hip_stream)
{
    if (!c || (!tenants && n)) return MT_EINVAL;
    for (uint32_t i = 0; i < n; ++i)
        if (tenants[i] >= c->cfg.max_tenants || !c->tenants[tenants[i]].registered)
            return fail(c, MT_ENOTFOUND, "tenant %u has no model", tenants[i]);
    const uint64_t stamp = ++c->use_clock;          // everything named here is used "now": none of it gives way to the rest
    bool missing = false;
    for (uint32_t i = 0; i < n; ++i) { c->tenants[tenants[i]].last_use = stamp; missing |= !c->tenants[tenants[i]].resident; }
    if (!missing) return MT_OK;                     // (always the case outside cache mode)
    hipStream_t s = (hipStream_t)hip_stream;
    if (!c->host_only) {
        HIP_TRY(c, hipSetDevice(c->cfg.device));
        // runs in flight keep their weights and tables: the changes below queue up behind them
        for (RunSlot& r : c->slots)
            if (r.used) HIP_TRY(c, hipStreamWaitEvent(s, r.done, 0));
        if (c->static_slot.used) HIP_TRY(c, hipStreamWaitEvent(s, c->static_slot.done, 0));
        if (c->cache_pending && c->cache_stream != s) HIP_TRY(c, hipStreamWaitEvent(s, c->cache_event, 0));
    }
    mt_status result = MT_OK;
    for (uint32_t i = 0; i < n && result == MT_OK; ++i) {
        HostTenant& ht = c->tenants[tenants[i]];
        if (ht.resident) continue;
        uint64_t off = 0;
        hipError_t e = hipSuccess;
        if (!make_room(c, ht.arena_len, stamp, s, true, &off, &e)) {
            result = e != hipSuccess ? fail(c, MT_EDEVICE, "eviction failed: %s", hipGetErrorString(e))
                                     : fail(c, MT_ENOMEM, "the models named do not fit the weight arena together (%llu of %llu bytes in use, tenant %u needs %llu)",
                                            (unsigned long long)c->arena_used, (unsigned long long)c->cfg.arena_bytes, tenants[i], (unsigned long long)ht.arena_len);
            break;
        }
        if (!c->host_only) {
            place_tenant(c, ht, off, ht.stage);
            e = upload_tenant(c, tenants[i], ht, ht.stage, s, true);
            if (e != hipSuccess) {
                arena_free(c, off, ht.arena_len);
                result = fail(c, MT_EDEVICE, "upload of tenant %u failed: %s", tenants[i], hipGetErrorString(e));
                break;
            }
        } else {
            ht.arena_off = off;
        }
        ht.resident = true;
    }
    if (!c->host_only) {                            // also after a failure: part of the changes may be enqueued
        const hipError_t e = hipEventRecord(c->cache_event, s);
        if (e != hipSuccess && result == MT_OK) result = fail(c, MT_EDEVICE, "hipEventRecord failed: %s", hipGetErrorString(e));
        c->cache_pending = true; c->cache_stream = s;
    }
    return result;
}

mt_status mt_unregister_model(mt_ctx* c, uint32_t tenant)
{
    if (!c) return MT_EINVAL;
    if (tenant >= c->cfg.max_tenants || !c->tenants[tenant].registered) return fail(c, MT_ENOTFOUND, "tenant %u has no model", tenant);
    for (const Segment& s : c->pending)
        if (!s.ids && s.tenant == (int32_t)tenant) return fail(c, MT_ESTATE, "tenant %u has pending requests", tenant);
    if (!c->host_only) {
        HIP_TRY(c, hipSetDevice(c->cfg.device));
        HIP_TRY(c, hipDeviceSynchronize());
        HIP_TRY(c, hide_tenant(c, tenant, nullptr, false));
        if (c->tenants[tenant].stage) (void)hipHostFree(c->tenants[tenant].stage);
    }
    close_plan(c);
    if (c->tenants[tenant].resident) arena_free(c, c->tenants[tenant].arena_off, c->tenants[tenant].arena_len);
    note_first_shape(c, c->tenants[tenant], -1);
    c->tenants[tenant] = HostTenant{};
    c->n_registered--;
    recompute_bounds(c);
    recompute_pool_fusion(c);
    return MT_OK;
}

static mt_status push_segment(mt_ctx* c, const Segment& s, uint32_t* first_index)
{
    if ((uint64_t)c->pending_rows + s.n_rows > c->cfg.max_requests)
        return fail(c, MT_EFULL, "%u rows pending, %u more exceed max_requests %u", c->pending_rows, s.n_rows, c->cfg.max_requests);
    Segment seg = s;
    seg.row_begin = c->pending_rows;
    if (first_index) *first_index = c->pending_rows;
    // consecutive submissions of one tenant from one contiguous buffer collapse into one run
    if (!c->pending.empty()) {
        Segment& b = c->pending.back();
        if (!b.ids && !seg.ids && b.tenant == seg.tenant && b.row_stride == seg.row_stride &&
            (const uint8_t*)b.src + (size_t)b.n_rows * b.row_stride * c->elem_size == (const uint8_t*)seg.src) {
            b.n_rows += seg.n_rows; c->pending_rows += seg.n_rows;
            return MT_OK;
        }
    }
    c->pending.push_back(seg);
    c->pending_rows += seg.n_rows;
    return MT_OK;
}

mt_status mt_submit(mt_ctx* c, uint32_t tenant, const void* inputs, uint32_t n_rows, uint32_t* first_index)
{
    if (!c) return MT_EINVAL;
    if (!inputs || n_rows == 0) return fail(c, MT_EINVAL, "null inputs or zero rows");
    if (tenant >= c->cfg.max_tenants || !c->tenants[tenant].registered) return fail(c, MT_ENOTFOUND, "tenant %u has no model", tenant);
    Segment s{};
    s.ids = nullptr; s.src = inputs; s.n_rows = n_rows; s.row_stride = c->tenants[tenant].dev.in_len; s.tenant = (int32_t)tenant;
    return push_segment(c, s, first_index);
}

mt_status mt_submit_batch(mt_ctx* c, const int32_t* tenant_ids, const void* inputs, uint32_t n_rows, uint32_t row_stride,
                          uint32_t* first_index)
{
    if (!c) return MT_EINVAL;
    if (!tenant_ids || !inputs || n_rows == 0 || row_stride == 0) return fail(c, MT_EINVAL, "null buffers, zero rows or zero stride");
    if (row_stride < c->max_in_len)
        return fail(c, MT_EINVAL, "row_stride %u is shorter than the longest registered input (%u)", row_stride, c->max_in_len);
    Segment s{};
    s.ids = tenant_ids; s.src = inputs; s.n_rows = n_rows; s.row_stride = row_stride; s.tenant = -1;
    return push_segment(c, s, first_index);
}

namespace {

__global__ void fill_zero_kernel(uint32_t* p, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// Packed rows a run of R rows can occupy: every tenant with traffic pads its segment to a multiple of 32.
constexpr uint32_t kBigWalkMinK = 256;     // the walking big-tile kernel needs seven stages of 32 (bf16) or 16 (fp32) per tile
// A convolution launch that can write at most this much stores through L2 (store_through): twice what the L2s hold (8 x 4 MiB).  Passes with
// the line at 0 / 32 / 64 / 128 MiB: residual nets, 64 images 642 / 630 / 630 us (on another box 629 / - / 616 / 613), 128 images 1110 / 1103 / 1096,
// 1000 32x32 images through small CNNs 104.6 / 103 / 100.8 / 101.2; with no line 256 images 2090 -> 2106 and 2048 unstrided CNNs 718 -> 737.
constexpr uint64_t kStoreThroughMaxBytes = 64u << 20;
constexpr uint32_t kConvLongK = 1024;      // reductions from here on are worth loader waves when a launch has at most one tile per CU

// Workgroups that share one packed row in the per-row kernels: `per_wg` units of work each, at most 64.
static uint32_t row_slices(uint64_t units, uint32_t per_wg)
{
    return (uint32_t)std::min<uint64_t>(std::max<uint64_t>((units + per_wg - 1) / per_wg, 1), 64);
}
// The same for the image kernels, whose threads take eight units each where there are rows enough to fill the chip
// with such workgroups, down to one where there are not (the max-pool of one 112x112x64 image on 13 workgroups of 2048
// chunks took 29.7 us, on 98 of 256 it takes 10.6, part of which is the loads of a window being in flight together).
static uint32_t image_slices(uint64_t units, uint32_t R)
{
    constexpr uint64_t kThreads = 256, kMostPerThread = 8, kFill = 2048, kMost = 256;
    const uint64_t per_wg = std::min(std::max(units * R / kFill, kThreads) / kThreads, kMostPerThread) * kThreads;
    return (uint32_t)std::min(std::max<uint64_t>((units + per_wg - 1) / per_wg, 1), kMost);
}

uint32_t packed_rows_bound(const mt_ctx* c, uint32_t R)
{
    return (uint32_t)std::min<uint64_t>(c->P_cap, (uint64_t)round_up(R, kBrickRows) + (uint64_t)kBrickRows * std::min(R, c->n_registered));
}

// Carve the buffers of a run of R rows out of the static scratch array.  Returns the bytes needed;
// the slot's pointers are set only when they fit.  The batch descriptors come first, in one block
// that is cleared before the run (descr_words 32-bit words from rs->d_M).
uint64_t carve_static_slot(const mt_ctx* c, uint32_t R, RunSlot* rs, uint32_t* descr_words)
{
    const uint64_t T = c->cfg.max_tenants, P = packed_rows_bound(c, R);
    uint64_t at = 0;
    auto take = [&](uint64_t bytes) { const uint64_t o = at; at += round_up64(bytes, 256); return o; };
    const uint64_t o_M = take(T * 4), o_off = take((T + 1) * 4), o_tb = take((kListKinds * MT_MAX_LAYERS * (T + 1) + 1) * 4);
    const uint64_t descr_end = at;
    const uint64_t o_rt = take((uint64_t)R * 4), o_rr = take((uint64_t)R * 4), o_h = take((uint64_t)kHistEntries * 4);
    const uint64_t o_src = take((uint64_t)R * sizeof(void*)), o_pos = take((uint64_t)R * 4), o_perm = take(P * 4);
    uint64_t o_act[kActBuffers] = {};
    for (uint32_t i = 0; i < c->act_buffers; ++i) o_act[i] = take(P * c->S * c->elem_size);
    const uint64_t o_lg = take(P * c->C_pad * 4);
    if (at <= MT_STATIC_SCRATCH_BYTES) {
        uint8_t* b = c->static_scratch;
        rs->d_M = (uint32_t*)(b + o_M); rs->d_off = (uint32_t*)(b + o_off); rs->d_tile_base = (uint32_t*)(b + o_tb);
        rs->d_row_tenant = (int32_t*)(b + o_rt); rs->d_row_rank = (uint32_t*)(b + o_rr); rs->d_hist_g = (uint32_t*)(b + o_h);
        rs->d_row_src = (const void**)(b + o_src); rs->d_pos_of = (int32_t*)(b + o_pos); rs->d_perm = (int32_t*)(b + o_perm);
        for (uint32_t i = 0; i < (uint32_t)kActBuffers; ++i) rs->d_act[i] = i < c->act_buffers ? b + o_act[i] : nullptr;
        rs->d_logits = (float*)(b + o_lg);
        *descr_words = (uint32_t)(descr_end / 4);
    }
    return at;
}

// The pending requests per tenant, if every submission named its tenant and some model has convolutions (which are
// planned by them); else null.  In the order of first submission.
const std::vector<NamedRows>* count_named(mt_ctx* c)
{
    bool convs = false;
    for (uint32_t g = 0; g < MT_MAX_LAYERS / kLayerGroup; ++g) convs = convs || ((c->list_mask[g] >> kLayerGroup) & ((1u << kLayerGroup) - 1));
    for (const Segment& s : c->pending) convs = convs && !s.ids;
    if (!convs) return nullptr;
    c->named.clear();
    for (const Segment& s : c->pending) {
        uint32_t& at = c->named_at[(uint32_t)s.tenant];
        if (!at) { c->named.push_back({(uint32_t)s.tenant, 0}); at = (uint32_t)c->named.size(); }
        c->named[at - 1].rows += s.n_rows;
    }
    for (const NamedRows& r : c->named) c->named_at[r.tenant] = 0;
    return &c->named;
}

mt_status run_impl(mt_ctx* c, void* hip_stream, const mt_outputs* out, uint32_t* n_rows, bool use_static);

}  // namespace

mt_status mt_run(mt_ctx* c, void* hip_stream, const mt_outputs* out, uint32_t* n_rows)
{
    return run_impl(c, hip_stream, out, n_rows, false);
}

mt_status mt_run_static(mt_ctx* c, void* hip_stream, const mt_outputs* out, uint32_t* n_rows)
{
    return run_impl(c, hip_stream, out, n_rows, true);
}

namespace {

mt_status run_impl(mt_ctx* c, void* hip_stream, const mt_outputs* out, uint32_t* n_rows, bool use_static)
{
    if (!c) return MT_EINVAL;
    if (n_rows) *n_rows = 0;
    if (c->host_only) return fail(c, MT_ESTATE, "host-only context cannot run");
    const uint32_t R = c->pending_rows;
    if (R == 0) { c->last_run_rows = 0; c->last_run_launches = 0; return MT_OK; }
    if (!out || !out->labels) return fail(c, MT_EINVAL, "null outputs");
    if (out->capacity < R) return fail(c, MT_EINVAL, "outputs hold %u rows, %u pending", out->capacity, R);
    if ((out->probs || out->logits) && out->row_stride < c->cfg.max_classes)
        return fail(c, MT_EINVAL, "row_stride %u is below max_classes %u", out->row_stride, c->cfg.max_classes);
    hipStream_t s = (hipStream_t)hip_stream;
    HIP_TRY(c, hipSetDevice(c->cfg.device));

    // Model cache: the tenants of per-tenant submissions are made resident here (the host knows
    // them); tenants that appear only in device-resident id arrays must have been prefetched.
    // A residency change enqueued on another stream comes first.
    if (c->cache) {
        std::vector<uint32_t> named;
        for (const Segment& sg : c->pending)
            if (!sg.ids && (named.empty() || named.back() != (uint32_t)sg.tenant)) named.push_back((uint32_t)sg.tenant);
        std::sort(named.begin(), named.end());
        named.erase(std::unique(named.begin(), named.end()), named.end());
        if (!named.empty()) { const mt_status st = mt_prefetch(c, named.data(), (uint32_t)named.size(), hip_stream); if (st != MT_OK) return st; }
        if (c->cache_pending && c->cache_stream != s) HIP_TRY(c, hipStreamWaitEvent(s, c->cache_event, 0));
    }
    // the run's slot of device scratch; a stream other than the one that used it last waits for that run
    // (the slot this stream used last, so that runs on one stream keep their buffers and never wait
    // across streams; else a slot nobody has used; else the one used longest ago)
    RunSlot* pick = nullptr;
    uint32_t static_descr_words = 0;
    if (use_static) {
        // the run's buffers come out of the static array, sized for this run; nothing is allocated
        const uint64_t need = carve_static_slot(c, R, &c->static_slot, &static_descr_words);
        if (need > MT_STATIC_SCRATCH_BYTES)
            return fail(c, MT_EINVAL, "a run of %u rows needs %llu bytes of scratch in this context, the static array holds %u",
                        R, (unsigned long long)need, (unsigned)MT_STATIC_SCRATCH_BYTES);
        pick = &c->static_slot;
    }
    if (!pick) for (RunSlot& r : c->slots) if (r.used && r.stream == s) { pick = &r; break; }
    if (!pick) for (RunSlot& r : c->slots) if (!r.used) { pick = &r; break; }
    if (!pick) { pick = &c->slots[0]; for (RunSlot& r : c->slots) if (r.last_run < pick->last_run) pick = &r; }
    RunSlot& rs = *pick;
    // A run of one submission carries its segment in the kernel arguments; only runs of several
    // submissions put the table into one of the pinned slots, which stays busy until the run is over.
    // The host never waits for one: when the GPU is still reading all of them the call is refused.
    const uint32_t n_segs = (uint32_t)c->pending.size();
    uint32_t slot = 0;
    if (n_segs > 1) {
        bool found = false;
        for (uint32_t i = 0; i < kSegSlots && !found; ++i) {
            const uint32_t cand = (uint32_t)((c->run_count + i) % kSegSlots);
            if (c->seg_busy[cand]) {
                const hipError_t q = hipEventQuery(c->seg_event[cand]);
                if (q == hipErrorNotReady) continue;
                if (q != hipSuccess) return fail(c, MT_EDEVICE, "hipEventQuery: %s", hipGetErrorString(q));
                c->seg_busy[cand] = false;
            }
            slot = cand; found = true;
        }
        if (!found) return fail(c, MT_EFULL, "%u runs of several submissions are still in flight; call again later", kSegSlots);
        std::memcpy(c->h_segs[slot], c->pending.data(), c->pending.size() * sizeof(Segment));
    }
    if (rs.used && rs.stream != s) HIP_TRY(c, hipStreamWaitEvent(s, rs.done, 0));
    bind_slot(c, rs);
    const uint32_t T = c->cfg.max_tenants;
    uint32_t launches = 0;

    // Big tiles are for runs that are compute bound as a whole: enough rows, and more flops per
    // byte of registered weights than the chip's ridge point.  Weight-streaming mixes keep every
    // tenant in the streaming kernel (no second launch per layer, layer 0 reads submitted rows).
    const double run_flops = 2.0 * R * (c->n_registered ? c->sum_macs / c->n_registered : 0.0);
    const bool big_enabled = R >= (uint32_t)kBigMinBatch && run_flops >= kRidgeFlopsPerByte * (double)c->arena_used;
    const bool split_k = run_split_k(c, R);
    const std::vector<NamedRows>* named = count_named(c);
    BatchArgs b{};
    b.segs = c->d_segs[slot]; b.n_segs = n_segs; b.R = R; b.T = T; b.n_layer_slots = c->n_layer_slots;
    b.first = c->pending[0]; b.row_src = c->d_row_src; b.elem_size = c->elem_size;
    b.tenants = c->d_tenants; b.facts = c->d_facts; b.served = (unsigned long long*)c->d_served;
    {   // large batches are ranked by a kernel of their own, where its per-workgroup histograms fit the batcher's LDS
        uint32_t Tp = 64;
        while (Tp < T) Tp <<= 1;
        const uint32_t groups = (R + kRankRows - 1) / kRankRows;
        const bool spread = R >= (uint32_t)kRankMinRows && T <= (uint32_t)kRankMaxTenants && (uint64_t)groups * Tp <= (uint64_t)kHistEntries;
        b.n_rank_groups = spread ? groups : 0; b.hist_g = c->d_hist_g;
    }
    b.row_tenant = c->d_row_tenant; b.row_rank = c->d_row_rank; b.pos_of = c->d_pos_of; b.perm = c->d_perm;
    b.M = c->d_M; b.off = c->d_off; b.tile_base = c->d_tile_base; b.big_layers = c->d_tile_base + (size_t)kListKinds * MT_MAX_LAYERS * (T + 1); b.fc_split_k = split_k;
    for (uint32_t g = 0; g < MT_MAX_LAYERS / kLayerGroup; ++g)
        b.list_mask[g] = big_enabled ? c->list_mask[g] : c->list_mask[g] & ((1u << (2 * kLayerGroup)) - 1);   // no big-tile lists to build
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess) { (void)hipGetLastError(); capture = hipStreamCaptureStatusNone; }
    const bool captured = capture != hipStreamCaptureStatusNone;
    b.big_enabled = big_enabled; b.big_min_tiles = c->big_min_tiles; b.plan = c->plan; b.captured = captured;
    if (captured) {
        c->used.act_buffers = c->used.any ? std::min(c->used.act_buffers, c->act_buffers) : c->act_buffers;
        c->used.any = true;
    }
    ConvPlan convs[MT_MAX_LAYERS]{};
    for (uint32_t l = 0; l < c->n_layer_slots; ++l) convs[l] = plan_conv(c, l, R, named, captured);
    if (const ConvPlan& first = convs[0]; first.first_cap) {     // its list is made apart from the others; a second convolution done with it has none
        b.first_cap = first.first_cap; b.first_pair = first.pair_mid != 0;
        b.list_mask[0] &= ~((first.pair_mid ? 3u : 1u) << kLayerGroup);
        if (captured) c->used.first = true;
    }
    for (uint32_t l = 0; l < c->n_layer_slots; ++l) {
        if (!convs[l].split) continue;
        b.conv_split[l / 32] |= 1u << l % 32;
        if (captured && c->conv_quad[l] && (c->max_conv_k[l] * c->elem_size + 31) / 32 > kSplitFewSteps) c->used.chunk_layers |= 1ull << l;
    }
    const OutPtrs outp{out->labels, out->probs, out->logits, out->n_classes, out->row_stride};
    b.out = outp;
    // A last layer of at most 32 classes is one column block: its FC tiles finish their rows themselves; and one of at most 128 classes is one tile of four column blocks,
    // or (the K-split shape of small runs) one that takes them in turn.
    const bool whole = run_whole(c, split_k, captured);
    const uint32_t fuse_head_max = fused_head_classes(c, split_k, whole);
    const bool fuse_head = fuse_head_max > 0 && c->min_reg_classes <= fuse_head_max;
    b.fc_whole = whole;
    const uint32_t head_min_classes = fuse_head ? fuse_head_max + 1 : 0;
    const bool out_vec_ok = out->row_stride % 4 == 0 && ((uintptr_t)out->probs & 15) == 0 && ((uintptr_t)out->logits & 15) == 0;
    if (c->profiling) for (uint32_t i = 0; i < kProfSlots; ++i) c->prof_used[i] = false;
    // From here on a failure may leave part of the run enqueued: the launches sit in a body of their
    // own, and the bookkeeping behind it (events, slot, pending list) is closed whatever it returns.
    auto enqueue = [&]() -> mt_status {
#define TIMED(slot, call)                                                                   \
    do {                                                                                    \
        if (c->profiling) HIP_TRY(c, hipEventRecord(c->prof_events[2 * (slot)], s));        \
        HIP_TRY(c, call); ++launches;                                                       \
        if (c->profiling) { HIP_TRY(c, hipEventRecord(c->prof_events[2 * (slot) + 1], s)); c->prof_used[slot] = true; c->prof_last = (slot); } \
    } while (0)
    if (use_static) {
        // the array keeps what the last run on this GPU left: the descriptors start from zero (a fill
        // kernel, not a memset node, so that the sequence can be captured into a graph)
        hipLaunchKernelGGL(fill_zero_kernel, dim3((static_descr_words + 255) / 256), dim3(256), 0, s, rs.d_M, static_descr_words);
        HIP_TRY(c, hipGetLastError()); ++launches;
    }
    // The FC kernel of layer 0 reads the submitted rows itself (first_rows); otherwise (and for CNN models, whose images are
    // channel-padded) a gather pass stages the inputs first.
    // The big-tile kernel reads bricks only (it was measured slower when it gathers rows itself,
    // since every row is then fetched in 16-byte pieces by each of a layer's column tiles):
    // whenever a tenant could reach it at layer 0, stage.
    const bool big_possible = big_enabled && c->max_nt[2][0] > 0 && tile_bound(c, 2, 0, R) >= c->big_min_tiles;
    const int rows = first_rows(c, R, split_k, big_possible, true);
    const bool fuse_gather = rows != kRowsStaged;
    // Every workgroup of fc_entry_kernel looks up for itself which tenants there are, so it goes by those registered now.  What is
    // captured goes on to serve models registered later, which the one workgroup of the batcher can look up.
    const int entry = n_segs == 1 && fuse_gather && !captured ? run_entry(c, R, split_k) : kEntryNone;
    if (entry) {                           // (the time of the whole run starts where the batcher's would)
        if (c->profiling) HIP_TRY(c, hipEventRecord(c->prof_events[2 * kProfBatcher], s));
    } else {
        TIMED(kProfBatcher, launch_batcher(b, s));
        if (b.n_rank_groups) launches += 2;
    }
    // packed rows: every tenant with traffic pads its segment to a multiple of 32
    const uint32_t P = packed_rows_bound(c, R);
    {
        GatherArgs g{};
        g.row_src = c->d_row_src; g.P = P; g.tenants = c->d_tenants; g.layers = c->d_layers;
        g.perm = c->d_perm; g.off = c->d_off; g.M = c->d_M; g.T = T; g.act = c->d_act[0]; g.S = c->S; g.elem_size = c->elem_size; g.zeros = c->d_zeros;
        // workgroups per block of 32 rows: each takes ~64 KiB of it, so that long rows have enough loads in flight
        const uint32_t gs = row_slices((uint64_t)c->max_in_len * c->elem_size * kBrickRows, 65536);      // c5: 146 -> 133 us with four
        if (c->any_fc_first && !fuse_gather) TIMED(kProfGather, launch_gather(g, gs, s));
        if (c->any_conv_first && !c->first_on) TIMED(kProfGatherImg, launch_gather_image(g, image_slices(c->max_image_pixels / 2, R), s));       // in pairs of pixels
    }

    ActBufs bufs{};                        // every layer names the buffers it reads and writes (LayerDev::in_buf ...)
    for (int i = 0; i < kActBuffers; ++i) bufs.p[i] = c->d_act[i];
    for (uint32_t l = 0; l < c->n_layer_slots; ++l) {
        // a pooling index that the convolutions before it have already served: nothing runs, the
        // pooled activation is where the pooling layer would have written it
        if (l > 0 && c->pool_fused[l - 1]) continue;
        for (int kind = 0; kind < kListKinds; ++kind) {
            const ConvPlan conv = kind == 1 ? convs[l] : ConvPlan{};
            const uint64_t grid = kind == 1 ? conv.tiles : tile_bound(c, kind, l, R, split_k, big_enabled);
            if (grid == 0 || (kind == 2 && (!big_enabled || grid < c->big_min_tiles))) continue;   // no big tiles possible: the batcher made none
            GemmArgs ga{};
            ga.tile_base = c->d_tile_base + ((size_t)kind * MT_MAX_LAYERS + l) * (T + 1);
            ga.T = T; ga.layer = l; ga.fc_split_k = split_k; ga.fc_whole = kind == 0 && whole && c->wide_last[l]; ga.big_layers = b.big_layers;
            ga.gather = kind == 0 && l == 0 ? rows : kRowsStaged; ga.perm = c->d_perm; ga.row_src = c->d_row_src;
            ga.fuse_head = fuse_head; ga.fuse_head_max = fuse_head_max; ga.out_vec_ok = out_vec_ok; ga.out = outp; ga.pool = kind == 1 && c->pool_fused[l];
            ga.store_through = kind == 1 && R * c->max_conv_work[l] * kBrickRows * c->elem_size <= kStoreThroughMaxBytes;
            ga.layers = c->d_layers; ga.off = c->d_off; ga.M = c->d_M; ga.act = bufs; ga.arena = c->d_arena;
            ga.logits = c->d_logits; ga.S = c->S; ga.C_pad = c->C_pad; ga.zeros = c->d_zeros;
            // a launch holds fewer than 2^32 work items; cannot be exceeded by activations that fit the device's memory
            if (grid > kMaxLaunchItems / (conv.split ? 1024 : kind == 2 || (conv.first_cap && c->first_pool) ? 512 : 256))
                return fail(c, MT_EUNSUPPORTED, "layer %u: %llu tiles exceed one launch", l, (unsigned long long)grid);
            const uint32_t g32 = (uint32_t)grid;
            ga.first_cap = conv.first_cap;
            if (kind == 0 && l == 0 && entry) TIMED(kProfFc + l, launch_fc_entry(ga, b, c->cfg.dtype, entry == kEntryWide, g32, s));
            else if (kind == 0) TIMED(kProfFc + l, launch_fc(ga, c->cfg.dtype, split_k || c->max_fc_cols[l] <= 2 * (uint32_t)kBrickRows, g32, s));
            else if (conv.pair_mid) TIMED(kProfConv + l, launch_conv_pair(ga, c->cfg.dtype, c->pair_blocks, conv.first_frame, conv.pair_mid, g32, s));
            else if (conv.first_cap) TIMED(kProfConv + l, launch_conv_first(ga, c->cfg.dtype, c->first_max_ks, c->first_pool, c->first_plain, conv.first_frame, g32, s));
            else if (conv.split) TIMED(kProfConv + l, launch_conv_split(ga, c->cfg.dtype, (c->max_conv_k[l] * c->elem_size + 31) / 32, c->conv_quad[l], g32, s));
            else if (kind == 1) TIMED(kProfConv + l, launch_conv(ga, c->cfg.dtype, c->max_conv_cb[l], c->conv_quad[l],
                                                                    conv.frames ? c->conv_img_lds[l] : 0, c->conv_img_two[l] == 1,
                                                                    !c->no_conv_loaders && c->min_conv_k[l] >= kConvLongK,
                                                                    c->conv_uniform[l] && !c->no_conv_uniform && (uint64_t)c->cfg.max_requests * c->S * c->elem_size < (1ull << 31), g32, s));
            else TIMED(kProfBig + l, launch_fc_big(ga, c->cfg.dtype, g32, (c->big_walk && c->min_fc_k[l] >= kBigWalkMinK) ? c->n_cus : 0, s));
        }
        if (c->has_gap[l]) {
            GapArgs pa{};
            pa.layer = l; pa.P = P; pa.layers = c->d_layers; pa.tenants = c->d_tenants;
            pa.off = c->d_off; pa.M = c->d_M; pa.T = T; pa.act = bufs; pa.S = c->S;
            pa.elem_size = c->elem_size;
            TIMED(kProfGap + l, launch_gap(pa, c->gap_chunks[l], s));
        }
        if (c->has_image_ops[l]) {         // max-pooling and residual additions of this layer index
            GapArgs pa{};
            pa.layer = l; pa.P = P; pa.layers = c->d_layers; pa.tenants = c->d_tenants;
            pa.off = c->d_off; pa.M = c->d_M; pa.T = T; pa.act = bufs; pa.S = c->S;
            pa.elem_size = c->elem_size; pa.first_pooled = l == 1 && c->first_on;
            TIMED(kProfImageOps + l, launch_image_ops(pa, image_slices(c->image_op_fill[l] * c->elem_size / 16, R), s));   // in 16-byte chunks
        }
    }

    if (!fuse_head || c->max_reg_classes > fuse_head_max) {
        HeadArgs h{};
        h.R = R; h.tenants = c->d_tenants; h.row_tenant = c->d_row_tenant; h.pos_of = c->d_pos_of; h.logits = c->d_logits;
        h.C_pad = c->C_pad; h.out = outp; h.min_classes = head_min_classes;
        h.vec_ok = out_vec_ok;
        TIMED(kProfHead, launch_head(h, s));
    }
#undef TIMED
    return MT_OK;
    };
    mt_status st = enqueue();
    if (st != MT_OK && launches == 0) return st;         // nothing was enqueued: the pending list is kept
    c->prof_valid = c->profiling && st == MT_OK;
    if (n_segs > 1) {
        const hipError_t e = hipEventRecord(c->seg_event[slot], s);
        if (e != hipSuccess && st == MT_OK) st = fail(c, MT_EDEVICE, "hipEventRecord: %s", hipGetErrorString(e));
        c->seg_busy[slot] = true;
    }
    {
        const hipError_t e = hipEventRecord(rs.done, s);
        if (e != hipSuccess && st == MT_OK) st = fail(c, MT_EDEVICE, "hipEventRecord: %s", hipGetErrorString(e));
    }
    rs.used = true; rs.stream = s; rs.last_run = c->run_count;
    c->run_count++;
    c->last_stream = s;
    c->pending.clear();
    c->pending_rows = 0;
    c->last_run_rows = st == MT_OK ? R : 0; c->last_run_launches = launches;
    if (n_rows && st == MT_OK) *n_rows = R;
    return st;
}

}  // namespace

mt_status mt_last_counts(mt_ctx* c, uint32_t* counts)
{
    if (!c || !counts) return MT_EINVAL;
    if (c->host_only) return fail(c, MT_ESTATE, "host-only context");
    HIP_TRY(c, hipSetDevice(c->cfg.device));
    HIP_TRY(c, hipStreamSynchronize(c->last_stream));
    HIP_TRY(c, hipMemcpy(counts, c->d_M, (size_t)c->cfg.max_tenants * 4, hipMemcpyDeviceToHost));
    return MT_OK;
}

// ---- accounting and cost prediction (paper section 3.2) -------------------------------------
namespace {

// Algorithmic cost of one request of a model, from its description alone.
void request_cost(const mt_ctx* c, const HostTenant& ht, uint64_t* flops, uint64_t* weight_bytes, uint64_t* io_bytes)
{
    const uint64_t es = c->elem_size;
    *flops = *weight_bytes = *io_bytes = 0;
    for (uint32_t l = 0; l < ht.n_layers; ++l) {
        const mt_layer_spec& s = ht.layers[l].spec;
        const LayerDev& d = ht.layers[l].dev;
        uint64_t in_len = 0;
        if (s.kind == MT_FC) {
            *flops += 2ull * s.in_features * s.out_features;
            *weight_bytes += (uint64_t)s.in_features * s.out_features * es + (uint64_t)s.out_features * 4;
            in_len = s.in_features;
        } else if (s.kind == MT_CONV2D) {
            *flops += 2ull * d.rows_per_req * s.kh * s.kw * s.in_features * s.out_features;
            *weight_bytes += (uint64_t)s.kh * s.kw * s.in_features * s.out_features * es + (uint64_t)s.out_features * 4;
            in_len = (uint64_t)s.in_h * s.in_w * s.in_features;
        } else {
            in_len = (uint64_t)s.in_h * s.in_w * s.in_features;
        }
        if (l == 0) *io_bytes += in_len * es;
        if (l + 1 < ht.n_layers) *io_bytes += 2ull * d.out_len * es;
        else *io_bytes += 2ull * d.out_len * 4 + 4;
    }
}

// Per-kernel time model, microseconds and megabytes; constants fitted on one MI355X (the
// measurements are in the design notes).  A streaming FC launch costs a fixed part, its bytes
// from HBM (weights of the active tenants) and the bytes its tiles re-read through L2 (weight
// panels re-read by further row tiles, activation rows re-read by every column group; three
// times that when layer 0 gathers the submitted rows in 16-byte pieces); it cannot be shorter
// than the chain of dependent loads through K of one tile.
// Weights that fit the 256 MB memory-side cache and are read by every run stream faster than
// weights that come from HBM every time (steady serving of the same tenants is assumed).
constexpr double kUsLaunchGap = 3.0;
constexpr double kUsFcFixed = 3.7, kUsPerMbCached = 0.132, kUsPerMbHbm = 0.18, kCachedMb = 240.0;
constexpr double kUsPerMbL2 = 0.056, kUsFcChainFixed = 4.0, kUsPerKStep = 0.12;
constexpr double kUsBigFixed = 4.0, kUsBigTileFixed = 7.0, kUsBigTilePer4096 = 108.0;
constexpr double kUsConvFixed = 5.0, kConvMbPerUs = 4.0, kConvMflopPerUs = 0.5e3;      // 4.0 TB/s, 0.5 PFLOP/s
constexpr double kUsConvFramePerKStep = 0.095, kConvFrameMflopPerUs = 0.6e3;   // the same for layer indices served from LDS frames: filter bricks are the only loads in the K loop
constexpr double kUsConvFirstFixed = 8.0, kConvFirstMbPerUs = 5.2, kConvFirstMflopPerUs = 0.38e3;     // first convolutions on the submitted images, by the multiplications that they need
constexpr double kUsConvSplitFixed = 1.0, kUsConvSplitPerKStep = 0.034;     // launches whose tiles split K among their waves: per k-step of a tile, one tile per compute unit at a time
constexpr double kUsConvPerKStep = 0.21;     // a convolution tile's walk through K, per k-step of 32 bytes per pixel: a launch lasts at least as long as its longest tile
constexpr double kUsBatcher = 7.0, kUsBatcherPer1024 = 1.1;     // kernel trace: 7.0 us at 64 rows, 9.2 at 2048, 11.3 at 4096
constexpr double kUsEntry = 3.0;             // what the segmentation costs a small run's first layer
constexpr double kUsEntryWideSaves = 3.7;    // what it saves where tiles of any kind do it: of the batcher's launch and the gap behind it (measured 2.9 to 4.7, beside run_entry)
constexpr double kUsSmallFixed = 3.0, kCopyMbPerUs = 3.7, kHeadMbPerUs = 5.7, kUsHeadPerRow = 0.0008;
constexpr double kComputeUnits = 256.0;
constexpr double kUploadBytesPerMs = 55e6, kUsUploadFixed = 20.0;     // pinned host memory to HBM over the host link: 55 GB/s measured

}  // namespace

mt_status mt_tenant_account_get(mt_ctx* c, uint32_t tenant, mt_tenant_account* out)
{
    if (!c || !out) return MT_EINVAL;
    if (tenant >= c->cfg.max_tenants) return fail(c, MT_EINVAL, "tenant %u is outside 0..%u", tenant, c->cfg.max_tenants - 1);
    if (!c->tenants[tenant].registered) return fail(c, MT_ENOTFOUND, "tenant %u has no model", tenant);
    *out = mt_tenant_account{};
    request_cost(c, c->tenants[tenant], &out->flops_per_request, &out->weight_bytes, &out->io_bytes_per_request);
    out->resident = c->tenants[tenant].resident;
    out->arena_bytes = c->tenants[tenant].arena_len;
    if (!c->host_only) {
        uint64_t counters[2] = {0, 0};
        HIP_TRY(c, hipSetDevice(c->cfg.device));
        HIP_TRY(c, hipDeviceSynchronize());
        HIP_TRY(c, hipMemcpy(counters, c->d_served + 2 * (size_t)tenant, sizeof counters, hipMemcpyDeviceToHost));
        out->requests = counters[0]; out->runs = counters[1];
    }
    return MT_OK;
}

namespace {

// mt_estimate_run.  *plan: a number that grows with the requests and differs wherever the run's launches or the kernels that serve it do: between counts of the
// same number, the larger take longer.
mt_status estimate_run(mt_ctx* c, const uint32_t* counts, mt_run_estimate* out, uint64_t* plan)
{
    *out = mt_run_estimate{};
    *plan = 0;
    const uint32_t T = c->cfg.max_tenants;
    const double es = c->elem_size, MB = 1e6;
    uint64_t R = 0;
    for (uint32_t t = 0; t < T; ++t) {
        if (!counts[t]) continue;
        if (!c->tenants[t].registered) return fail(c, MT_ENOTFOUND, "tenant %u has no model", t);
        R += counts[t];
        uint64_t f, wb, io;
        request_cost(c, c->tenants[t], &f, &wb, &io);
        out->flops += (double)f * counts[t];
        out->hbm_bytes += (double)wb + (double)io * counts[t];
    }
    if (R > c->cfg.max_requests) return fail(c, MT_EINVAL, "%llu rows exceed max_requests %u", (unsigned long long)R, c->cfg.max_requests);
    out->rows = (uint32_t)R;
    if (R == 0) return MT_OK;

    // the same decisions as mt_run and the batcher take
    const double run_flops = 2.0 * R * (c->n_registered ? c->sum_macs / c->n_registered : 0.0);
    const bool big_enabled = R >= (uint64_t)kBigMinBatch && run_flops >= kRidgeFlopsPerByte * (double)c->arena_used;
    const bool big_possible = big_enabled && c->max_nt[2][0] > 0 && tile_bound(c, 2, 0, R) >= c->big_min_tiles;
    const bool split_k = run_split_k(c, R), fuse_gather = first_rows(c, R, split_k, big_possible, c->pending_rows == R) != kRowsStaged;
    const uint32_t fuse_head_max = fused_head_classes(c, split_k, run_whole(c, split_k, false));
    const bool fuse_head = fuse_head_max > 0 && c->min_reg_classes <= fuse_head_max;
    uint32_t Tp = 64;
    while (Tp < T) Tp <<= 1;
    const uint64_t groups_r = (R + kRankRows - 1) / kRankRows;
    const bool spread = R >= (uint64_t)kRankMinRows && T <= (uint32_t)kRankMaxTenants && groups_r * Tp <= (uint64_t)kHistEntries;

    double weights_mb = 0.0;                 // weights this run reads, all layers
    for (uint32_t t = 0; t < T; ++t) {
        if (!counts[t]) continue;
        uint64_t f, wb, io;
        request_cost(c, c->tenants[t], &f, &wb, &io);
        weights_mb += wb / MB;
    }
    // (each of these turns once as R grows, those that go by the tiles' shape once in either shape)
    *plan = (split_k ? 0u : 1u << 20) + (first_rows(c, R, split_k, big_possible, false) == kRowsStaged) + big_enabled + (R >= (uint64_t)kRankMinRows) + (R >= (uint64_t)kRankMinRows && !spread) +
            (R > kEntryMaxRows) + (R >= kEntryWideMin) + (R > kEntryWideRows) + (tile_bound(c, 0, 0, R, split_k) > kEntryWideTilesPerCu * c->n_cus);

    const double us_per_mb = weights_mb <= kCachedMb ? kUsPerMbCached : kUsPerMbHbm;
    double us = 0.0;
    uint32_t launches = 0;
    auto launch = [&](double t) { us += t + (launches ? kUsLaunchGap : 0.0); ++launches; };
    // one submission, unless these are the requests that are pending in several
    const bool one_submission = c->pending.size() <= 1 || c->pending_rows != R;
    const double batcher_us = kUsBatcher + kUsBatcherPer1024 * R / 1024.0;
    const int entry = one_submission && fuse_gather ? run_entry(c, R, split_k) : kEntryNone;
    if (entry == kEntryNarrow) us += kUsEntry;                             // done by the first layer's launch
    else if (entry == kEntryWide) us += batcher_us + kUsLaunchGap - kUsEntryWideSaves;
    else if (spread) { launch(20.0 + 0.15 * R / 1024.0); launches += 2; }       // ranking, scan, placement
    else launch(batcher_us);

    double fc_in_mb = 0.0, img_in_mb = 0.0, img_out_mb = 0.0;
    for (uint32_t t = 0; t < T; ++t) {
        if (!counts[t]) continue;
        const HostTenant& ht = c->tenants[t];
        if (ht.dev.in_layout == kLayoutBricks) fc_in_mb += counts[t] * (double)ht.dev.in_len * es / MB;
        else { img_in_mb += counts[t] * (double)ht.dev.in_len * es / MB; img_out_mb += counts[t] * (double)ht.dev.in_fill * es / MB; }
    }
    if (c->any_fc_first && !fuse_gather) launch(kUsSmallFixed + 2.0 * fc_in_mb / kCopyMbPerUs);
    if (c->any_conv_first && !c->first_on) launch(kUsSmallFixed + (img_in_mb + img_out_mb) / kCopyMbPerUs);

    for (uint32_t l = 0; l < c->n_layer_slots; ++l) {
        if (l > 0 && c->pool_fused[l - 1]) continue;           // pooled by the convolutions of the index before
        // which tenants take big tiles at this layer index (the batcher's rule)
        uint64_t big_tiles = 0;
        if (big_enabled && c->max_nt[2][l] > 0)
            for (uint32_t t = 0; t < T; ++t) {
                if (!counts[t] || l >= c->tenants[t].n_layers) continue;
                const LayerDev& d = c->tenants[t].layers[l].dev;
                if (d.kind == MT_FC && fc_is_big(counts[t], d.N_pad))
                    big_tiles += (uint64_t)((big_rows(counts[t]) + kBigTile - 1) / kBigTile) * ((d.N_pad + kBigTile - 1) / kBigTile);
            }
        const bool big_layer = big_tiles >= c->big_min_tiles;
        *plan += big_layer + (big_enabled && tile_bound(c, 2, l, R) >= c->big_min_tiles);
        double w_mb = 0.0, l2_mb = 0.0, chain = 0.0, big_us = 0.0, conv_mb = 0.0, conv_mflop = 0.0, gap_mb = 0.0, ops_mb = 0.0;
        double big_rounds_k = 0.0, conv_chain = 0.0, first_mb = 0.0, first_mflop = 0.0;
        const ConvPlan conv_plan = plan_conv(c, l, R, nullptr);                                      // the launch decision of run_impl where the tenants stand in an id array
        const bool conv_frames = conv_plan.frames;
        *plan += !conv_plan.split;
        double split_steps = 0.0, split_longest = 0.0;
        for (uint32_t t = 0; t < T; ++t) {
            if (!counts[t] || l >= c->tenants[t].n_layers) continue;
            const LayerDev& d = c->tenants[t].layers[l].dev;
            const double M = counts[t];
            if (d.kind == MT_FC) {
                const bool big = big_layer && fc_is_big(counts[t], d.N_pad);
                const uint32_t Mb = big ? big_rows(counts[t]) : 0, Ms = counts[t] - Mb;
                if (big) big_rounds_k += (double)((Mb + kBigTile - 1) / kBigTile) * ((d.N_pad + kBigTile - 1) / kBigTile) * d.K;
                if (Ms) {
                    const uint32_t groups = fc_groups(d.N_pad, split_k), trows = fc_tile_rows(d.N_pad, split_k);
                    const double panel_mb = (double)d.N_pad * d.K * es / MB / groups;
                    const double row_tiles = (Ms + trows - 1) / trows;
                    const double act_mb = (double)Ms * d.K * es / MB;
                    w_mb += panel_mb * groups;
                    l2_mb += panel_mb * groups * (row_tiles - 1) + act_mb * groups * ((l == 0 && fuse_gather) ? 3.0 : 1.0);
                    const uint32_t nblk = d.N_pad / kBrickRows, split = split_k ? 1u : (nblk >= 3 ? 4u : nblk);
                    const double k_steps = d.K * es / 32.0 / (4 / split);       // bricks one wave walks (the waves split K when split < 4)
                    chain = std::max(chain, kUsFcChainFixed + kUsPerKStep * k_steps);
                }
            } else if (l == 1 && c->pair_on && d.pair_rows) {
                // done with the convolution in front of it
            } else if (d.kind == MT_CONV2D) {
                const double out_elems = (c->pool_fused[l] ? d.N : d.out_len) + (d.fuse_add ? d.out_len : 0);      // pooled on the way out; the other operand of an addition done here
                conv_mb += (M * ((double)d.in_h * d.in_w * d.cin + out_elems) * es + (double)d.N_pad * d.K * es) / MB;
                conv_mflop += 2.0 * M * d.rows_per_req * d.k_valid * d.N / 1e6;
                if (conv_plan.first_cap) {
                    const LayerDev& last = d.first_pool || c->pair_on ? c->tenants[t].layers[1].dev : d;
                    first_mb += (M * ((double)d.in_h * d.in_w * d.first_cin + last.out_len) * es + (double)d.N_pad * d.K * es) / MB;
                    if (c->pair_on) first_mflop += 2.0 * M * last.rows_per_req * last.k_valid * last.N / 1e6;
                    first_mflop += 2.0 * M * d.rows_per_req * d.ksize * d.ksize * d.first_cin * d.N / 1e6;
                }
                const double k_steps = std::ceil(d.k_valid * es / 32.0);
                split_longest = std::max(split_longest, k_steps);
                split_steps += std::ceil(M * d.rows_per_req / kBrickRows) * (d.N_pad / kBrickRows) * k_steps;
                conv_chain = std::max(conv_chain, (conv_frames ? kUsConvFramePerKStep : kUsConvPerKStep) * d.k_valid * es / 32.0);
            } else if (d.kind == MT_GAP) {
                gap_mb += M * ((double)d.in_h * d.in_w * d.cin + d.out_len) * es / MB;
            } else if (l == 1 && c->first_on && c->tenants[t].layers[0].dev.first_pool) {
                // done with the convolution in front of it
            } else if (d.kind == MT_MAXPOOL || d.kind == MT_ADD) {    // an addition has two inputs
                ops_mb += M * ((double)d.in_h * d.in_w * d.cin * (d.kind == MT_ADD ? 2.0 : 1.0) + d.out_len) * es / MB;
            }
        }
        if (c->max_nt[0][l] > 0) launch(std::max(chain, kUsFcFixed + us_per_mb * w_mb + kUsPerMbL2 * l2_mb));
        if (conv_plan.first_cap) launch(kUsConvFirstFixed + std::max(first_mb / kConvFirstMbPerUs, first_mflop / kConvFirstMflopPerUs));
        else if (conv_plan.split) launch(kUsConvSplitFixed + kUsConvSplitPerKStep * std::max(split_longest, split_steps / kComputeUnits));
        else if (conv_plan.tiles > 0) launch(kUsConvFixed + std::max(conv_chain, std::max(conv_mb / kConvMbPerUs, conv_mflop / (conv_frames ? kConvFrameMflopPerUs : kConvMflopPerUs))));
        if (big_enabled && c->max_nt[2][l] > 0 && tile_bound(c, 2, l, R) >= c->big_min_tiles) {
            // tiles share the chip in rounds of one per compute unit; a tile's time grows with K
            if (big_layer) big_us = std::ceil(big_tiles / kComputeUnits) * kUsBigTileFixed + big_rounds_k / kComputeUnits / 4096.0 * kUsBigTilePer4096;
            launch(kUsBigFixed + big_us);
        }
        if (c->has_gap[l]) launch(kUsSmallFixed + gap_mb / kCopyMbPerUs);
        if (c->has_image_ops[l]) launch(kUsSmallFixed + ops_mb / kCopyMbPerUs);
    }
    if (!fuse_head || c->max_reg_classes > fuse_head_max)
        launch(kUsSmallFixed + std::max(3.0 * R * c->C_pad * 4.0 / MB / kHeadMbPerUs, kUsHeadPerRow * R));
    out->launches = launches;
    out->device_ms = us * 1e-3;
    // models that are not resident have to cross the host link first: their footprint is fixed, so
    // that time is as predictable as the run itself (section 3.3)
    for (uint32_t t = 0; t < T; ++t)
        if (counts[t] && !c->tenants[t].resident) out->upload_bytes += (double)c->tenants[t].arena_len;
    out->upload_ms = out->upload_bytes ? kUsUploadFixed * 1e-3 + out->upload_bytes / kUploadBytesPerMs : 0.0;
    return MT_OK;
}

}  // namespace

mt_status mt_estimate_run(mt_ctx* c, const uint32_t* counts, mt_run_estimate* out)
{
    if (!c || !counts || !out) return MT_EINVAL;
    uint64_t plan;
    return estimate_run(c, counts, out, &plan);
}

mt_status mt_admit(mt_ctx* c, const uint32_t* pending, double budget_ms, uint32_t* admitted, mt_run_estimate* est)
{
    if (!c || !pending || !admitted) return MT_EINVAL;
    if (!(budget_ms > 0.0)) return fail(c, MT_EINVAL, "the budget must be positive");
    const uint32_t T = c->cfg.max_tenants;
    uint32_t top = 0;
    for (uint32_t t = 0; t < T; ++t) {
        if (pending[t] && !c->tenants[t].registered) return fail(c, MT_ENOTFOUND, "tenant %u has no model", t);
        top = std::max(top, pending[t]);
    }
    std::vector<uint32_t> trial(T);
    auto rows_at = [&](uint32_t level) {
        uint64_t rows = 0;
        for (uint32_t t = 0; t < T; ++t) rows += std::min(pending[t], level);
        return rows;
    };
    if (rows_at(top) > c->cfg.max_requests) {                        // the highest level that a run has room for
        uint32_t lo = 0, hi = top - 1;
        while (lo < hi) { const uint32_t mid = lo + (hi - lo + 1) / 2; if (rows_at(mid) <= c->cfg.max_requests) lo = mid; else hi = mid - 1; }
        top = lo;
    }
    struct Level { uint32_t level; uint64_t plan; double ms; mt_run_estimate e; };
    auto look = [&](uint32_t level) {
        Level v{level, 0, 0.0, {}};
        for (uint32_t t = 0; t < T; ++t) trial[t] = std::min(pending[t], level);
        v.ms = estimate_run(c, trial.data(), &v.e, &v.plan) == MT_OK ? v.e.device_ms + v.e.upload_ms : HUGE_VAL;
        return v;
    };
    // Among the levels of one plan the predicted time grows (but for the rows that big tiles leave), and the highest that fits is found by bisection; from one plan to the next
    // it may fall (a launch less).  So the levels above are looked through plan by plan, as far as runs of twice the budget: no plan saves half of a run.
    auto highest = [&](auto& self, const Level& lo, const Level& hi) -> Level {       // of [lo, hi]; level 0: none fits
        if (hi.ms <= budget_ms) return hi;
        if (lo.plan == hi.plan) {
            if (lo.ms > budget_ms) return Level{};
            Level a = lo, b = hi;                                    // a fits, b does not
            while (b.level - a.level > 1) { const Level m = look(a.level + (b.level - a.level) / 2); (m.ms <= budget_ms ? a : b) = m; }
            return a;
        }
        if (hi.level - lo.level <= 1) return lo.ms <= budget_ms ? lo : Level{};
        const uint32_t mid = lo.level + (hi.level - lo.level) / 2;
        const Level above = self(self, look(mid + 1), hi);
        return above.level ? above : self(self, lo, look(mid));
    };
    Level best = look(top);
    if (top > 0 && best.ms > budget_ms) {
        best = Level{};
        uint32_t none = top;                                         // some level that fits: the highest, if the time only grew
        while (none - best.level > 1) { const Level m = look(best.level + (none - best.level) / 2); if (m.ms <= budget_ms) best = m; else none = m.level; }
        uint32_t from = best.level + 1, to = std::min(top, from + best.level);
        while (from <= top) {                                        // [from, to], more levels each time
            const Level lo = look(from), hi = look(to);
            const Level found = highest(highest, lo, hi);
            if (found.level) best = found;
            if (hi.ms > 2.0 * budget_ms && lo.ms > 2.0 * budget_ms) break;
            from = to + 1;
            to += std::min(top - to, to + 1);
        }
    }
    for (uint32_t t = 0; t < T; ++t) trial[t] = std::min(pending[t], best.level);
    const mt_run_estimate e = best.e;
    for (uint32_t t = 0; t < T; ++t) admitted[t] = trial[t];
    if (est) *est = e;
    return MT_OK;
}

mt_status mt_set_profiling(mt_ctx* c, int enable)
{
    if (!c) return MT_EINVAL;
    if (c->host_only) return fail(c, MT_ESTATE, "host-only context");
    if (enable && c->prof_events.empty()) {
        HIP_TRY(c, hipSetDevice(c->cfg.device));
        c->prof_events.resize(2 * kProfSlots);
        for (hipEvent_t& e : c->prof_events) HIP_TRY(c, hipEventCreate(&e));
    }
    c->profiling = enable != 0;
    if (!enable) c->prof_valid = false;
    return MT_OK;
}

mt_status mt_get_profile(mt_ctx* c, mt_profile* out)
{
    if (!c || !out) return MT_EINVAL;
    std::memset(out, 0, sizeof *out);
    if (!c->prof_valid) return fail(c, MT_ESTATE, "no profiled run to read");
    HIP_TRY(c, hipSetDevice(c->cfg.device));
    HIP_TRY(c, hipStreamSynchronize(c->last_stream));
    auto ms = [&](uint32_t slot, float* dst) -> hipError_t {
        *dst = 0.0f;
        if (!c->prof_used[slot]) return hipSuccess;
        return hipEventElapsedTime(dst, c->prof_events[2 * slot], c->prof_events[2 * slot + 1]);
    };
    HIP_TRY(c, ms(kProfBatcher, &out->batcher_ms));
    HIP_TRY(c, ms(kProfGather, &out->gather_ms));
    { float img = 0.0f; HIP_TRY(c, ms(kProfGatherImg, &img)); out->gather_ms += img; }
    HIP_TRY(c, ms(kProfHead, &out->head_ms));
    for (uint32_t l = 0; l < MT_MAX_LAYERS; ++l) {
        HIP_TRY(c, ms(kProfFc + l, &out->fc_ms[l]));
        HIP_TRY(c, ms(kProfConv + l, &out->conv_ms[l]));
        HIP_TRY(c, ms(kProfBig + l, &out->fc_big_ms[l]));
        HIP_TRY(c, ms(kProfGap + l, &out->gap_ms[l]));
        HIP_TRY(c, ms(kProfImageOps + l, &out->ops_ms[l]));
    }
    HIP_TRY(c, hipEventElapsedTime(&out->total_ms, c->prof_events[2 * kProfBatcher], c->prof_events[2 * c->prof_last + 1]));
    return MT_OK;
}

mt_status mt_debug_copy(void* dst, const void* src, uint64_t bytes, void* stream)
{
    if (!dst || !src || bytes % 16) return MT_EINVAL;
    return launch_copy(dst, src, bytes, (hipStream_t)stream) == hipSuccess ? MT_OK : MT_EDEVICE;
}

mt_status mt_debug_mfma_rate(void* stream, double* tflops)
{
    if (!tflops) return MT_EINVAL;
    *tflops = 0.0;
    constexpr uint32_t kGrid = 2048, kIters = 500;          // 2048 workgroups of 8 waves x 500 x 64 MFMAs: ~10 ms
    hipStream_t s = (hipStream_t)stream;
    float* buf = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    float ms = 0.0f;
    hipError_t e = hipMalloc((void**)&buf, (size_t)kGrid * 512 * 4);
    if (e == hipSuccess) e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e == hipSuccess) e = launch_mfma_rate(buf, kIters / 10, kGrid, s);      // warm-up
    if (e == hipSuccess) e = hipEventRecord(e0, s);
    if (e == hipSuccess) e = launch_mfma_rate(buf, kIters, kGrid, s);
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (buf) (void)hipFree(buf);
    if (e != hipSuccess || ms <= 0.0f) return MT_EDEVICE;
    *tflops = (double)kGrid * 8 * kIters * 64 * 32768.0 / (ms * 1e-3) / 1e12;
    return MT_OK;
}

uint32_t mt_debug_big_tile_rows(uint32_t rows, uint32_t out_features)
{
    return fc_is_big(rows, round_up(out_features, (uint32_t)kBrickRows)) ? big_rows(rows) : 0;
}

uint32_t mt_debug_big_tile_walk(uint32_t in_features)
{
    return round_up(in_features, (uint32_t)kWidthAlign) >= kBigWalkMinK ? 1 : 0;
}

uint32_t mt_debug_conv_frame_ahead(uint32_t max_tenants, uint32_t channel_blocks, uint32_t frame_bytes, uint64_t workgroups)
{
    return conv_img_few(max_tenants, channel_blocks, frame_bytes, workgroups) ? 1 : 0;
}

int mt_debug_conv_row_tiling(uint32_t in_h, uint32_t in_w, uint32_t in_channels, uint32_t ksize, uint32_t stride, uint32_t elem_size,
                             uint32_t* rows_per_tile, uint32_t* images_per_tile, uint32_t* tiles_per_image, uint64_t* frame_bytes)
{
    RowTiling r{0, 0, 0};
    uint64_t frame = 0;
    if (ksize >= 1 && (ksize & 1) && (stride == 1 || stride == 2) && (elem_size == 2 || elem_size == 4) && in_h && in_w && in_channels) {
        LayerDev d{};
        const uint32_t pad = (ksize - 1) / 2;
        const uint32_t oh = (in_h + 2 * pad - ksize) / stride + 1, ow = (in_w + 2 * pad - ksize) / stride + 1;
        d.kind = MT_CONV2D; d.cin = round_up(in_channels, (uint32_t)kChanPad); d.in_h = in_h; d.in_w = in_w; d.stride = stride;
        d.out_w = ow; d.ksize = ksize; d.pad = pad; d.rows_per_req = oh * ow;
        const uint32_t packed = choose_row_tiling(d, elem_size);
        if (packed) { r = unpack_row_tiling(packed); frame = row_tile_frame_bytes(d, elem_size, r); }
    }
    if (rows_per_tile) *rows_per_tile = r.n_oh;
    if (images_per_tile) *images_per_tile = r.ni;
    if (tiles_per_image) *tiles_per_image = r.tpi;
    if (frame_bytes) *frame_bytes = frame;
    return r.n_oh != 0;
}

mt_status mt_debug_conv_launch(mt_ctx* c, uint32_t layer, uint32_t rows, const uint32_t* counts, uint32_t* split, uint64_t* workgroups)
{
    if (!c) return MT_EINVAL;
    if (layer >= MT_MAX_LAYERS || rows == 0) return fail(c, MT_EINVAL, "layer %u, %u rows", layer, rows);
    std::vector<NamedRows> named;
    for (uint32_t t = 0; counts && t < c->cfg.max_tenants; ++t) {
        if (!counts[t]) continue;
        if (!c->tenants[t].registered) return fail(c, MT_ENOTFOUND, "tenant %u has no model", t);
        named.push_back({t, counts[t]});
    }
    const ConvPlan p = plan_conv(c, layer, rows, counts ? &named : nullptr);
    if (split) *split = p.split;
    if (workgroups) *workgroups = p.tiles;
    return MT_OK;
}

mt_status mt_debug_poison(mt_ctx* c)
{
    if (!c) return MT_EINVAL;
    if (c->host_only) return fail(c, MT_ESTATE, "host-only context");
    HIP_TRY(c, hipSetDevice(c->cfg.device));
    HIP_TRY(c, hipDeviceSynchronize());
    const size_t act_bytes = (size_t)c->P_cap * c->S * c->elem_size;
    for (RunSlot& r : c->slots) {
        for (uint32_t i = 0; i < c->act_buffers; ++i) HIP_TRY(c, hipMemset(r.d_act[i], 0xFF, act_bytes));
        HIP_TRY(c, hipMemset(r.d_logits, 0xFF, (size_t)c->P_cap * c->C_pad * 4));
    }
    HIP_TRY(c, hipDeviceSynchronize());
    return MT_OK;
}

mt_status mt_cache_stats_get(const mt_ctx* c, mt_cache_stats* out)
{
    if (!c || !out) return MT_EINVAL;
    *out = mt_cache_stats{};
    for (const HostTenant& t : c->tenants) if (t.registered && t.resident) out->resident_models++;
    out->uploads = c->n_uploads; out->upload_bytes = c->upload_bytes; out->evictions = c->n_evictions;
    return MT_OK;
}

mt_status mt_get_stats(const mt_ctx* c, mt_stats* out)
{
    if (!c || !out) return MT_EINVAL;
    out->n_tenants = c->n_registered;
    out->arena_used = c->arena_used;
    out->arena_bytes = c->cfg.arena_bytes;
    out->last_run_rows = c->last_run_rows;
    out->last_run_launches = c->last_run_launches;
    return MT_OK;
}

}  // extern "C"

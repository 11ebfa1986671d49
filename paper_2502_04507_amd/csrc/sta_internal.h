// Internal declarations shared by the translation units of libsta (GPU side only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include <type_traits>

namespace sta {

// A launch without the call that keeps its grid for another to fetch, which <<<>>> makes of it: 2.40 -> 2.19 us a launch, as many as the
// host can make, whatever the arguments (2.4 KB of them 2.65 -> 2.43).  It returns its own error alone: one that an earlier call of the
// program left stays for whoever made that call.
template <typename... Params>
hipError_t launch_kernel(void (*kernel)(Params...), dim3 grid, dim3 block, hipStream_t stream, const std::common_type_t<Params> &...args)
{
    void *arguments[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    const hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, arguments, 0, stream);
    if (e != hipSuccess) (void)hipGetLastError();           // it is returned, and not left for the next call to find
    return e;
}

// Division of any 32-bit number by a launch constant with one multiplication: n / d = (((n - q) >> pre) + q) >> post
// with q = the upper half of n * magic (Granlund and Montgomery, Division by Invariant Integers using Multiplication, 1994).
struct FastDiv {
    uint32_t d, magic;
    uint32_t pre, post;
};
inline FastDiv fast_div_of(uint32_t d)
{
    const uint32_t s = d <= 1 ? 0 : 32 - __builtin_clz(d - 1);      // ceil(log2 d)
    FastDiv f;
    f.d = d;
    f.magic = (uint32_t)(((((uint64_t)1 << s) - d) << 32) / d) + 1;
    f.pre = s < 1 ? s : 1;
    f.post = s < 1 ? 0 : s - 1;
    return f;
}

// ---- permutation -----------------------------------------------------------
struct PermuteParams {
    FastDiv by_row;             // workgroups per row of tiles along w
    FastDiv by_parts;           // workgroups per tile
    FastDiv by_n_h;             // rows of tiles per layer of tiles (tiles at one place along t)
    uint32_t blocks;            // workgroups
    uint32_t in_rounds;         // workgroups in full rounds of eight rows of tiles, one row per XCD
    uint32_t n_w;               // tiles per row
    // in chunks of 8 elements
    uint32_t chunks_per_tile;   // P * D / 8
    uint32_t seg, seg_magic;    // contiguous run of a tile in raster order, ceil(2^32/seg)
    uint32_t T_h, T_h_magic;    // runs of a tile in one raster plane, ceil(2^32 / T_h)
    uint32_t line;              // raster line of tokens: at most 30000 runs of less than 2^16, which stays below 2^31
    uint64_t plane;             // and plane: 2^32 where one of D = 64 holds 2^29 tokens (64 GB)
    uint64_t tile_h;            // from a tile to the next along h
    uint64_t tile_t;            // and along t; slices follow each other at multiples of it
};
constexpr int kPermuteThreads = 256;

// n / d with magic = ceil(2^32 / d) for d > 1; exact while n * d < 2^32 (checked on the host).
__host__ __device__ __forceinline__ uint32_t small_div(uint32_t n, uint32_t d, uint32_t magic)
{
    return d == 1 ? n : (uint32_t)(((uint64_t)n * magic) >> 32);
}

__host__ __device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv &f);

// The tile that a workgroup moves a part of: the chunks where it begins in either order.
struct PermuteTile {
    uint64_t raster, tiled;
    uint32_t part;
};
__host__ __device__ __forceinline__ PermuteTile permute_tile(uint32_t id, const PermuteParams &p)
{
    const bool left_over = id >= p.in_rounds;
    const uint32_t turn = left_over ? id : id >> 3;
    const uint32_t q = fast_div(turn, p.by_row), in_row = turn - q * p.by_row.d;
    const uint32_t row = left_over ? q : 8 * q + (id & 7);                  // row of tiles along w, of all slices
    const uint32_t tw = fast_div(in_row, p.by_parts), part = in_row - tw * p.by_parts.d;
    const uint32_t layer = fast_div(row, p.by_n_h), th = row - layer * p.by_n_h.d;
    return {layer * p.tile_t + th * p.tile_h + tw * p.seg, ((uint64_t)row * p.n_w + tw) * p.chunks_per_tile, part};
}
// Raster chunk, from the tile's first, of chunk idx of the tile.
__host__ __device__ __forceinline__ uint64_t permute_piece(uint32_t idx, const PermuteParams &p)
{
    const uint32_t seg = small_div(idx, p.seg, p.seg_magic);                // which (i_t, i_h) run
    const uint32_t off = idx - seg * p.seg;
    const uint32_t it = small_div(seg, p.T_h, p.T_h_magic);
    const uint32_t ih = seg - it * p.T_h;
    return it * p.plane + ((uint64_t)ih * p.line + off);
}

// Split of the tiles of all slices over workgroups, of so many chunks each; false: more of them than are numbered.
bool permute_split(PermuteParams *p, bool src_f32, bool dst_f32, uint64_t tiles, uint32_t *per_block, bool *streamed);

hipError_t launch_permute(const void *src, void *dst, bool src_f32, bool dst_f32, bool to_tiled,
                          PermuteParams p, uint64_t tiles, hipStream_t stream);

// ---- attention -------------------------------------------------------------
// What a launch would run, as text, one line per kernel: for tests of the rules that choose the shapes, without a GPU.
struct LaunchNote {
    char *text;
    size_t size, used = 0;
    __attribute__((format(printf, 2, 3))) hipError_t add(const char *format, ...)
    {
        va_list args;
        va_start(args, format);
        const int n = vsnprintf(text + used, size - used, format, args);
        va_end(args);
        if (n < 0 || (size_t)n + 1 >= size - used) return hipErrorInvalidValue;
        used += (size_t)n + 1;
        text[used - 1] = '\n';
        text[used] = 0;
        return hipSuccess;
    }
};

uint32_t compute_units();           // of the device that is current at the first call

constexpr int kMaxHeadsPerLaunch = 256;

struct WindowTable {
    uint16_t w[kMaxHeadsPerLaunch][3];   // window in tiles per head of this launch (clamped to 2*n)
};

// Heads of one launch in the order the kernel visits them (most expensive first).
struct HeadOrder {
    uint16_t h[kMaxHeadsPerLaunch];
};

struct FwdParams {
    uint32_t N;            // tokens per head
    uint32_t P;            // tokens per tile
    uint32_t n_t, n_h, n_w;
    uint32_t n_tiles;
    uint32_t H;            // heads in the tensor
    uint32_t head_base;    // first head of this launch
    uint32_t heads;        // heads in this launch
    float scale_log2e;     // softmax scale * log2(e)
    uint32_t T_t = 1, T_h = 1, T_w = 1;   // tile shape in tokens (used by the token-masked sliding-window kernel only)
    float *lse = nullptr;  // optional output [B,H,N] (tiled order): ln of each row's softmax denominator; may be null
    // work splitting below one query block (filled in by the launcher): item ids from split_first on are run
    // by split_parts workgroups each, which leave partial results in split_ws
    uint32_t split_first = 0xffffffffu;
    uint32_t split_parts = 1;
    float *split_ws = nullptr;
};

// The DMA into LDS fetches 16 bytes per lane; tensors are only asked to hold elements.
inline bool dma_aligned(const void *p) { return ((uintptr_t)p & 15) == 0; }

// n divided by the launch constant of f.
__host__ __device__ __forceinline__ uint32_t fast_div(uint32_t n, const FastDiv &f)
{
    const uint32_t q = (uint32_t)(((uint64_t)n * f.magic) >> 32);
    return (((n - q) >> f.pre) + q) >> f.post;
}

// How the items of a launch are dealt to the workgroup ids, which the hardware gives to the 8 XCDs in turn: rounds of
// eight chunks of consecutive items, one per XCD, and a last round that divides what is left evenly (the first last_more XCDs
// get one item more).  Every id below total names an item, and no XCD gets more than one item more than another.
struct Deal {
    uint32_t total;            // items
    FastDiv chunk;             // consecutive items of one XCD
    uint32_t last_slot;        // slots (ids of one XCD) in full rounds
    uint32_t last_len, last_more;
};
inline Deal deal_in_chunks(uint32_t total, uint32_t chunk)
{
    Deal d;
    d.total = total;
    d.chunk = fast_div_of(chunk);
    d.last_slot = (uint32_t)(total / (8 * (uint64_t)chunk)) * chunk;
    const uint32_t left = total - 8 * d.last_slot;
    d.last_len = left / 8;
    d.last_more = left % 8;
    return d;
}
// per_head items of each of n_bh (batch, head) slices: as many rounds of chunks as eighths of a head would take.
inline Deal deal_of(uint32_t per_head, uint32_t n_bh)
{
    const uint32_t total = per_head * n_bh;
    const uint32_t eighth = (per_head + 7) / 8, rounds = (total + 8 * eighth - 1) / (8 * eighth);
    return deal_in_chunks(total, (total + 8 * rounds - 1) / (8 * rounds));
}
__host__ __device__ __forceinline__ uint32_t dealt_item(uint32_t id, const Deal &d)
{
    // without a branch: a workgroup waits for this before anything else
    const uint32_t xcd = id & 7, slot = id >> 3, first_slot = fast_div(slot, d.chunk) * d.chunk.d;       // of the round
    const bool last = slot >= d.last_slot;
    const uint32_t more = xcd < d.last_more ? xcd : d.last_more;
    return slot + 7 * first_slot + xcd * (last ? d.last_len : d.chunk.d) + (last ? more : 0);
}

// The work items of one launch of a forward kernel, with everything a workgroup would otherwise have to find by division
// (see group_item_of).
struct FwdPlan {
    // what leads to the head stands first: one scalar load brings it, and the rest is on its way with the head's window
    Deal deal;
    FastDiv per_head;          // items of one (batch, head)
    FastDiv batch;
    FastDiv per_tile;          // items of one query tile
    FastDiv pair_items;        // query tiles of two tile rows
    FastDiv n_t;
    FastDiv sub_per_tile;      // 32-key units of a key tile
    struct Head {
        uint16_t h, w[3];      // head inside the launch, its window in tiles; most expensive head first
    } head[kMaxHeadsPerLaunch];
};

// Returns hipErrorInvalidValue if no kernel instance exists for (P, D).
// split_ws: optional device scratch for work splitting (null: every item is run by one workgroup).
hipError_t launch_forward(const void *q, const void *k, const void *v, void *o, int B, int D,
                          const FwdParams &p, const WindowTable &win, const HeadOrder &order, float *split_ws,
                          size_t split_ws_floats, hipStream_t stream, LaunchNote *note = nullptr);
size_t forward_split_workspace_bytes(int P, int D);    // upper bound of what the splitting ever uses
// The general (register-staged) kernel for any supported shape.  token_window = false: the STA mask, win in tiles
// (same results as launch_forward).  token_window = true: the token-granular sliding window, win in tokens.
hipError_t launch_forward_general(const void *q, const void *k, const void *v, void *o, int B, int D, const FwdParams &p,
                                  const WindowTable &win, bool token_window, hipStream_t stream);
constexpr uint32_t kMaxTokenWindowTile = 1024;         // tokens per tile the sliding-window kernel's table holds
bool forward_supported(int P, int D);

// ---- gradients ---------------------------------------------------------------
// stats: float [2][stat_rows] scratch, stat_rows = B * H * N: minus dO_i . O_i and minus lse_i / scale of every query row
// (filled by the call, for the heads of the launch).
hipError_t launch_backward(const void *q, const void *k, const void *v, const void *o, const void *d_o, const float *lse,
                           float *stats, size_t stat_rows, void *d_q, void *d_k, void *d_v, int B, int D, const FwdParams &p,
                           const WindowTable &win, const HeadOrder &order, hipStream_t stream, LaunchNote *note = nullptr);
bool backward_supported(int P, int D);

// ---- reductions around the attention kernel ----------------------------------
constexpr int kMseSlices = 64;     // partial sums per (batch, head) slab
// best: null, or int32 [H] that receives the index of the first smallest of n_before + 1 losses of every head; the n_before
// others, [n_before][H], stand in front of mse_per_head.
hipError_t launch_head_mse(const void *a, const void *b, int B, int H, size_t elems_per_head, double *partial,
                           float *mse_per_head, int n_before, int32_t *best, hipStream_t stream);
// Allocation-free variant: the partial sums live in a file-scope device array of kStaticMseMaxSlabs * kMseSlices
// doubles.  static_mse_scratch returns the current device's address of that array (looked up once per device).
constexpr int kStaticMseMaxSlabs = 1024;
hipError_t static_mse_scratch(double **out);
hipError_t launch_recall(const float *lse_window, const float *lse_full, int BH, size_t N, float *recall,
                         double *partial, float *mean_bh, hipStream_t stream);

hipError_t launch_dump_key_tiles(const FwdParams &p, const WindowTable &win, int32_t *counts,
                                 int32_t *lists, hipStream_t stream);

}  // namespace sta

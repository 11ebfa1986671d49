// Tile / untile permutation kernels (HBM-bound).
//
// STA orders tokens so that each (T_t, T_h, T_w) tile occupies one contiguous
// run of the sequence (Sec. 3.1; appendix "Tiling in STA").  In
// raster order a tile is T_t*T_h runs of T_w consecutive tokens, so both sides
// of the copy are made of contiguous segments of T_w*D elements: a workgroup
// moves 256 or 512 pieces of 8 elements (16 B of bf16) of one tile of one
// (batch, head) slice, with the tiled side fully linear.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sta_device_util.h"
#include "sta_internal.h"

namespace {

struct alignas(16) Chunk8bf16 { uint32_t w[4]; };
struct alignas(16) Chunk8f32 { float4 lo, hi; };

__device__ __forceinline__ uint32_t pack2_bf16(float a, float b)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    bf16x2_t v;
    v[0] = static_cast<__bf16>(a);   // round to nearest even
    v[1] = static_cast<__bf16>(b);
    return __builtin_bit_cast(uint32_t, v);
}

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// STREAM: a load that is not to stay in the caches.
template <bool STREAM>
__device__ __forceinline__ u32x4_t load16(const void *base, size_t chunk16)
{
    const u32x4_t *p = reinterpret_cast<const u32x4_t *>(base) + chunk16;
    if constexpr (STREAM) return __builtin_nontemporal_load(p);
    else return *p;
}

// Load 8 elements as raw bf16 bits (4 dwords) or as 8 floats.
template <bool SRC_F32, bool STREAM>
__device__ __forceinline__ void load8(const void *base, size_t chunk, Chunk8bf16 &b, Chunk8f32 &f)
{
    if constexpr (SRC_F32) {
        f.lo = __builtin_bit_cast(float4, load16<STREAM>(base, 2 * chunk));
        f.hi = __builtin_bit_cast(float4, load16<STREAM>(base, 2 * chunk + 1));
    } else {
        b = __builtin_bit_cast(Chunk8bf16, load16<STREAM>(base, chunk));
    }
}

// 16-byte store that does not leave a dirty line in L2.  The outputs are written once and read by a later kernel;
// with ordinary stores the dirty lines are written back when the kernel ends, which at small sizes costs more than
// the copy itself (measured: 4 MB tensor 17 -> 2.7 us per launch, 85 MB tensor 33 -> 25.6 us, 1.4 GB 261 -> 247 us).
__device__ __forceinline__ void store16_streaming(void *base, size_t chunk16, u32x4_t v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t *>(base) + chunk16);
}

template <bool SRC_F32, bool DST_F32>
__device__ __forceinline__ void store8(void *base, size_t chunk, const Chunk8bf16 &b, const Chunk8f32 &f)
{
    if constexpr (!DST_F32) {
        u32x4_t o;
        if constexpr (SRC_F32) {                 // f32 -> bf16
            o[0] = pack2_bf16(f.lo.x, f.lo.y);
            o[1] = pack2_bf16(f.lo.z, f.lo.w);
            o[2] = pack2_bf16(f.hi.x, f.hi.y);
            o[3] = pack2_bf16(f.hi.z, f.hi.w);
        } else {
            o[0] = b.w[0]; o[1] = b.w[1]; o[2] = b.w[2]; o[3] = b.w[3];
        }
        store16_streaming(base, chunk, o);
    } else {
        u32x4_t lo, hi;
        if constexpr (SRC_F32) {
            lo[0] = __float_as_uint(f.lo.x); lo[1] = __float_as_uint(f.lo.y);
            lo[2] = __float_as_uint(f.lo.z); lo[3] = __float_as_uint(f.lo.w);
            hi[0] = __float_as_uint(f.hi.x); hi[1] = __float_as_uint(f.hi.y);
            hi[2] = __float_as_uint(f.hi.z); hi[3] = __float_as_uint(f.hi.w);
        } else {                                 // bf16 -> f32 (exact)
            lo[0] = b.w[0] << 16; lo[1] = b.w[0] & 0xffff0000u; lo[2] = b.w[1] << 16; lo[3] = b.w[1] & 0xffff0000u;
            hi[0] = b.w[2] << 16; hi[1] = b.w[2] & 0xffff0000u; hi[2] = b.w[3] << 16; hi[3] = b.w[3] & 0xffff0000u;
        }
        store16_streaming(base, 2 * chunk, lo);
        store16_streaming(base, 2 * chunk + 1, hi);
    }
}

using sta::kPermuteThreads;
constexpr int kGridShift = 23;                              // a grid holds fewer than 2^32 lanes along x

// TO_TILED: src is raster, dst is tiled.  Otherwise the reverse.
// What bounds it: HBM, and how reads and writes mix there.  CHUNKS pieces of 8 elements per lane: one, so that a workgroup reads and
// writes one run of 4 KB and is gone; two for fp32 sources that are rounded to bf16 and not streamed (26 MB 13.4 -> 12.3 us, 170 MB 50
// -> 44).  us in whole layers, to tiles and back, four pieces (what was here before), two, one, one in the order below: 708 MB 231,
// 236; 234, 241; 217, 224; 214, 216.  85 MB 30.0, 29.6; 29.8, 30.1; 28.6, 29.2; 28.6, 28.4.  96-token tiles, 43 MB 16.9, 17.3; 15.0,
// 16.8; 14.6, 15.8; 14.9, 15.3.  64-token tiles of dimension 64, 67 MB 23.8, 23.8; 24.2, 24.0; 23.1, 23.3; 23.0, 22.8.  32-token tiles
// of dimension 64, a piece per lane before as well, 157 MB 50.3, 49.6; ordered 50.0, 50.3.  One or two by 512 or 1024 lanes: no better.
// From a graph, tensors in turn, four pieces and one: 0.4 MB 2.2, 1.9; 2 MB 2.45, 2.15; 4 MB 3.3, 3.1; but 8 MB 3.95, 4.2; 16 MB 6.2, 6.5
// (two pieces 4.1 and 6.3); 22 MB 8.4, 8.4; 37 MB 14.8, 13.9.
// Order: workgroup ids go round-robin over the 8 XCDs; every XCD takes whole rows of tiles along w, whose tokens are one piece of each
// raster row, in turn with the others (full rounds of eight rows; what is left over in the order of the ids).
template <bool SRC_F32, bool DST_F32, bool TO_TILED, bool STREAM, int CHUNKS>
__global__ __launch_bounds__(kPermuteThreads) void sta_permute_kernel(const void *__restrict__ src,
                                                                     void *__restrict__ dst,
                                                                     sta::PermuteParams p)
{
    // Every argument is asked for at once and waited for once.  Left to the compiler they come where they are first used, behind the
    // bounds of the grid, of a round and of the tile: four waits one after the other, and three more divisions (the places of a tile along
    // t and of its slice are one number, since slices follow each other like the layers of tiles of one).  us from tensors in turn that are
    // not in the L2 caches, before and now, a plain copy of the size: 0.2 MB 2.38, 2.27; fp32 to 1.3 MB of bf16 2.64, 2.50; 4 MB 2.98, 2.73,
    // 2.61; 17 MB 6.39, 6.01, 5.91; 43 MB 15.4, 15.2, 15.8; 67 MB 23.6, 23.2, 23.3; 85 MB 28.7, 28.4, 28.6; back 4 MB 2.94, 2.67; 67 MB 23.4, 22.9.
    asm volatile("" ::"s"(src), "s"(dst), "s"(p.by_row.d), "s"(p.by_row.magic), "s"(p.by_row.pre), "s"(p.by_row.post), "s"(p.by_parts.d), "s"(p.by_parts.magic),
                 "s"(p.by_parts.pre), "s"(p.by_parts.post), "s"(p.by_n_h.d), "s"(p.by_n_h.magic), "s"(p.by_n_h.pre), "s"(p.by_n_h.post));
    asm volatile("" ::"s"(p.blocks), "s"(p.in_rounds), "s"(p.n_w), "s"(p.chunks_per_tile), "s"(p.seg), "s"(p.seg_magic), "s"(p.T_h),
                 "s"(p.T_h_magic), "s"(p.line), "s"(p.plane), "s"(p.tile_h), "s"(p.tile_t));
    const uint32_t id = (blockIdx.y << kGridShift) + blockIdx.x;
    const sta::PermuteTile tile = sta::permute_tile(id, p);
    const uint32_t first = tile.part * (kPermuteThreads * CHUNKS) + threadIdx.x;
    Chunk8bf16 b[CHUNKS];
    Chunk8f32 f[CHUNKS];
    size_t dst_idx[CHUNKS];
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) {
        const uint32_t idx = first + u * kPermuteThreads;
        const size_t raster = tile.raster + sta::permute_piece(idx, p);
        const size_t tiled = tile.tiled + idx;
        dst_idx[u] = TO_TILED ? tiled : raster;
        if (idx < p.chunks_per_tile && id < p.blocks) load8<SRC_F32, STREAM>(src, TO_TILED ? raster : tiled, b[u], f[u]);
    }
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u)
        if (first + u * kPermuteThreads < p.chunks_per_tile && id < p.blocks) store8<SRC_F32, DST_F32>(dst, dst_idx[u], b[u], f[u]);
}

template <bool TO_TILED, bool STREAM>
hipError_t launch(const void *src, void *dst, bool src_f32, bool dst_f32, const sta::PermuteParams &p,
                  hipStream_t stream)
{
    constexpr int kRounded = STREAM ? 1 : 2;                // fp32 to bf16
    dim3 g(p.blocks >> kGridShift ? 1u << kGridShift : p.blocks, ((p.blocks - 1) >> kGridShift) + 1), b(kPermuteThreads);
    if (!src_f32 && !dst_f32) return sta::launch_kernel(sta_permute_kernel<false, false, TO_TILED, STREAM, 1>, g, b, stream, src, dst, p);
    if (src_f32 && !dst_f32) return sta::launch_kernel(sta_permute_kernel<true, false, TO_TILED, STREAM, kRounded>, g, b, stream, src, dst, p);
    if (!src_f32 && dst_f32) return sta::launch_kernel(sta_permute_kernel<false, true, TO_TILED, STREAM, 1>, g, b, stream, src, dst, p);
    return sta::launch_kernel(sta_permute_kernel<true, true, TO_TILED, STREAM, 1>, g, b, stream, src, dst, p);
}

// Sources larger than the 256 MB Infinity Cache are read with streaming loads.  us, ordinary against streaming, source written
// by the kernel before and, in brackets, another tensor of its size: 294 MB (fp32) 97, 85 (109, 78); 354 MB (bf16) 148, 120 (161,
// 118); 708 MB 277, 240 (300, 235).  So they are the faster ones also where most of the source is still in the cache; below that
// size they lose on a source that is there: 177 MB (fp32) 41, 55 (59, 50), 17 MB 6.2, 7.6.
constexpr size_t kStreamAbove = (size_t)256 << 20;

}  // namespace

namespace sta {

bool permute_split(PermuteParams *p, bool src_f32, bool dst_f32, uint64_t tiles, uint32_t *per_block, bool *streamed)
{
    *streamed = tiles * p->chunks_per_tile * (src_f32 ? 32 : 16) > kStreamAbove;
    *per_block = kPermuteThreads * (src_f32 && !dst_f32 && !*streamed ? 2 : 1);
    const uint32_t parts = (p->chunks_per_tile + *per_block - 1) / *per_block;
    if (tiles * parts >= ((uint64_t)1 << 31)) return false;                          // terabytes
    p->blocks = (uint32_t)(tiles * parts);
    p->by_parts = fast_div_of(parts);
    p->by_row = fast_div_of(p->n_w * parts);
    const uint64_t round = (uint64_t)8 * p->by_row.d;
    p->in_rounds = (uint32_t)(p->blocks / round * round);
    return true;
}

hipError_t launch_permute(const void *src, void *dst, bool src_f32, bool dst_f32, bool to_tiled,
                          PermuteParams p, uint64_t tiles, hipStream_t stream)
{
    uint32_t per_block;
    bool streamed;
    if (!permute_split(&p, src_f32, dst_f32, tiles, &per_block, &streamed)) return hipErrorInvalidValue;
    if (streamed)
        return to_tiled ? launch<true, true>(src, dst, src_f32, dst_f32, p, stream)
                        : launch<false, true>(src, dst, src_f32, dst_f32, p, stream);
    return to_tiled ? launch<true, false>(src, dst, src_f32, dst_f32, p, stream)
                    : launch<false, false>(src, dst, src_f32, dst_f32, p, stream);
}

}  // namespace sta

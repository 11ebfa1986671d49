// Staging of K/V (or Q/dO) sub-blocks through LDS, shared by the kernels built on v_mfma_f32_16x16x32_bf16: the walk over
// the tiles of a box, the LDS layout of a staged operand, and the two kinds of product with it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sta_device_util.h"
#include "sta_geometry.h"
#include "sta_internal.h"

namespace {

constexpr int kSub = 32;               // tokens per staged sub-block

// Walks the sub-blocks of the tiles of a box; next_row is the first token row (tiled order, inside the head) of
// the sub-block to request next.  Along each axis the box [lo, hi] holds e = hi-lo+1 consecutive tiles, hence
// one tile of every residue class mod e; they are taken in the order of that residue, i.e. the walk starts
// inside the box and wraps from hi to lo.  Neighbouring workgroups, whose boxes are shifted by one tile, then
// reach the tiles they share at the same step of their walks and find them in their XCD's L2.
struct BoxWalk {
    StaBox box;
    int n_h, n_w, P, sub_per_tile;
    int e_h, e_w, start_h, start_w, left_h, left_w;
    int t, h, w, s;
    uint32_t next_row;
    // a / b for 0 <= a, b <= 30000 (tile coordinates and box sides): the quotient is at least 0.5 / b away from where
    // truncation would go wrong, which the rounding of the reciprocal and the product cannot reach
    __device__ __forceinline__ static int small_div(int a, int b)
    {
        return __builtin_amdgcn_readfirstlane((int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b)));
    }
    __device__ __forceinline__ static int first_of(const StaAxisRange &r)      // the tile of the box with k mod e == 0
    {
        const int e = r.hi - r.lo + 1, rest = r.lo - small_div(r.lo, e) * e;
        return rest == 0 ? r.lo : r.lo + e - rest;
    }
    __device__ __forceinline__ void start(const StaBox &b, int nh, int nw, int tokens_per_tile)
    {
        box = b; n_h = nh; n_w = nw; P = tokens_per_tile; sub_per_tile = tokens_per_tile / kSub;
        e_h = b.h.hi - b.h.lo + 1; e_w = b.w.hi - b.w.lo + 1;
        start_h = first_of(b.h); start_w = first_of(b.w);
        t = first_of(b.t); h = start_h; w = start_w; s = 0;
        left_h = e_h; left_w = e_w;
        next_row = tile_row();
    }
    // From the start of the walk to sub-block `sub` of its tile number `tiles`.
    __device__ __forceinline__ void skip(uint32_t tiles, uint32_t sub)
    {
        const uint32_t rows = tiles / (uint32_t)e_w, planes = rows / (uint32_t)e_h;
        const int jw = (int)(tiles - rows * e_w), jh = (int)(rows - planes * e_h);
        left_w = e_w - jw;
        left_h = e_h - jh;
        w += jw; if (w > box.w.hi) w -= e_w;
        h += jh; if (h > box.h.hi) h -= e_h;
        t += (int)planes; if (t > box.t.hi) t -= box.t.hi - box.t.lo + 1;
        s = (int)sub;
        next_row = tile_row() + sub * kSub;
    }
    __device__ __forceinline__ void next_tile()
    {
        if (++w > box.w.hi) w = box.w.lo;
        if (--left_w == 0) {
            left_w = e_w;
            w = start_w;
            if (++h > box.h.hi) h = box.h.lo;
            if (--left_h == 0) {
                left_h = e_h;
                h = start_h;
                if (++t > box.t.hi) t = box.t.lo;
            }
        }
    }
    __device__ __forceinline__ uint32_t tile_row() const { return (uint32_t)(((t * n_h + h) * n_w + w) * P); }
    __device__ __forceinline__ void advance()
    {
        next_row += kSub;
        if (++s == sub_per_tile) {
            s = 0;
            next_tile();
            next_row = tile_row();
        }
    }
};

// ---------------------------------------------------------------------------------------------------------
// Staged operands and the two kinds of product.  Register layout of v_mfma_f32_16x16x32_bf16: a lane holds column
// c16 = lane & 15 of a 16x16 result and the rows 4*g4 .. 4*g4+3 (g4 = lane >> 4); of an operand it holds row/column
// c16 and the k-chunk 8*g4 .. 8*g4+7.  A wave's columns are NC blocks of 16, and every fragment read from LDS feeds
// all of them.
// LDS layout of a staged operand (32 token rows).  A DMA instruction fills 1 KB, and a lane's place in it is fixed
// (16 * lane), so any swizzle is applied on the global side: the lane fetches the chunk that belongs at its place.
//  Head dimension 128 (rows of 256 bytes = all 64 banks): groups of 4 rows, 1024 + 32 bytes apart, chunk c of row j
//  of a group at c ^ (j << 2).
//  - by rows (16-byte reads, served for lanes 0-7 together with 24-31, i.e. rows 0..7 at chunk x with rows 8..15
//    at chunk x ^ 1): the four rows of a group land in the four quarters of the 256 bytes, and consecutive groups
//    are turned by 32 bytes, which together with the odd chunk of the second half covers all sixteen positions;
//  - transposed (8-byte reads, served 32 lanes at a time: 8 consecutive rows, two neighbouring chunks each).
//  The stage, the operand, the row block of a row read and the odd channel blocks of a transposing read are
//  offsets inside the instructions: a wave keeps four row addresses (one per k-step) and four transposing ones.
//  Head dimension 64 (rows of 128 bytes, two rows span the banks): rows 128 bytes apart without padding, chunk c of
//  row r at c ^ (((r >> 1) & 3) << 1).
//  - by rows: even rows sit in the lower 128 bytes of a bank line and odd rows in the upper; rows 0, 2, 4, 6 at chunk
//    x take the four even positions of their half, rows 8, 10, 12, 14 at chunk x ^ 1 the four odd ones;
//  - transposed: rows 0, 2, 4, 6 take four different 32-byte pairs of their half, rows 1, 3, 5, 7 the same of theirs.
//  A wave keeps two row addresses (one per k-step) and four transposing ones (one per channel block).
// In both layouts no address is computed inside the loop.
// ---------------------------------------------------------------------------------------------------------
template <int D>
struct Staged {
    static_assert(D == 64 || D == 128, "head dimension");
    static constexpr int RowB = 2 * D;                          // bytes per token row
    static constexpr int KS = D / 32;                           // k-steps of a product over the channels
    static constexpr int CB = D / 16;                           // 16-channel blocks of an accumulator
    static constexpr int GroupRows = 1024 / RowB;               // rows per DMA instruction: 4 or 8
    static constexpr int Groups = kSub / GroupRows;             // DMA instructions per operand: 8 or 4
    static constexpr int Group = D == 128 ? 1024 + 32 : 1024;   // bytes from one group to the next
    static constexpr int Tile = Groups * Group;                 // one staged operand
    static constexpr int Rows16 = (16 / GroupRows) * Group;     // from row r to row r + 16

    // where the 16-byte chunk c of row r (0..31) of a staged operand sits, in bytes from its start
    static __device__ __forceinline__ uint32_t place(int r, int c)
    {
        if constexpr (D == 128) return (uint32_t)((r >> 2) * Group + (r & 3) * RowB + ((c ^ ((r & 3) << 2)) << 4));
        else return (uint32_t)(r * RowB + ((c ^ (((r >> 1) & 3) << 1)) << 4));
    }
    // byte offset, inside a DMA group of the source (GroupRows rows, contiguous), of what the lane fetches
    static __device__ __forceinline__ uint32_t dma_lane_offset(int lane)
    {
        constexpr int LPR = RowB / 16;                          // lanes (chunks) per row
        const int r = lane / LPR, pos = lane % LPR;             // row inside the group, place inside the row
        if constexpr (D == 128) return (uint32_t)(r * RowB + ((pos ^ (r << 2)) << 4));
        else return (uint32_t)(r * RowB + ((pos ^ (((r >> 1) & 3) << 1)) << 4));   // groups start at multiples of 8 rows
    }
    // Per-lane addresses of the operand reads, relative to the start of a staged operand at LDS address `base`.
    //  Row reads (A = 16 tokens x 32 channels): token row c16 (+16 for the second row block), chunk 4*ks + g4.
    //  Transposing reads (A = 16 channels x 32 tokens): within each block of 16 lanes, lane 4*j4 + s4 supplies
    //  channels 4*s4 .. 4*s4+3 of the block's 16 of token row 4*g4 + j4 (+16 for the second read); chunk
    //  2*cb + (s4 >> 1).  With 256-byte rows the XOR reaches cb >> 1 only (cb & 1 is 32 bytes in the instruction),
    //  with 128-byte rows it reaches all of cb: four addresses either way.
    static __device__ __forceinline__ void addresses(uint32_t base, int lane, uint32_t (&row_addr)[KS], uint32_t (&tr_addr)[4])
    {
        const int c16 = lane & 15, g4 = lane >> 4;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) row_addr[ks] = base + place(c16, 4 * ks + g4);
        transposed_addresses(base, lane, tr_addr);
    }
    static __device__ __forceinline__ void transposed_addresses(uint32_t base, int lane, uint32_t (&tr_addr)[4])
    {
        const int g4 = lane >> 4, j4 = (lane & 15) >> 2, s4 = lane & 3;
#pragma unroll
        for (int m = 0; m < 4; ++m)
            tr_addr[m] = base + place(4 * g4 + j4, (D == 128 ? 4 * m : 2 * m) + (s4 >> 1)) + 8 * (s4 & 1);
    }
    static constexpr int tr_index(int cb) { return D == 128 ? cb >> 1 : cb; }
    static constexpr int tr_offset(int cb) { return D == 128 ? (cb & 1) * 32 : 0; }
};

// Brings the 1 KB group of a staged operand whose chunk for this lane starts at src to LDS address dst: by DMA, or, for sources
// that do not start at a multiple of 16 bytes, through a register (a barrier with a wait for LDS has to follow).
template <bool DMA>
__device__ __forceinline__ void stage_group(const char *src, char *dst, int lane)
{
    if constexpr (DMA) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, STA_LDS_PTR(dst), 16, 0, 0);
    } else {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        typedef u32x4 u32x4_anywhere __attribute__((aligned(1)));
        *reinterpret_cast<u32x4 *>(dst + 16 * lane) = *reinterpret_cast<const u32x4_anywhere *>(src);
    }
}

// Waits until at most PENDING of the wave's own requests are outstanding (they complete in order).
template <int PENDING>
__device__ __forceinline__ void wait_dma()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PENDING) : "memory");
}

// Layout of an operand that is read by rows only: groups (one DMA instruction) 1024 + 64 bytes apart, the chunk's two
// low bits XORed with the row inside the group (256-byte rows) or with half of it (128-byte rows).
//  - 256-byte rows: the four rows of a group land in four 16-byte positions of one 64-byte quarter, and consecutive
//    groups are turned by a quarter;
//  - 128-byte rows: even and odd rows take different halves of a bank line, rows 0, 2, 4, 6 the four positions of one
//    quarter of their half; the second group of eight rows is turned by a quarter.
// Either way the k-step (64 bytes) and the row block are offsets inside the instruction: one address per wave.
template <int D>
struct StagedRows {
    static constexpr int RowB = 2 * D;
    static constexpr int KS = D / 32;
    static constexpr int GroupRows = 1024 / RowB;
    static constexpr int Groups = kSub / GroupRows;
    static constexpr int Group = 1024 + 64;
    static constexpr int Tile = Groups * Group;
    static constexpr int Rows16 = (16 / GroupRows) * Group;
    static __device__ __forceinline__ int turn(int r) { return D == 128 ? r & 3 : (r >> 1) & 3; }
    static __device__ __forceinline__ uint32_t dma_lane_offset(int lane)
    {
        constexpr int LPR = RowB / 16;
        const int r = lane / LPR, pos = lane % LPR;
        return (uint32_t)(r * RowB + ((pos ^ turn(r)) << 4));
    }
    // token row c16 (+16 for the second row block), chunk 4*ks + g4
    static __device__ __forceinline__ uint32_t address(uint32_t base, int lane)
    {
        const int r = lane & 15, g4 = lane >> 4;
        return base + (uint32_t)((r / GroupRows) * Group + (r % GroupRows) * RowB + ((g4 ^ turn(r)) << 4));
    }
};

// X[rb][col] += A B with A in the rows-only layout at byte offset OFF of the wave's one address.
template <int D, int OFF, int NC>
__device__ __forceinline__ void rows_times_resident(uint32_t addr, const bf16x8 (&resident)[NC][D / 32], floatx4 (&X)[2][NC])
{
    constexpr int KS = D / 32;
    constexpr int N = 2 * KS;                                   // fragments: KS k-steps of two row blocks
    constexpr int AHEAD = N < 6 ? N : 6;                        // reads in flight
    bf16x8 a[N];
    auto read = [&](auto fc) {
        constexpr int f = decltype(fc)::value;
        a[f] = ds_read_b128_at<OFF + (f / KS) * StagedRows<D>::Rows16 + (f % KS) * 64>(addr);
    };
    static_for<0, AHEAD>(read);
    static_for<0, N / 2>([&](auto pc) {
        constexpr int f = 2 * decltype(pc)::value;              // fragments f and f + 1
        constexpr int issued = f + AHEAD < N ? f + AHEAD : N;
        lds_wait2<issued - f - 2>(a[f], a[f + 1]);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const int col = t ? NC - 1 - i : i;             // one operand changes at a time
                X[f / KS][col] = mfma_16x16x32(a[f + t], resident[col][(f + t) % KS], X[f / KS][col]);
            }
        __builtin_amdgcn_sched_barrier(0);                      // keep each group ahead of the next group's wait
        static_for<(issued < N ? issued : N), (issued + 2 < N ? issued + 2 : N)>(read);
    });
}

// X[rb][col] (16 staged rows x 16 resident columns) += A B: A = the staged operand at byte offset OFF read by rows
// (k = channels), B = resident fragments of the wave's columns; the caller has set X to the value the sums start
// from.  Four reads in flight; a fragment feeds all column blocks, taken 0, 1, 1, 0, .. so that one operand changes
// from one matrix instruction to the next.
template <int D, int OFF, int NC>
__device__ __forceinline__ void staged_rows_times_resident(const uint32_t (&row_addr)[D / 32],
                                                           const bf16x8 (&resident)[NC][D / 32], floatx4 (&X)[2][NC])
{
    constexpr int ROWS16 = OFF + Staged<D>::Rows16;             // rows 16..31
    if constexpr (D == 128) {
        bf16x8 a0 = ds_read_b128_at<OFF>(row_addr[0]), a1 = ds_read_b128_at<OFF>(row_addr[1]);
        bf16x8 a2 = ds_read_b128_at<OFF>(row_addr[2]), a3 = ds_read_b128_at<OFF>(row_addr[3]);
        lds_wait2<2>(a0, a1);
#pragma unroll
        for (int col = 0; col < NC; ++col) X[0][col] = mfma_16x16x32(a0, resident[col][0], X[0][col]);
#pragma unroll
        for (int col = NC - 1; col >= 0; --col) X[0][col] = mfma_16x16x32(a1, resident[col][1], X[0][col]);
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 b0 = ds_read_b128_at<ROWS16>(row_addr[0]), b1 = ds_read_b128_at<ROWS16>(row_addr[1]);
        lds_wait2<2>(a2, a3);
#pragma unroll
        for (int col = 0; col < NC; ++col) X[0][col] = mfma_16x16x32(a2, resident[col][2], X[0][col]);
#pragma unroll
        for (int col = NC - 1; col >= 0; --col) X[0][col] = mfma_16x16x32(a3, resident[col][3], X[0][col]);
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 b2 = ds_read_b128_at<ROWS16>(row_addr[2]), b3 = ds_read_b128_at<ROWS16>(row_addr[3]);
        lds_wait2<2>(b0, b1);
#pragma unroll
        for (int col = 0; col < NC; ++col) X[1][col] = mfma_16x16x32(b0, resident[col][0], X[1][col]);
#pragma unroll
        for (int col = NC - 1; col >= 0; --col) X[1][col] = mfma_16x16x32(b1, resident[col][1], X[1][col]);
        __builtin_amdgcn_sched_barrier(0);
        lds_wait2<0>(b2, b3);
#pragma unroll
        for (int col = 0; col < NC; ++col) X[1][col] = mfma_16x16x32(b2, resident[col][2], X[1][col]);
#pragma unroll
        for (int col = NC - 1; col >= 0; --col) X[1][col] = mfma_16x16x32(b3, resident[col][3], X[1][col]);
        __builtin_amdgcn_sched_barrier(0);
    } else {
        bf16x8 a0 = ds_read_b128_at<OFF>(row_addr[0]), a1 = ds_read_b128_at<OFF>(row_addr[1]);
        bf16x8 b0 = ds_read_b128_at<ROWS16>(row_addr[0]), b1 = ds_read_b128_at<ROWS16>(row_addr[1]);
        lds_wait2<2>(a0, a1);
#pragma unroll
        for (int col = 0; col < NC; ++col) X[0][col] = mfma_16x16x32(a0, resident[col][0], X[0][col]);
#pragma unroll
        for (int col = NC - 1; col >= 0; --col) X[0][col] = mfma_16x16x32(a1, resident[col][1], X[0][col]);
        __builtin_amdgcn_sched_barrier(0);
        lds_wait2<0>(b0, b1);
#pragma unroll
        for (int col = 0; col < NC; ++col) X[1][col] = mfma_16x16x32(b0, resident[col][0], X[1][col]);
#pragma unroll
        for (int col = NC - 1; col >= 0; --col) X[1][col] = mfma_16x16x32(b1, resident[col][1], X[1][col]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// acc[cb][col] (16 channels x 16 resident columns) += A B: A = the staged operand at OFF read transposed (A rows =
// channels, k = its 32 rows: index 8*g4 + i is row 4*g4 + i of the first 16 for i < 4, of the second 16 otherwise),
// B = packed[col].  The reads of the first group of channel blocks can go out before B exists.
template <int D, int OFF, int AT_ONCE = 4>
struct StagedTransposedProduct {
    static constexpr int CB = D / 16;                   // channel blocks: read AT_ONCE at a time
    static constexpr int NG = CB / AT_ONCE;
    shortx4 frag[NG][AT_ONCE][2];
    template <int G>
    __device__ __forceinline__ void issue(const uint32_t (&tr_addr)[4])
    {
        static_for<0, AT_ONCE>([&](auto i) {
            constexpr int cb = AT_ONCE * G + decltype(i)::value;
            constexpr int at = OFF + Staged<D>::tr_offset(cb);
            frag[G][cb % AT_ONCE][0] = ds_read_tr16<at>(tr_addr[Staged<D>::tr_index(cb)]);
            frag[G][cb % AT_ONCE][1] = ds_read_tr16<at + Staged<D>::Rows16>(tr_addr[Staged<D>::tr_index(cb)]);
        });
    }
    __device__ __forceinline__ void prefetch(const uint32_t (&tr_addr)[4]) { issue<0>(tr_addr); }
    template <int NC>
    __device__ __forceinline__ void run(const uint32_t (&tr_addr)[4], const bf16x8 (&packed)[NC], floatx4 (&acc)[CB][NC])
    {
        typedef short shortx8 __attribute__((ext_vector_type(8)));
        static_for<0, NG>([&](auto gi) {
            constexpr int g = decltype(gi)::value;
            if constexpr (g + 1 < NG) {
                issue<g + 1>(tr_addr);
                pv_wait<2 * AT_ONCE>(frag[g]);
            } else {
                pv_wait<0>(frag[g]);
            }
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) {
                const shortx8 a = __builtin_shufflevector(frag[g][i][0], frag[g][i][1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int t = 0; t < NC; ++t) {
                    const int col = (i & 1) ? NC - 1 - t : t;
                    acc[AT_ONCE * g + i][col] = mfma_16x16x32(__builtin_bit_cast(bf16x8, a), packed[col], acc[AT_ONCE * g + i][col]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    }
};

}  // namespace

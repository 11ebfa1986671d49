// Gradients of Sliding Tile Attention for gfx950 (MI355X): dQ, dK, dV of Eq. 1 under the STA mask, for the
// finetuning use of the paper (Sec. 3.2 trains through STA layers).  The paper gives no backward kernel; this
// is the chain rule of Eq. 1 evaluated block by block over the kept (query tile, key tile) pairs only:
//
//   P_ij  = exp(S_ij - lse_i)          S = Q K^T * scale, lse_i = ln sum_j exp(S_ij) from the forward pass
//   dV_j  = sum_i P_ij dO_i
//   dP_ij = dO_i . V_j
//   dS_ij = P_ij (dP_ij - delta_i)     delta_i = dO_i . O_i
//   dQ_i  = scale * sum_j dS_ij K_j    dK_j = scale * sum_i dS_ij Q_i
//
// Two kernels, no atomics, results repeatable:
//   sta_bwd_dq_kernel     one workgroup per query block, walks the key tiles of its window (as the forward
//                         kernel does): 3 MFMA products per block (K Q^T, V dO^T, K^T dS^T); it also forms
//                         -delta_i and -lse_i / scale of its queries and leaves them for the second kernel;
//   sta_bwd_dkv_kernel    one wave per 32 keys, walks the QUERY tiles that keep its key tile (the
//                         transposed box): 4 MFMA products per block (Q K^T, dO V^T, dO^T P, Q^T dS);
//   sta_bwd_dkv_pair_kernel   the same with the products split over pairs of waves (head dimension 128: tiles of 96 and 32 tokens'
//                         multiples, short walks on other multiples of 64, one full round of equal walks on multiples of 384).
// S and dP are thus computed twice (7 products against the 5 of a single-pass scheme with atomics on dQ).
//
// Same MFMA formulation as the forward kernel (v_mfma_f32_16x16x32_bf16, the shape that costs the least energy per
// flop on this power-limited chip): the block is held so that one lane owns one column (a query in the dQ kernel,
// a key in the dK/dV kernel), and the bf16-rounded P or dS goes from the accumulators straight into the B operand
// of the next product, the contraction index being fed in accumulator order.  Staged operands are brought in by
// global_load_lds; an operand may be read both by rows (A rows = tokens, 16-byte reads) and transposed (A rows =
// channels, ds_read_b64_tr_b16), and one LDS layout serves both without bank conflicts (described where the two
// products are defined).
// All kernels: any tile of a multiple of 32 tokens.  A workgroup's columns are the largest of a few sizes that divides the
// tile; launches too small for the chip are cut into walk groups (see WalkShare), the smallest ones into four groups of one
// wave each, or eight, which has its LDS to itself and passes no barrier until the groups are summed.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sta_device_util.h"
#include "sta_geometry.h"
#include "sta_internal.h"
#include "sta_staged.h"

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// How the column blocks (queries or keys) of one launch are dealt to the workgroups, with every division prepared.
struct BwdPlan {
    sta::Deal deal;            // of the column blocks
    sta::FastDiv per_row;      // blocks of one row of tiles along w
    sta::FastDiv rows;         // such rows of one (batch, head)
    sta::FastDiv slices;       // (batch, head) pairs
    sta::FastDiv per_tile;     // blocks of one tile
    sta::FastDiv n_h, batch;
    uint32_t row_major;        // the same row of every (batch, head), then the next row; otherwise head after head
    uint32_t longest_first;    // ... in the order of visit_order along t and h
    sta::FastDiv sub_per_tile; // 32-token sub-blocks of a tile
    float inv_scale;           // 1 / softmax scale
    struct Head {
        uint16_t h, w[3];      // head inside the launch, its window in tiles; most expensive head first
    } head[sta::kMaxHeadsPerLaunch];
};

// The i-th tile to visit along an axis of n tiles with window w.  At window 2 * half + 1 the tiles 2 * half and n - 1 - 2 * half
// are kept by the most query tiles (3 * half + 1) and the border tiles by the fewest (half + 1): the order starts at the
// former and ends with the border, so that the last items of a launch are short ones.
__device__ __forceinline__ int visit_order(int n, int w, int i)
{
    const int first = 2 * (w >> 1);
    if (first >= n - 1) return i;
    return i + first < n ? i + first : n - 1 - i;
}

// Work item of a workgroup.  The hardware deals workgroup ids round-robin over the 8 XCDs (each with its own
// L2).  The launch's column blocks, taken row of tiles after row of tiles, are dealt to the XCDs by whole rows in
// turn, the rows left over evenly (see Deal and deal_blocks): the blocks resident on one XCD at a time are then neighbours that
// share most of their windows, while all XCDs together still work on one region of one head.
// QUERY_COLS: the columns are queries and the box holds the key tiles of their tile; otherwise the columns are keys and
// the box holds the query tiles that keep their tile.
struct BwdItem {
    uint32_t block;            // column block inside the head
    size_t bh;
    StaBox box;
};
template <bool QUERY_COLS>
__device__ __forceinline__ BwdItem bwd_item_of(uint32_t id, const sta::FwdParams &p, const BwdPlan &plan)
{
    BwdItem it;
    const uint32_t linear = sta::dealt_item(id, plan.deal);
    const uint32_t line = fast_div(linear, plan.per_row), pos = linear - line * plan.per_row.d;
    uint32_t row, rank;
    if (plan.row_major) {
        row = fast_div(line, plan.slices);
        rank = line - row * plan.slices.d;
    } else {
        rank = fast_div(line, plan.rows);
        row = line - rank * plan.rows.d;
    }
    const uint32_t head_rank = fast_div(rank, plan.batch);          // batch entries of one head are adjacent
    const BwdPlan::Head head = plan.head[head_rank];
    it.bh = (size_t)(rank - head_rank * plan.batch.d) * p.H + p.head_base + head.h;
    const uint32_t w = fast_div(pos, plan.per_tile);
    const uint32_t sub = pos - w * plan.per_tile.d;
    uint32_t t = fast_div(row, plan.n_h), h = row - t * plan.n_h.d;
    if constexpr (QUERY_COLS) {
        it.box.t = sta_axis_range(p.n_t, head.w[0], t);
        it.box.h = sta_axis_range(p.n_h, head.w[1], h);
        it.box.w = sta_axis_range(p.n_w, head.w[2], w);
    } else {
        if (plan.longest_first) {
            t = visit_order(p.n_t, head.w[0], t);
            h = visit_order(p.n_h, head.w[1], h);
        }
        it.box.t = sta_axis_query_range(p.n_t, head.w[0], t);
        it.box.h = sta_axis_query_range(p.n_h, head.w[1], h);
        it.box.w = sta_axis_query_range(p.n_w, head.w[2], w);
    }
    it.block = ((t * p.n_h + h) * p.n_w + w) * plan.per_tile.d + sub;
    return it;
}

// A walk group's share of an item's walk, in sub-blocks: group g of G takes [n * g / G, n * (g + 1) / G).  The groups of a
// workgroup hold the same columns, have LDS stages of their own and are summed through LDS at the end.
template <int G>
struct WalkShare {
    BoxWalk walk;
    int n_units, n_steps;      // this group's sub-blocks; the largest share of any group (all groups pass the same barriers)
    __device__ __forceinline__ void start(const StaBox &box, const sta::FwdParams &p, const BwdPlan &plan, int group)
    {
        walk.start(box, p.n_h, p.n_w, p.P);
        const int n_all = box.count() * walk.sub_per_tile;
        n_steps = (n_all + G - 1) / G;
        n_units = n_all;
        if constexpr (G > 1) {
            const int lo = n_all * group / G;
            n_units = n_all * (group + 1) / G - lo;
            const uint32_t tiles = fast_div((uint32_t)lo, plan.sub_per_tile);
            walk.skip(tiles, (uint32_t)lo - tiles * plan.sub_per_tile.d);
        }
    }
};

// Sums the accumulators of the walk groups into group 0, in a fixed order: the upper half of the remaining groups hands
// its accumulators to the lower half through LDS until one is left.  WAVES: waves per group, wave: index inside it.
// Every wave of the workgroup calls this; all LDS reads of the stages are over when it starts to write.
template <int G, int WAVES, int CB>
__device__ __forceinline__ void merge_groups(char *smem, int group, int wave, int lane, floatx4 (&acc)[CB][2])
{
    constexpr int PART = CB * 2 * 1024;
    __syncthreads();
#pragma unroll
    for (int n = G; n > 1; n = (n + 1) / 2) {
        const int half = (n + 1) / 2;                           // groups half .. n-1 give, groups 0 .. n-1-half take
        if (n != G) __syncthreads();                            // the previous round has been read
        if (group >= half && group < n) {
            char *to = smem + ((group - half) * WAVES + wave) * PART + lane * 16;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int col = 0; col < 2; ++col) *reinterpret_cast<floatx4 *>(to + (cb * 2 + col) * 1024) = acc[cb][col];
        }
        __syncthreads();
        if (group + half < n) {
            const char *from = smem + (group * WAVES + wave) * PART + lane * 16;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int col = 0; col < 2; ++col) acc[cb][col] += *reinterpret_cast<const floatx4 *>(from + (cb * 2 + col) * 1024);
        }
    }
    __syncthreads();
}

// The same for groups of one wave each, all of them at work: every wave leaves its accumulators in its own part of LDS
// (REGION bytes apart), sums the groups' parts of its share of the 16x16 blocks in ascending order and puts the result,
// scaled and rounded, where the rows are assembled; then the rows leave 16 bytes per lane.  DMA into the regions is over.
template <int D, int G, int REGION>
__device__ __forceinline__ void merge_waves(char *smem, char *rows, int group, int lane, const floatx4 (&acc)[D / 16][2], float mul)
{
    constexpr int RowB = 2 * D, BLOCKS = D / 16 * 2, SHARE = BLOCKS / G;
    static_assert(BLOCKS % G == 0 && BLOCKS * 1024 <= REGION, "a wave's accumulators fit its region");
    const int c16 = lane & 15, g4 = lane >> 4;
#pragma unroll
    for (int b = 0; b < BLOCKS; ++b) *reinterpret_cast<floatx4 *>(smem + group * REGION + b * 1024 + lane * 16) = acc[b / 2][b % 2];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < SHARE; ++j) {
        const int b = group * SHARE + j;
        floatx4 sum = *reinterpret_cast<const floatx4 *>(smem + b * 1024 + lane * 16);
#pragma unroll
        for (int g = 1; g < G; ++g) sum += *reinterpret_cast<const floatx4 *>(smem + g * REGION + b * 1024 + lane * 16);
        bf16x4 ov;
#pragma unroll
        for (int t = 0; t < 4; ++t) ov[t] = static_cast<__bf16>(sum[t] * mul);
        *reinterpret_cast<bf16x4 *>(rows + (16 * (b % 2) + c16) * RowB + (16 * (b / 2) + 4 * g4) * 2) = ov;
    }
    __syncthreads();
}
template <int D, int THREADS>
__device__ __forceinline__ void store_rows(const char *rows, bf16_raw *dst, int tid)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < 32 * 2 * D; i += THREADS * 16)
        if (i + tid * 16 < 32 * 2 * D)
            __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(rows + i + tid * 16),
                                        reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(dst) + i + tid * 16));
}

// A wave's 32 result rows (columns of its accumulators), scaled, rounded to bf16 and written as whole rows, 1 KB contiguous
// per store instruction, through a part of LDS that belongs to the wave (16 rows at a time).
template <int D>
__device__ __forceinline__ void store_columns(char *wave_lds, const floatx4 (&acc)[D / 16][2], float mul, bf16_raw *dst, int lane)
{
    using L = Staged<D>;
    constexpr int LPR = L::RowB / 16;                           // 16-byte chunks per row
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int c16 = lane & 15, g4 = lane >> 4;
#pragma unroll
    for (int col = 0; col < 2; ++col) {
        // acc[cb][col][i] = channel 16*cb + 4*g4 + i of row 16*col + c16
#pragma unroll
        for (int cb = 0; cb < L::CB; ++cb) {
            bf16x4 ov;
#pragma unroll
            for (int t = 0; t < 4; ++t) ov[t] = static_cast<__bf16>(acc[cb][col][t] * mul);
            const int chunk = 2 * cb + (g4 >> 1);
            *reinterpret_cast<bf16x4 *>(wave_lds + c16 * L::RowB + ((chunk ^ (c16 & (LPR - 1))) << 4) + 8 * (g4 & 1)) = ov;
        }
        char *out = reinterpret_cast<char *>(dst + (size_t)(16 * col) * D);
#pragma unroll
        for (int i = 0; i < 16 / L::GroupRows; ++i) {
            const int r = L::GroupRows * i + lane / LPR, cpos = lane % LPR;
            const u32x4 x = *reinterpret_cast<const u32x4 *>(wave_lds + r * L::RowB + ((cpos ^ (r & (LPR - 1))) << 4));
            __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(out + (size_t)r * L::RowB + (cpos << 4)));
        }
    }
}

constexpr int max_of(int a, int b) { return a > b ? a : b; }

// ---------------------------------------------------------------------------------------------------------
// dQ.  One workgroup of QW waves per 32 * QW queries (times G walk groups); a lane holds query column c16 of its wave's two
// 16-query blocks.  At head dimension 128 206-210 registers, two waves per SIMD; at 64 128 and four (8 bytes of scratch in the
// shape of three waves and two walk groups; the
// statistic enters the exponent by a fused multiply-add instead of occupying eight registers of initial values, and the
// transposed fragments are read two channel blocks at a time; three waves per SIMD before: 32 heads of a 64x64 image 42.7 ->
// 37.7 us, 128 heads 165 -> 147, 12x48x48 x 4 156 -> 148, 30x48x80 x 24 9.11 -> 8.89 ms).  LDS stage: K (read by rows and
// transposed) and V (read by rows), in the layout described above.  Per wave and 32-key sub-block: S^T = K Q^T - lse / scale
// and dP^T = V dO^T - delta (the statistics of the lane's query as the initial value, so that neither a subtraction nor a
// fused multiply-add per element is left), dS^T = 2^(c S^T) o dP^T, dQ^T += K^T dS^T; 16 matrix instructions each at head
// dimension 128, 8 at 64.
// SOLO (a single wave in each walk group, or alone beyond a round of them): as in the dK/dV kernel the stage belongs to one wave, which refills V as
// soon as dP is formed and K after its last product.  One buffer for each instead of two: eight groups at head dimension 128 then take the 140 KB of
// LDS that four take with two, and a CU holds two workgroups of four groups (four at 64) where it holds one (two) with two.  The wave waits longer
// for a buffer that it has just emptied, so four groups keep two where the launch has no workgroup that does not find its place.  Gradients alone,
// 220 drawn launches, one buffer's time over that of two: up to 256 waves of columns, walks below 40, 128 1.015, 64 1.011; 64 up to 512 waves
// 1.012; beyond those 128 0.91, 64 0.96.
// Without groups (tiles of 32 tokens' multiples) a CU holds eight such waves at head dimension 128 and sixteen at 64, with two buffers four and
// nine: `one_buffer_alone` says which take it.
// The row statistics are formed here, from the dO fragments the wave holds anyway and the same fragments of O, and written
// for the dK/dV kernel (a kernel of their own for them read dO once more: 6.8 us of a 345 us training step at 16,384 tokens
// x 8 heads of dimension 64, 0.23 ms of 53 ms at 115,200 x 24 of 128).
// ---------------------------------------------------------------------------------------------------------
template <int D, int QW, int G, bool DMA, bool SOLO>
__global__ __attribute__((amdgpu_flat_work_group_size(QW * G * 64, QW * G * 64), amdgpu_waves_per_eu(SOLO && G == 1 ? (D == 64 ? 4 : 2) : QW == 1 ? (D == 64 || G == 8 ? 2 : 1) : (D == 64 ? 4 : 2))))
void sta_bwd_dq_kernel(const bf16_raw *__restrict__ q, const bf16_raw *__restrict__ k, const bf16_raw *__restrict__ v,
                       const bf16_raw *__restrict__ o, const bf16_raw *__restrict__ d_o, const float *__restrict__ lse,
                       float *__restrict__ neg_delta, float *__restrict__ neg_lse, bf16_raw *__restrict__ d_q,
                       sta::FwdParams p, BwdPlan plan)
{
    using L = Staged<D>;
    constexpr int KS = L::KS, CB = L::CB;
    constexpr int COLS = QW * 32;                       // queries per workgroup
    constexpr int STAGE_B = 2 * L::Tile;
    constexpr int K_TILE = 0, V_TILE = L::Tile;
    static_assert(!SOLO || (QW == 1 && DMA), "SOLO: a wave with a stage of its own, no barriers, single buffers");
    constexpr int GROUP_B = SOLO ? STAGE_B : 2 * STAGE_B;       // LDS of one walk group
    constexpr int OPS = 2 * L::Groups;                  // DMA instructions per sub-block
    constexpr int WAVE_OPS = (OPS + QW - 1) / QW;       // at most this many per wave
    constexpr int WAVE_OUT = 16 * L::RowB;
    constexpr int SMEM = QW == 1 && G > 1 ? G * GROUP_B + 32 * L::RowB
                                          : max_of(G * GROUP_B, max_of((G / 2) * QW * CB * 2 * 1024, QW * WAVE_OUT));
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];

    const BwdItem item = bwd_item_of<true>(blockIdx.x, p, plan);
    const size_t bh = item.bh;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave / QW, qw = wave % QW;
    const int lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;

    const size_t my_row = bh * p.N + (size_t)item.block * COLS + (size_t)qw * 32;
    const char *kh = reinterpret_cast<const char *>(k + bh * p.N * D);
    const char *vh = reinterpret_cast<const char *>(v + bh * p.N * D);

    WalkShare<G> share;
    share.start(item.box, p, plan, group);

    // DMA: each operand is L::Groups instructions of 1 KB; wave qw of the group issues the instructions qw, qw + QW, ..
    const uint32_t src_lane_off = L::dma_lane_offset(lane);
    int issued = 0;
    auto issue_next = [&]() __attribute__((always_inline)) {
        if (issued >= share.n_units) return;
        uint32_t off = src_lane_off;
        asm volatile("" : "+v"(off));                   // keep the lane offset 32-bit next to a scalar base
        const uint32_t first_row = share.walk.next_row;
        share.walk.advance();
        char *stage = smem + group * GROUP_B + (issued & 1) * STAGE_B;
#pragma unroll
        for (int i = 0; i < WAVE_OPS; ++i) {
            const int j = qw + i * QW;
            if (OPS % QW == 0 || j < OPS) {
                const bool is_v = j >= L::Groups;
                const int part = j % L::Groups;
                const char *src = (is_v ? vh : kh) + (size_t)(first_row + L::GroupRows * part) * L::RowB;
                stage_group<DMA>(src + off, stage + (is_v ? V_TILE : K_TILE) + part * L::Group, lane);
            }
        }
        ++issued;
    };
    auto issue_operand = [&](auto is_v_c, uint32_t row) __attribute__((always_inline)) {     // single buffers
        constexpr bool IS_V = decltype(is_v_c)::value;
        uint32_t off = src_lane_off;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int j = 0; j < L::Groups; ++j)
            stage_group<DMA>((IS_V ? vh : kh) + (size_t)(row + L::GroupRows * j) * L::RowB + off,
                             smem + group * GROUP_B + (IS_V ? V_TILE : K_TILE) + j * L::Group, lane);
    };
    if constexpr (SOLO) {
        if (share.n_units > 0) {
            issue_operand(std::true_type{}, share.walk.next_row);
            issue_operand(std::false_type{}, share.walk.next_row);
        }
    } else {
        issue_next();
    }

    uint32_t row_addr[KS], tr_addr[4];
    L::addresses((uint32_t)(uintptr_t)smem + (uint32_t)(group * GROUP_B), lane, row_addr, tr_addr);

    // resident B fragments: query 16*qb + c16, channels 32*ks + 8*g4 ..
    bf16x8 Qr[2][KS], Gr[2][KS];
    float delta[2] = {0.f, 0.f};
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const size_t at = (my_row + 16 * qb + c16) * D + ks * 32 + g4 * 8;
            Qr[qb][ks] = *reinterpret_cast<const bf16x8 *>(q + at);
            Gr[qb][ks] = *reinterpret_cast<const bf16x8 *>(d_o + at);
            const bf16x8 out = *reinterpret_cast<const bf16x8 *>(o + at);
#pragma unroll
            for (int e = 0; e < 8; ++e) delta[qb] = fmaf(static_cast<float>(out[e]), static_cast<float>(Gr[qb][ks][e]), delta[qb]);
        }
    const float c = p.scale_log2e;
    // a lane owns one query column per block: the four registers of an accumulator all start at that query's statistic
    floatx4 s_init[2], dp_init[2];
    float exp_init[2];                                  // head dimension 64: added to the exponents in base 2 instead of s_init
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const size_t row = my_row + 16 * qb + c16;
        const float a = -lse[row] * plan.inv_scale, d = -quad_lane_sum(delta[qb]);
        s_init[qb] = D == 64 ? floatx4{0.f, 0.f, 0.f, 0.f} : floatx4{a, a, a, a};
        exp_init[qb] = a * c;
        dp_init[qb] = floatx4{d, d, d, d};
        if (group == 0 && g4 == 0) {
            neg_lse[row] = a;
            neg_delta[row] = d;
        }
    }

    floatx4 dQ[CB][2];                                  // [channel block][query block]
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) dQ[cb][qb] = floatx4{0.f, 0.f, 0.f, 0.f};

    auto start_at_statistics = [&](floatx4 (&S)[2][2], floatx4 (&dP)[2][2]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                S[kb][qb] = s_init[qb];
                dP[kb][qb] = dp_init[qb];
            }
    };
    // An element of dS^T, rounded to bf16; eight of a column are the B operand of the last product: k index 8*g4 + i is key 4*g4 + i of
    // the first key block (i < 4) or of the second.  The stages of one buffer form it by a function of whole blocks, those of two in place:
    // the compiler then takes the exponentials in another order.  Gradients at head dimension 64, two buffers by the function and in place:
    // two groups, 720 waves of 600 438, 429 us, three waves a workgroup 0.995 in the mean of 43 launches; eight groups, one buffer, in place 1.005.
    auto ds_of = [&](float s, float dp, int qb) __attribute__((always_inline)) {
        const float x = D == 64 ? fmaf(s, c, exp_init[qb]) : s * c;
        return static_cast<__bf16>(__builtin_amdgcn_exp2f(x) * dp);
    };
    auto products = [&](const floatx4 (&S)[2][2], const floatx4 (&dP)[2][2], bf16x8 (&dSb)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int e = 0; e < 4; ++e) dSb[qb][4 * kb + e] = ds_of(S[kb][qb][e], dP[kb][qb][e], qb);
    };
    auto sub_block = [&](auto stage_c, int unit) __attribute__((always_inline)) {
        constexpr int ST = decltype(stage_c)::value * STAGE_B;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // (the stages of a single wave are its own; operands staged by plain stores have to be waited for)
        if constexpr (QW > 1 || !DMA) __syncthreads();
        issue_next();
        if (G > 1 && unit >= share.n_units) return;
        floatx4 S[2][2], dP[2][2];                      // [key block][query block]
        start_at_statistics(S, dP);
        staged_rows_times_resident<D, ST + K_TILE>(row_addr, Qr, S);    // K Q^T - lse / scale (128), K Q^T (64)
        staged_rows_times_resident<D, ST + V_TILE>(row_addr, Gr, dP);   // V dO^T - delta
        StagedTransposedProduct<D, ST + K_TILE, D == 64 ? 2 : 4> k_t;
        k_t.prefetch(tr_addr);
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 dSb[2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int e = 0; e < 4; ++e) dSb[qb][4 * kb + e] = ds_of(S[kb][qb][e], dP[kb][qb][e], qb);
        k_t.run(tr_addr, dSb, dQ);                                       // dQ^T += K^T dS^T
    };
    if constexpr (SOLO) {
#pragma unroll 1
        for (int u = 0; u < share.n_units; ++u) {
            const bool more = u + 1 < share.n_units;
            floatx4 S[2][2], dP[2][2];
            bf16x8 dSb[2];
            start_at_statistics(S, dP);
            wait_dma<L::Groups>();                                        // V; K has been requested behind it
            staged_rows_times_resident<D, V_TILE>(row_addr, Gr, dP);
            share.walk.advance();
            if (more) {
                issue_operand(std::true_type{}, share.walk.next_row);
                wait_dma<L::Groups>();                                    // K; the next V has been requested behind it
            } else {
                wait_dma<0>();
            }
            staged_rows_times_resident<D, K_TILE>(row_addr, Qr, S);
            StagedTransposedProduct<D, K_TILE, D == 64 ? 2 : 4> k_t;
            k_t.prefetch(tr_addr);
            __builtin_amdgcn_sched_barrier(0);
            products(S, dP, dSb);
            k_t.run(tr_addr, dSb, dQ);
            if (more) issue_operand(std::false_type{}, share.walk.next_row);
        }
    } else {
        for (int u = 0; u < share.n_steps; u += 2) {
            sub_block(std::integral_constant<int, 0>{}, u);
            if (u + 1 < share.n_steps) sub_block(std::integral_constant<int, 1>{}, u + 1);
        }
    }
    if constexpr (QW == 1 && G > 1) {
        char *rows = smem + G * GROUP_B;
        merge_waves<D, G, GROUP_B>(smem, rows, group, lane, dQ, c * kLn2);
        store_rows<D, G * 64>(rows, d_q + my_row * D, tid);
        return;
    } else if constexpr (G > 1) {
        merge_groups<G, QW>(smem, group, qw, lane, dQ);
        if (group != 0) return;
    } else {
        __syncthreads();                                // every wave has finished reading the stages
    }
    store_columns<D>(smem + qw * WAVE_OUT, dQ, c * kLn2, d_q + my_row * D, lane);
}

// ---------------------------------------------------------------------------------------------------------
// dK, dV.  One workgroup of NW waves per 32 * NW keys (times G walk groups); a wave holds K and V of its 32 keys, accumulates
// dK and dV and forms all four products, S = Q K^T, dV^T += dO^T P, dP = dO V^T, dK^T += Q^T dS, in this order: P stays in
// registers in fp32 and no other wave is waited for.  At head dimension 64 158 registers, three waves per SIMD; at 128 all 256
// that two waves per SIMD allow (128 accumulator, 64 resident operand; 20 bytes of scratch outside the loop).  Per wave and 32-query
// sub-block 64 matrix instructions at head dimension 128, 32 at 64, next to about 64 vector instructions.
// LDS stage: Q and dO (each read by rows and transposed) and the row statistics of the 32 queries, from which the accumulators of
// S and dP start.  UPS sub-blocks per stage, i.e. per barrier.
// NW = 1 ("solo", for the small launches): the stage belongs to one wave, which needs no barrier, only its own requests to have
// landed, and refills either operand as soon as it has read it: half the LDS, so that a CU holds eight such waves at head
// dimension 128 and twelve at 64 (168 registers and up to 12 bytes of scratch outside the loop, at 128 256 and up to 56; of eight groups,
// one workgroup and two waves a SIMD at either, 170 and none at 64: 0.994 of the time under the bound of three waves, which spilled 12).  There dP and dS come before the product with P, which frees dO first.
// What bounds it: matrix pipe and power on large launches (30x48x80, 24 heads, window 3x3x3, head dimension 128: 22.1 ms, 1330
// TFLOP/s; 64: 11.5 ms, 1280).  Before, each 32 keys were served by a pair of waves, one for S, P and dV, one for dP, dS and dK,
// with P handed over through LDS at a barrier of its own.  Entry point, pairs against this kernel, us: 30x48x80, 24 heads of 128
// 40,040, 38,810; of 64 21,720, 20,320; 12x24x40 in 4x8x8 tiles, 28 heads of 128 2640, 2420; 16x48x48 in 8x8x8 tiles, 48 heads
// of 128 23,215, 21,995; 16x40x120 in 4x4x8 tiles, 16 heads of 64 2825, 2585; 64x64 images in 64-token tiles, 128 heads of 64 326,
// 299.  The error of dK on tiles of 128 tokens' multiples at head dimension 128 went from 2.88e-3 to 2.35e-3 against 64 bits
// (2-norm): P had been handed over in bf16 there.
// dP before P in the shared form (as in the solo one) spills 56 bytes at head dimension 128 and is slower (24,073 against
// 21,995 us on the 8x8x8 case); two sub-blocks per stage give 0.5 to 1 % at 64 and lose as much at 128.
// A lane holds key column c16 of its wave's two 16-key blocks and the query rows 4*g4 .. 4*g4+3 of a result.
// ---------------------------------------------------------------------------------------------------------
template <int D, int NW, int G, int UPS, bool DMA>
__global__ __attribute__((amdgpu_flat_work_group_size(NW * G * 64, NW * G * 64), amdgpu_waves_per_eu(D == 64 && G < 8 ? 3 : 2)))
void sta_bwd_dkv_kernel(const bf16_raw *__restrict__ q, const bf16_raw *__restrict__ k, const bf16_raw *__restrict__ v,
                        const bf16_raw *__restrict__ d_o, const float *__restrict__ neg_lse,
                        const float *__restrict__ neg_delta, bf16_raw *__restrict__ d_k, bf16_raw *__restrict__ d_v,
                        sta::FwdParams p, BwdPlan plan)
{
    using L = Staged<D>;
    constexpr int KS = L::KS, CB = L::CB;
    constexpr bool SOLO = NW == 1 && DMA;               // a wave with a stage of its own: no barriers, single buffers
    constexpr int COLS = NW * 32;                       // keys per workgroup
    constexpr int UNIT_B = 2 * L::Tile;
    constexpr int Q_TILE = 0, G_TILE = L::Tile;
    constexpr int UNITS = SOLO ? 1 : 2 * UPS;           // sub-blocks in LDS, per walk group
    constexpr int STATS = UNITS * UNIT_B;               // per sub-block: -lse / scale then -delta of the 32 staged query rows
    constexpr int STAT_B = 2 * kSub * 4;
    constexpr int GROUP_B = STATS + UNITS * STAT_B;     // LDS of one walk group
    constexpr int OPS = 2 * L::Groups;                  // DMA instructions per sub-block: Q, dO
    constexpr int WAVE_OPS = (OPS + NW - 1) / NW;
    constexpr int WAVE_OUT = 16 * L::RowB;
    constexpr int ROWS_B = 32 * L::RowB;
    constexpr int SMEM = SOLO && G > 1 ? G * GROUP_B + ROWS_B
                                       : max_of(G * GROUP_B, max_of((G / 2) * NW * CB * 2 * 1024, NW * WAVE_OUT));
    static_assert(UPS == 1 || G == 1, "shares of a walk are counted in single units");
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];

    const BwdItem item = bwd_item_of<false>(blockIdx.x, p, plan);
    const size_t bh = item.bh;
    const int tid = threadIdx.x;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave_all / NW, wave = wave_all % NW;
    const int lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;

    const size_t head_row = bh * p.N;
    const size_t my_row = head_row + (size_t)item.block * COLS + (size_t)wave * 32;
    const char *qh = reinterpret_cast<const char *>(q + head_row * D);
    const char *gh = reinterpret_cast<const char *>(d_o + head_row * D);

    WalkShare<G> share;
    share.start(item.box, p, plan, group);

    // DMA: each operand is L::Groups instructions of 1 KB; wave w of the group issues the instructions w, w + NW, .., the last
    // wave also the one of 4 bytes per lane that brings the row statistics (32 + 32 floats).
    const uint32_t src_lane_off = L::dma_lane_offset(lane);
    const uint32_t stat_lane_off = (uint32_t)((lane & (kSub - 1)) * 4);
    const char *stat_base = reinterpret_cast<const char *>((lane < kSub ? neg_lse : neg_delta) + head_row);
    char *group_lds = smem + group * GROUP_B;
    auto issue_stats = [&](uint32_t row, int unit) __attribute__((always_inline)) {
        uint32_t soff = stat_lane_off;
        asm volatile("" : "+v"(soff));                  // keep the lane offsets 32-bit next to a scalar base
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(stat_base + (size_t)row * 4 + soff),
                                         STA_LDS_PTR(group_lds + STATS + unit * STAT_B), 4, 0, 0);
    };
    auto issue_operand = [&](auto is_g_c, uint32_t row) __attribute__((always_inline)) {     // single buffers
        constexpr bool IS_G = decltype(is_g_c)::value;
        uint32_t off = src_lane_off;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int j = 0; j < L::Groups; ++j)
            stage_group<DMA>((IS_G ? gh : qh) + (size_t)(row + L::GroupRows * j) * L::RowB + off,
                             group_lds + (IS_G ? G_TILE : Q_TILE) + j * L::Group, lane);
    };
    int issued = 0;
    auto issue_next = [&]() __attribute__((always_inline)) {
        if (issued >= share.n_units) return;
        uint32_t off = src_lane_off;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int su = 0; su < UPS; ++su) {
            const int unit = issued % (2 * UPS) + su;
            const uint32_t first_row = share.walk.next_row;
            share.walk.advance();
#pragma unroll
            for (int i = 0; i < WAVE_OPS; ++i) {
                const int j = wave + i * NW;
                if (OPS % NW == 0 || j < OPS) {
                    const bool is_g = j >= L::Groups;
                    const int part = j % L::Groups;
                    const char *src = (is_g ? gh : qh) + (size_t)(first_row + L::GroupRows * part) * L::RowB;
                    stage_group<DMA>(src + off, group_lds + unit * UNIT_B + (is_g ? G_TILE : Q_TILE) + part * L::Group, lane);
                }
            }
            if (wave == NW - 1) issue_stats(first_row, unit);
        }
        issued += UPS;
    };
    if constexpr (SOLO) {
        if (share.n_units > 0) {
            issue_stats(share.walk.next_row, 0);
            issue_operand(std::true_type{}, share.walk.next_row);
            issue_operand(std::false_type{}, share.walk.next_row);
        }
    } else {
        issue_next();
    }

    const uint32_t group_addr = (uint32_t)(uintptr_t)smem + (uint32_t)(group * GROUP_B);
    uint32_t row_addr[KS], tr_addr[4];
    L::addresses(group_addr, lane, row_addr, tr_addr);
    const uint32_t stat_addr = group_addr + STATS + 16 * g4;

    // resident B fragments: key 16*kb + c16, channels 32*ks + 8*g4 ..
    bf16x8 Kr[2][KS], Vr[2][KS];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const size_t at = (my_row + 16 * kb + c16) * D + ks * 32 + g4 * 8;
            Kr[kb][ks] = *reinterpret_cast<const bf16x8 *>(k + at);
            Vr[kb][ks] = *reinterpret_cast<const bf16x8 *>(v + at);
        }
    const float c = p.scale_log2e;

    floatx4 dV[CB][2], dK[CB][2];                       // [channel block][key block]
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            dV[cb][kb] = floatx4{0.f, 0.f, 0.f, 0.f};
            dK[cb][kb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }

    // Accumulators [query block][key block] that start at the statistics of their query rows 16*qb + 4*g4 ..
    auto start_at = [&](auto off_c, floatx4 (&X)[2][2]) __attribute__((always_inline)) {
        constexpr int OFF = decltype(off_c)::value;
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 r0, r1;
        asm volatile("ds_read_b128 %0, %2 offset:%3\n\tds_read_b128 %1, %2 offset:%4\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(r0), "=&v"(r1)
                     : "v"(stat_addr), "n"(OFF), "n"(OFF + 64));
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            X[0][kb] = __builtin_bit_cast(floatx4, r0);
            X[1][kb] = __builtin_bit_cast(floatx4, r1);
        }
    };
    // S becomes P = 2^(c S); Pb: rounded, packed as the B operand of the product over the queries
    auto probabilities = [&](floatx4 (&S)[2][2], bf16x8 (&Pb)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    S[qb][kb][e] = __builtin_amdgcn_exp2f(S[qb][kb][e] * c);
                    Pb[kb][4 * qb + e] = static_cast<__bf16>(S[qb][kb][e]);
                }
    };
    auto products = [&](const floatx4 (&P)[2][2], const floatx4 (&dP)[2][2], bf16x8 (&dSb)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                for (int e = 0; e < 4; ++e) dSb[kb][4 * qb + e] = static_cast<__bf16>(P[qb][kb][e] * dP[qb][kb][e]);
    };
    auto sub_block = [&](auto unit_c) __attribute__((always_inline)) {
        constexpr int ST = decltype(unit_c)::value * UNIT_B;
        constexpr int ST_STATS = decltype(unit_c)::value * STAT_B;
        floatx4 S[2][2], dP[2][2];                      // [query block][key block]
        bf16x8 Pb[2], dSb[2];
        start_at(std::integral_constant<int, ST_STATS>{}, S);
        staged_rows_times_resident<D, ST + Q_TILE>(row_addr, Kr, S);      // Q K^T - lse / scale
        StagedTransposedProduct<D, ST + G_TILE, 2> g_t;
        g_t.prefetch(tr_addr);
        __builtin_amdgcn_sched_barrier(0);
        probabilities(S, Pb);
        g_t.run(tr_addr, Pb, dV);                                         // dV^T += dO^T P
        start_at(std::integral_constant<int, ST_STATS + kSub * 4>{}, dP);
        staged_rows_times_resident<D, ST + G_TILE>(row_addr, Vr, dP);     // dO V^T - delta
        StagedTransposedProduct<D, ST + Q_TILE, 2> q_t;
        q_t.prefetch(tr_addr);
        __builtin_amdgcn_sched_barrier(0);
        products(S, dP, dSb);
        q_t.run(tr_addr, dSb, dK);                                        // dK^T += Q^T dS
    };
    if constexpr (SOLO) {
#pragma unroll 1
        for (int u = 0; u < share.n_units; ++u) {
            floatx4 S[2][2], dP[2][2];
            bf16x8 Pb[2], dSb[2];
            wait_dma<L::Groups>();                                        // statistics and dO; Q has been requested behind them
            start_at(std::integral_constant<int, kSub * 4>{}, dP);
            start_at(std::integral_constant<int, 0>{}, S);
            staged_rows_times_resident<D, G_TILE>(row_addr, Vr, dP);      // dO V^T - delta
            wait_dma<0>();
            staged_rows_times_resident<D, Q_TILE>(row_addr, Kr, S);       // Q K^T - lse / scale
            StagedTransposedProduct<D, G_TILE, 2> g_t;
            g_t.prefetch(tr_addr);
            __builtin_amdgcn_sched_barrier(0);
            probabilities(S, Pb);
            products(S, dP, dSb);
            g_t.run(tr_addr, Pb, dV);                                     // dV^T += dO^T P
            share.walk.advance();
            if (u + 1 < share.n_units) {
                issue_stats(share.walk.next_row, 0);
                issue_operand(std::true_type{}, share.walk.next_row);
            }
            StagedTransposedProduct<D, Q_TILE, 2> q_t;
            q_t.prefetch(tr_addr);
            q_t.run(tr_addr, dSb, dK);                                    // dK^T += Q^T dS
            if (u + 1 < share.n_units) issue_operand(std::false_type{}, share.walk.next_row);
        }
    } else {
        auto next_stage = [&]() __attribute__((always_inline)) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            issue_next();
        };
        for (int u = 0; u < share.n_steps; u += 2 * UPS) {
            next_stage();
            if (G == 1 || u < share.n_units) sub_block(std::integral_constant<int, 0>{});
            if constexpr (UPS == 2) sub_block(std::integral_constant<int, 1>{});
            if (u + UPS < share.n_steps) {
                next_stage();
                if (G == 1 || u + UPS < share.n_units) sub_block(std::integral_constant<int, UPS>{});
                if constexpr (UPS == 2) sub_block(std::integral_constant<int, UPS + 1>{});
            }
        }
    }
    if constexpr (SOLO && G > 1) {
        char *rows = smem + G * GROUP_B;
        merge_waves<D, G, GROUP_B>(smem, rows, group, lane, dV, 1.0f);
        store_rows<D, G * 64>(rows, d_v + my_row * D, tid);
        merge_waves<D, G, GROUP_B>(smem, rows, group, lane, dK, c * kLn2);
        store_rows<D, G * 64>(rows, d_k + my_row * D, tid);
        return;
    } else if constexpr (G > 1) {
        merge_groups<G, NW>(smem, group, wave, lane, dV);
        merge_groups<G, NW>(smem, group, wave, lane, dK);
        if (group != 0) return;
    } else {
        __syncthreads();                                // every wave has finished reading the stages
    }
    store_columns<D>(smem + wave * WAVE_OUT, dV, 1.0f, d_v + my_row * D, lane);
    store_columns<D>(smem + wave * WAVE_OUT, dK, c * kLn2, d_k + my_row * D, lane);
}

// ---------------------------------------------------------------------------------------------------------
// dK, dV at head dimension 128 on tiles of 96 and 32 tokens' multiples, and where the shapes above would half fill the chip.  One
// workgroup of 2 * NPAIR waves per 32 * NPAIR keys (times G walk groups).  Each 32-key column block is served by a PAIR of waves: the first holds K and accumulates dV (S = Q K^T,
// P, dV^T += dO^T P), the second holds V and accumulates dK (dP = dO V^T, dS = P o (dP - delta), dK^T += Q^T dS).  P goes from the
// first to the second through LDS in fp32.  165-172 registers, three waves per SIMD: on these tiles the two waves per SIMD of
// the kernel above do not fill the CU (three waves of 96 keys leave every fourth place empty) or need more LDS than there is
// (one wave of 32).  Entry point, this kernel against the other, us: 10x30x56 in 96-token tiles, window 3x3x3, four slices
// 356, 373, eight 643, 659, forty 3346, 3346; window 1x3x3, four 147, 153; 32x64 images in 32-token tiles, 16 heads 37, 47, 64
// heads 127, 150.
// A lane holds key column c16 of its wave's two 16-key blocks and the query rows 4*g4 .. 4*g4+3 of a result.
// ---------------------------------------------------------------------------------------------------------
template <int NPAIR, int G, bool DMA>
__global__ __attribute__((amdgpu_flat_work_group_size(NPAIR * G * 128, NPAIR * G * 128), amdgpu_waves_per_eu(NPAIR == 1 ? 2 : 3)))
void sta_bwd_dkv_pair_kernel(const bf16_raw *__restrict__ q, const bf16_raw *__restrict__ k, const bf16_raw *__restrict__ v,
                        const bf16_raw *__restrict__ d_o, const float *__restrict__ neg_lse,
                        const float *__restrict__ neg_delta, bf16_raw *__restrict__ d_k, bf16_raw *__restrict__ d_v,
                        sta::FwdParams p, BwdPlan plan)
{
    constexpr int D = 128;
    using L = Staged<D>;
    constexpr int KS = L::KS, CB = L::CB;
    constexpr int COLS = NPAIR * 32;                    // keys per workgroup
    constexpr int WAVES = 2 * NPAIR;                    // per walk group
    constexpr int STAGE_B = 2 * L::Tile;
    constexpr int Q_TILE = 0, G_TILE = L::Tile;
    constexpr int P_XCHG = 2 * STAGE_B;                 // per pair: planes of 64 lanes x 16 B, one per key and query block
    constexpr int PAIR_B = 4096;
    constexpr int STATS = P_XCHG + NPAIR * PAIR_B;      // per stage: -lse / scale then -delta of the 32 staged query rows
    constexpr int STAT_B = 2 * kSub * 4;
    constexpr int GROUP_B = STATS + 2 * STAT_B;         // LDS of one walk group
    constexpr int OPS = 2 * L::Groups;                  // DMA instructions per sub-block: Q, dO
    constexpr int LOADERS = WAVES > 8 ? 8 : WAVES;      // waves that issue them, at most WAVE_OPS each
    constexpr int WAVE_OPS = (OPS + LOADERS - 1) / LOADERS;
    constexpr int STAT_WAVE = WAVES > LOADERS ? LOADERS : WAVES - 1;       // brings the row statistics
    constexpr int WAVE_OUT = 16 * L::RowB;
    constexpr int SMEM = max_of(G * GROUP_B, max_of((G / 2) * WAVES * CB * 2 * 1024, WAVES * WAVE_OUT));
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];

    const BwdItem item = bwd_item_of<false>(blockIdx.x, p, plan);
    const size_t bh = item.bh;
    const int tid = threadIdx.x;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave_all / WAVES, wave = wave_all % WAVES;
    const int lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;
    const bool probs_role = wave < NPAIR;               // S, P, dV; the other role: dP, dS, dK
    const int pair = probs_role ? wave : wave - NPAIR;

    const size_t head_row = bh * p.N;
    const size_t my_row = head_row + (size_t)item.block * COLS + (size_t)pair * 32;
    const char *qh = reinterpret_cast<const char *>(q + head_row * D);
    const char *gh = reinterpret_cast<const char *>(d_o + head_row * D);

    WalkShare<G> share;
    share.start(item.box, p, plan, group);

    // DMA: each operand is L::Groups instructions of 1 KB; wave w of the group issues the instructions w, w + LOADERS, ..
    // The row statistics of the sub-block (32 + 32 floats) are one of 4 bytes per lane.  (Dealt to all twelve waves of six
    // pairs, one or two each: 30x48x80, 24 heads, window 3x3x3 43.3 against 43.0 ms, 1x3x3 14.93, 14.82.)
    const uint32_t src_lane_off = L::dma_lane_offset(lane);
    const uint32_t stat_lane_off = (uint32_t)((lane & (kSub - 1)) * 4);
    const char *stat_base = reinterpret_cast<const char *>((lane < kSub ? neg_lse : neg_delta) + head_row);
    char *group_lds = smem + group * GROUP_B;
    int issued = 0;
    auto issue_next = [&]() __attribute__((always_inline)) {
        if (issued >= share.n_units) return;
        uint32_t off = src_lane_off, soff = stat_lane_off;
        asm volatile("" : "+v"(off), "+v"(soff));       // keep the lane offsets 32-bit next to a scalar base
        const uint32_t first_row = share.walk.next_row;
        share.walk.advance();
        const int stage = issued & 1;
#pragma unroll
        for (int i = 0; i < WAVE_OPS; ++i) {
            const int j = wave + i * LOADERS;
            if (wave < LOADERS && (OPS % LOADERS == 0 || j < OPS)) {
                const bool is_g = j >= L::Groups;
                const int part = j % L::Groups;
                const char *src = (is_g ? gh : qh) + (size_t)(first_row + L::GroupRows * part) * L::RowB;
                stage_group<DMA>(src + off, group_lds + stage * STAGE_B + (is_g ? G_TILE : Q_TILE) + part * L::Group, lane);
            }
        }
        if (wave == STAT_WAVE)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(stat_base + (size_t)first_row * 4 + soff),
                STA_LDS_PTR(group_lds + STATS + stage * STAT_B), 4, 0, 0);
        ++issued;
    };
    issue_next();

    const uint32_t group_addr = (uint32_t)(uintptr_t)smem + (uint32_t)(group * GROUP_B);
    uint32_t row_addr[KS], tr_addr[4];
    L::addresses(group_addr, lane, row_addr, tr_addr);
    const uint32_t xchg_addr = group_addr + P_XCHG + pair * PAIR_B + lane * 16;
    const uint32_t stat_addr = group_addr + STATS + (probs_role ? 0 : kSub * 4) + 16 * g4;

    // resident B fragments: K rows (first role) or V rows (second role) of key 16*kb + c16, channels 32*ks + 8*g4 ..
    bf16x8 resident[2][KS];
    {
        const bf16_raw *rows = (probs_role ? k : v) + my_row * D;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                resident[kb][ks] = *reinterpret_cast<const bf16x8 *>(rows + (size_t)(16 * kb + c16) * D + ks * 32 + g4 * 8);
    }
    const float c = p.scale_log2e;

    floatx4 acc[CB][2];                                 // dV^T (first role) or dK^T (second role): [channel block][key block]
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) acc[cb][kb] = floatx4{0.f, 0.f, 0.f, 0.f};

    // One sub-block in one role.  (The role is a compile-time argument and each role has its own loop: with the
    // branch inside a common loop the register allocator serves both paths at once and spills.)
    auto sub_block = [&](auto role_c, auto stage_c, int unit) __attribute__((always_inline)) {
        constexpr bool PROBS = decltype(role_c)::value;
        constexpr int ST = decltype(stage_c)::value * STAGE_B;
        constexpr int ST_STATS = decltype(stage_c)::value * STAT_B;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();       // the stage is complete; the other stage and the exchange buffer are free
        issue_next();
        if (G > 1 && unit >= share.n_units) {
            __builtin_amdgcn_s_barrier();               // the one at the hand-over below
            return;
        }
        // the accumulators of the first product start at the statistics of their query rows 16*qb + 4*g4 ..
        floatx4 init[2];
        {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            u32x4 r0, r1;
            asm volatile("ds_read_b128 %0, %2 offset:%3\n\tds_read_b128 %1, %2 offset:%4\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(r0), "=&v"(r1)
                         : "v"(stat_addr), "n"(ST_STATS), "n"(ST_STATS + 64));
            init[0] = __builtin_bit_cast(floatx4, r0);
            init[1] = __builtin_bit_cast(floatx4, r1);
        }
        floatx4 X[2][2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) X[qb][kb] = init[qb];
        if constexpr (PROBS) {
            staged_rows_times_resident<D, ST + Q_TILE>(row_addr, resident, X);      // Q K^T - lse / scale
            StagedTransposedProduct<D, ST + G_TILE> g_t;
            g_t.prefetch(tr_addr);
            __builtin_amdgcn_sched_barrier(0);
            floatx4 P[2][2];                            // [query block][key block]
            bf16x8 Pb[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        P[qb][kb][e] = __builtin_amdgcn_exp2f(X[qb][kb][e] * c);
                        Pb[kb][4 * qb + e] = static_cast<__bf16>(P[qb][kb][e]);
                    }
            // plain stores: the compiler gives them the wait states that exponentials and matrix results need
            floatx4 *out = reinterpret_cast<floatx4 *>(group_lds + P_XCHG + pair * PAIR_B + lane * 16);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) out[64 * (2 * kb + qb)] = P[qb][kb];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            g_t.run(tr_addr, Pb, acc);                                              // dV^T += dO^T P
        } else {
            staged_rows_times_resident<D, ST + G_TILE>(row_addr, resident, X);      // dO V^T - delta
            StagedTransposedProduct<D, ST + Q_TILE> q_t;
            q_t.prefetch(tr_addr);
            __builtin_amdgcn_s_barrier();
            bf16x8 dSb[2];
            bf16x8 raw[4];                              // key block 0: query blocks 0, 1; key block 1
            raw[0] = ds_read_b128_at<0>(xchg_addr);
            raw[1] = ds_read_b128_at<1024>(xchg_addr);
            raw[2] = ds_read_b128_at<2048>(xchg_addr);
            raw[3] = ds_read_b128_at<3072>(xchg_addr);
            lds_wait2<2>(raw[0], raw[1]);
            lds_wait2<0>(raw[2], raw[3]);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) {
                    const floatx4 P = __builtin_bit_cast(floatx4, raw[2 * kb + qb]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dSb[kb][4 * qb + e] = static_cast<__bf16>(P[e] * X[qb][kb][e]);
                }
            q_t.run(tr_addr, dSb, acc);                                             // dK^T += Q^T dS
        }
    };
    auto all_sub_blocks = [&](auto role_c) __attribute__((always_inline)) {
        for (int u = 0; u < share.n_steps; u += 2) {
            sub_block(role_c, std::integral_constant<int, 0>{}, u);
            if (u + 1 < share.n_steps) sub_block(role_c, std::integral_constant<int, 1>{}, u + 1);
        }
    };
    if (probs_role) all_sub_blocks(std::true_type{});
    else all_sub_blocks(std::false_type{});
    if constexpr (G > 1) {
        merge_groups<G, WAVES>(smem, group, wave, lane, acc);
        if (group != 0) return;
    } else {
        __syncthreads();                                // every wave has finished reading the stages
    }
    store_columns<D>(smem + wave * WAVE_OUT, acc, probs_role ? 1.0f : c * kLn2, (probs_role ? d_v : d_k) + my_row * D, lane);
}

struct BwdArgs {
    const bf16_raw *q, *k, *v, *o, *d_o;
    const float *lse;
    float *neg_delta, *neg_lse;
    bf16_raw *d_q, *d_k, *d_v;
    int B, D;
    sta::FwdParams p;
    const sta::WindowTable &win;
    const sta::HeadOrder &order;
    hipStream_t stream;
    sta::LaunchNote *note;      // not null: the shape is written there and nothing is launched
};

// Sub-blocks of the walk of a head away from the borders; heads by rank, the one with the most key tiles first.
uint32_t walk_of_rank(const BwdArgs &a, uint32_t rank)
{
    const sta::FwdParams &p = a.p;
    uint32_t units = p.P / kSub;
    const uint32_t n[3] = {p.n_t, p.n_h, p.n_w};
    for (int i = 0; i < 3; ++i) {
        const uint32_t kept = 2 * (a.win.w[a.order.h[rank]][i] / 2u) + 1;
        units *= kept < n[i] ? kept : n[i];
    }
    return units;
}
uint32_t longest_walk(const BwdArgs &a) { return walk_of_rank(a, 0); }
// Sub-blocks of the longest walk over the queries of a key tile: a window of 2 * half + 1 tiles keeps the tiles 2 * half from a border
// for 3 * half + 1 query tiles, or for all where both borders see them.
uint32_t longest_key_walk(const BwdArgs &a)
{
    const sta::FwdParams &p = a.p;
    const uint32_t n[3] = {p.n_t, p.n_h, p.n_w};
    uint32_t most = 0;
    for (uint32_t h = 0; h < p.heads; ++h) {
        uint32_t units = p.P / kSub;
        for (int i = 0; i < 3; ++i) {
            const uint32_t half = a.win.w[h][i] / 2u;
            units *= n[i] - 1 <= 4 * half ? n[i] : 3 * half + 1;
        }
        most = units > most ? units : most;
    }
    return most;
}

// Sub-blocks that the XCD with the most of them walks, of a launch that is dealt head after head; per_rank blocks per head.
uint64_t fullest_xcd(const BwdArgs &a, const sta::Deal &deal, uint64_t per_rank)
{
    uint64_t before[sta::kMaxHeadsPerLaunch + 1] = {}, load[8] = {}, most = 0;
    for (uint32_t r = 0; r < a.p.heads; ++r) before[r + 1] = before[r] + per_rank * walk_of_rank(a, r);
    auto up_to = [&](uint64_t block) {
        const uint64_t r = block / per_rank;
        return before[r] + (r < a.p.heads ? (block - r * per_rank) * walk_of_rank(a, (uint32_t)r) : 0);
    };
    uint64_t at = 0;
    for (uint32_t c = 0; c < 8 * (deal.last_slot / deal.chunk.d + 1); ++c) {
        const uint32_t xcd = c & 7;
        const uint64_t to = at + (at < 8 * (uint64_t)deal.last_slot ? deal.chunk.d : deal.last_len + (xcd < deal.last_more));
        load[xcd] += up_to(to) - up_to(at);
        at = to;
    }
    for (uint64_t l : load) most = l > most ? l : most;
    return most;
}

// How the blocks are dealt.  One chunk = the column blocks of one row of tiles along w.  Measured at the 30x48x80 grid (chunk sizes 1, 3,
// 6, 30, 60, 120 in one session): dK/dV kernel 32.7, 31.5, 31.6, 31.0, 31.1, 34.0 ms; dQ kernel 18.9, 18.8, 18.7,
// 18.5, 18.5, 19.3 ms.  Where the walks of the heads differ, a round of eight rows can hold rows of two heads, and an XCD gets the long
// ones: launches of fewer than twenty rounds are then cut into as many rounds of equal chunks, but only where that makes the walks of the
// fullest XCD shorter by more than 1 % (22 heads of 12x8x40 in 384-token tiles, 2x1x4 and 2x1x2, by 1.8 %: step 662 -> 638 us; not ten of
// 6x24x24, eight of them with walks of 108 sub-blocks and two of 36, whose 24 long rows are three for every XCD: chosen by the number
// of blocks alone, equal chunks gave two XCDs 68 long ones for 64 places, 115 -> 150 us dK/dV, training step 281 -> 325).
sta::Deal deal_blocks(const BwdArgs &a, uint32_t cols)
{
    const sta::FwdParams &p = a.p;
    const uint64_t per_rank = (uint64_t)(p.N / cols) * a.B;
    const uint32_t total = (uint32_t)(per_rank * p.heads), row = p.n_w * (p.P / cols);
    const sta::Deal rows = sta::deal_in_chunks(total, row);
    const uint32_t rounds = (uint32_t)((total + 8 * (uint64_t)row - 1) / (8 * (uint64_t)row));
    if (rounds > 20 || walk_of_rank(a, 0) == walk_of_rank(a, p.heads - 1)) return rows;
    const sta::Deal equal = sta::deal_in_chunks(total, (total + 8 * rounds - 1) / (8 * rounds));
    return 100 * fullest_xcd(a, rows, per_rank) > 101 * fullest_xcd(a, equal, per_rank) ? equal : rows;
}

BwdPlan make_plan(const BwdArgs &a, uint32_t cols, bool row_major, bool longest_first)
{
    const sta::FwdParams &p = a.p;
    BwdPlan plan;
    const uint32_t per_tile = p.P / cols;
    plan.deal = deal_blocks(a, cols);
    plan.per_row = sta::fast_div_of(p.n_w * per_tile);
    plan.rows = sta::fast_div_of(p.n_t * p.n_h);
    plan.slices = sta::fast_div_of((uint32_t)a.B * p.heads);
    plan.row_major = row_major;
    plan.longest_first = longest_first;
    plan.per_tile = sta::fast_div_of(per_tile);
    plan.n_h = sta::fast_div_of(p.n_h);
    plan.batch = sta::fast_div_of((uint32_t)a.B);
    plan.sub_per_tile = sta::fast_div_of(p.P / kSub);
    plan.inv_scale = kLog2e / p.scale_log2e;
    for (uint32_t r = 0; r < p.heads; ++r) {
        const uint16_t h = a.order.h[r];
        plan.head[r].h = h;
        for (int i = 0; i < 3; ++i) plan.head[r].w[i] = a.win.w[h][i];
    }
    return plan;
}

// The shape of a launch as text, with the sub-blocks that the XCD with the most of them walks and those of all.
hipError_t note_launch(const BwdArgs &a, const BwdPlan &plan, const char *shape)
{
    uint64_t load[8] = {}, all = 0, most = 0;
    for (uint32_t id = 0; id < plan.deal.total; ++id) {
        const uint32_t line = sta::dealt_item(id, plan.deal) / plan.per_row.d;
        const uint32_t rank = plan.row_major ? line % plan.slices.d : line / plan.rows.d;
        load[id & 7] += walk_of_rank(a, rank / plan.batch.d);
    }
    for (uint64_t l : load) {
        all += l;
        most = l > most ? l : most;
    }
    return a.note->add("%s items %u, fullest XCD %llu of %llu sub-blocks, %s", shape, plan.deal.total, (unsigned long long)most, (unsigned long long)all,
                       plan.row_major ? "rows of all heads in turn" : "head after head");
}

template <int D, int QW, int G, bool DMA = true, bool SOLO = (QW == 1 && G > 1)>
hipError_t launch_dq(const BwdArgs &a)
{
    const BwdPlan plan = make_plan(a, QW * 32, false, false);
    if (a.note) {
        char shape[64];
        snprintf(shape, sizeof shape, "%s<%d,%d,%d,%d>", SOLO ? "dq_one_buffer" : "dq", D, QW, G, (int)DMA);
        return note_launch(a, plan, shape);
    }
    return sta::launch_kernel(sta_bwd_dq_kernel<D, QW, G, DMA, SOLO>, dim3(plan.deal.total), dim3(QW * G * 64), a.stream, a.q, a.k, a.v, a.o, a.d_o, a.lse,
                              a.neg_delta, a.neg_lse, a.d_q, a.p, plan);
}

// Order of the dK/dV items where all heads' walks are equal (otherwise head after head: heads of long walks must not have rows
// left at the end; 16x48x64 in 256-token tiles, 3x3x3 and 3x3x5 2046 us head after head, 2377 row after row; 30x48x80, windows
// from 1x3x3 to the whole grid 17.5, 26.6 ms).  Entry point, head after head against the rows of all heads in turn:
// - Rows of tiles per head a multiple of eight: head after head an XCD gets the same rows of every head, and border rows have
//   half the work of inner ones.  16x48x64 in 256-token tiles, 24 heads, head dimension 64 7443, 6488 us, 128 -12 %;
//   20x64x64 in 64-token tiles -19 %, four images -20 %.
// - Otherwise it shortens the tail, which tells in launches of up to about sixteen rounds of workgroups (18x40x64 in 192-token
//   tiles, 16 heads -7 %; 10x30x56 in 96-token tiles -11 %; 30x48x80 in 384-token tiles, two heads -9 %, four -5 %).  Beyond that
//   what counts is that the next row of a head finds operands of this one in the caches: its box of Q and dO rows either fits an XCD's L2 (20x48x64 in 128-token tiles, head dimension 64, 40 heads -1 %;
//   12x48x48, 48 heads of 128 -3 %) or the rows of a head should stay together (30x48x80, head dimension 64, 12 to 24 heads
//   +0.4 to +1.5 %; 128 +1 %).
// - Not where every workgroup has a CU of its own and no order can even anything out (24x32x32, two heads of 128 +3 to +4 %), as in
//   every launch of six pairs and of eight walk groups (sixty drawn launches of those at head dimension 64: either order, 0.99 to 1.02, 1.00 in
//   the mean).
bool rows_of_all_heads(const BwdArgs &a, uint32_t cols, uint64_t resident)
{
    const sta::FwdParams &p = a.p;
    const uint64_t slices = (uint64_t)a.B * p.heads;
    const uint64_t blocks = slices * (p.N / cols);
    if (walk_of_rank(a, 0) != walk_of_rank(a, p.heads - 1)) return false;
    if (resident <= sta::compute_units() && blocks <= resident) return false;
    const uint32_t kept_w = 2 * (a.win.w[a.order.h[0]][2] / 2u) + 1;
    const uint64_t box_rows = (uint64_t)longest_walk(a) * kSub / (kept_w < p.n_w ? kept_w : p.n_w) * p.n_w;
    return p.n_t * p.n_h % 8 == 0 || blocks <= 16 * resident || box_rows * a.D * 4 <= (4u << 20);
}

// The longest rows first on tiles of 96 tokens' multiples (workgroups that a CU holds few of: 10x30x56, us, rows as they come
// and longest first: three heads 371, 341, five 439, 421; 192-token tiles, eight heads of 128 3057, 2947).  Not elsewhere: few
// heads are then dealt unevenly (16x48x64, four heads -15 % as they come, -12 %; 30x48x80, two -9, -3 %), and not along w: every
// fourth item of an XCD goes to the same part of it, and a row of eight tiles at window 4 would put the long ones there (20x12x64
// in 128-token tiles, five heads 761, 957 us).
template <int D, int NW, int G, int UPS = 1, bool DMA = true>
hipError_t launch_dkv(const BwdArgs &a)
{
    const uint64_t resident = (uint64_t)sta::compute_units() * max_of(1, (D == 64 ? 12 : 8) / (NW * G));     // workgroups: whole ones per CU
    const bool row_major = rows_of_all_heads(a, NW * 32, resident), longest_first = a.p.P % 96 == 0 && a.p.P % 128 != 0;
    const BwdPlan plan = make_plan(a, NW * 32, row_major, row_major && longest_first);
    if (a.note) {
        char shape[64];
        snprintf(shape, sizeof shape, "dkv<%d,%d,%d,%d,%d>", D, NW, G, UPS, (int)DMA);
        return note_launch(a, plan, shape);
    }
    return sta::launch_kernel(sta_bwd_dkv_kernel<D, NW, G, UPS, DMA>, dim3(plan.deal.total), dim3(NW * G * 64), a.stream, a.q, a.k, a.v, a.d_o,
                              a.neg_lse, a.neg_delta, a.d_k, a.d_v, a.p, plan);
}

template <int NPAIR, int G, bool DMA = true>
hipError_t launch_dkv_pairs(const BwdArgs &a)
{
    const uint64_t resident = (uint64_t)sta::compute_units() * 12 / (2 * NPAIR * G);     // workgroups
    const bool row_major = rows_of_all_heads(a, NPAIR * 32, resident), longest_first = a.p.P % 96 == 0;
    const BwdPlan plan = make_plan(a, NPAIR * 32, row_major, row_major && longest_first);
    if (a.note) {
        char shape[64];
        snprintf(shape, sizeof shape, "dkv_pair<%d,%d,%d>", NPAIR, G, (int)DMA);
        return note_launch(a, plan, shape);
    }
    return sta::launch_kernel(sta_bwd_dkv_pair_kernel<NPAIR, G, DMA>, dim3(plan.deal.total), dim3(NPAIR * G * 128), a.stream, a.q, a.k, a.v, a.d_o,
                              a.neg_lse, a.neg_delta, a.d_k, a.d_v, a.p, plan);
}

// Operands at an odd address: tiles that have not always been staged by DMA (no multiple of 128 tokens) take the smallest
// shape of either kernel, with plain loads.
// Shapes of the two kernels.  Measured in us, kernel alone; "clip" is the 12x48x48 grid in 384-token tiles at window 1x3x3
// (108 sub-blocks per walk), "image" the 64x64 grid in 64-token tiles at 3x3 (18), "full" 12x32x48 in 384-token tiles at the
// whole grid (576), then the number of heads.
//
// dQ: waves of queries as many as the tile allows up to four, because a staged sub-block serves them all (four against two at
// head dimension 128: clip x 12 695 against 772, full x 8 1613 against 1726).  Two walk groups where the launch then still fits
// the chip (8 waves per CU at head dimension 128, 12 at 64); one against two at 128: clip x 1 (864 waves) 128, 121, full x 1
// (576) 390, 308, image x 2 (256) 18.1, 15.0, image x 8 (1024) 24.5, 22.7, clip x 2 (1728) 141, 160; at 64: image x 8 (1024)
// 16.8, 14.2, image x 16 (2048) 21.1, 23.4; but walks of 32 and more on tiles of odd multiples of 64, whose one group has two waves as well,
// up to the 16 that a CU holds (entry point, waves and units: (1664, 50) 104, 98, (2048, 50) 117, 110, (2000, 90) 199, 184; the other tiles,
// of four and three waves a group, -1 to +1 %).  Four groups of one wave, without barriers, up to one such workgroup per CU
// (two on 96-token tiles at head dimension 64), and up to four where walks are long (below); entry point, two groups of two or three waves against these,
// on two buffers for each operand: 12x24x24 in
// 384-token tiles, one head (216 waves) of 64 100, 87, of 128 151, 131, two (432) 107, 110; 64x64 image, 5x5, one head (128) of 128 149,
// 140, three (384) 150, 157; 4x12x24 in 96-token tiles, one head (36) of 64 39.5, 31.2, of 128 59.6, 47.3; twelve (432) 40.6, 35.4
// and 61.3, 61.9.
//
// Eight groups of one wave in both kernels where no CU gets a second workgroup and the walk has 40 sub-blocks or more, 44 at head dimension 128: two waves a
// SIMD, of which one computes while the other waits, and half the steps.  Entry point (with the permutation), four against eight, dQ
// alone, dK/dV alone and both; waves and units: head dimension 64 (216, 216) 125.1, -6.6, -13.4, -19.2 %; (108, 108) 79.3, -4.0,
// -8.6, -12.6; (72, 48) 64.0, -2.7, -6.0, -8.9; (56, 40) 54.3, -0.6, -5.9, -6.3; (240, 45) 59.9, -1.3, -4.8, -6.3; (144, 36) 50.5,
// +0.2, -2.1, -1.9; (256, 18) 48.4, +0.4, +0.5, +0.1; 128 (216, 216) 203.4, -6.2, -9.8, -15.2; (108, 108) 120.3, -4.3, -5.8, -10.0;
// (72, 48) 92.6, -2.7, -4.4, -7.0; (56, 40) 75.7, 0.0, -3.3, -3.2; (240, 45) 83.7, -0.4, -2.6, -2.8; (144, 36) 69.0, +1.4, +0.4, +1.9;
// (256, 18) 63.4, +3.1, -0.9, +2.3.  With a second workgroup on some CUs the sum of eight and the LDS that they hold cost more:
// 64 (324, 108) 99.3, 0.0, +5.5, +5.5; (432, 54) 78.6, +2.0, +5.5, +7.5; 128 (288, 27) 85.7, 0.0, +8.9, +8.9 (and (384, 50), 64x64
// images, -5.7 and -4.2 % in dK/dV, which the rule leaves out).  Gradients alone, 300 drawn launches, eight groups' time over that of four (on two
// buffers): 64, 40 to 79 sub-blocks 0.80 to 0.94, from 80 on 0.79; 128, 40 to 43 1.00, from 0.93 to 1.04, 44 to 63 0.95, at most 1.001, 64 to 79 0.91, from 80 on 0.88.
bool eight_groups(int D, uint64_t waves, uint32_t units) { return waves <= (uint64_t)sta::compute_units() && units >= (D == 64 ? 40 : 44); }

// Four groups of one wave beyond one workgroup per CU, which at head dimension 64 holds four of them (36 KB and 126 registers) and at 128
// two (74 KB): they wait for no barrier, halve or quarter long walks, and a CU's share is one or two waves a SIMD whatever the tile.
// Entry point (with the permutation and dK/dV), the shapes by barriers against these, waves and units:
// - head dimension 64 (up to two workgroups a CU on two buffers since, 0.99): 384-token tiles (432, 108) 102.5, 98.0, (648, 108) 147, 141, (432, 216) 164, 155, (600, 36) 82.8, 81.9, but (864, 108)
//   152.6, 156.3, (960, 36) 90.8, 94.3; 256 (768, 96) 138, 135; 64 (384, 50) 79.6, 77.9, (512, 128) 119, 116, (640, 128) 156, 152, but (512, 18)
//   53.7, 56.5, (768, 50) 102.6, 103.2, (1024, 50) 112.8, 117; 320 (450, 90) 104.6, 101.4, (750, 90) 136.7, 136.9; 192 (720, 36) 88.7, 87.5,
//   (960, 36) 100, 95, (960, 108) 201, 186, but (768, 18) 64.1, 65.0; 96 (576, 54) 95.7, 93.6, (1008, 54) 134, 130, but (576, 9) 53.2, 55.3;
//   32 (512, 35) 76.8, 68.2, (1024, 35) 104.8, 101.2, (512, 15) 57.0, 54.9, but (512, 9) 49.9, 50.5, (640, 15) 67.4, 67.6;
//   160 (480, 45) 85.5, 75.4, (960, 45) 124, 115;
// - head dimension 128: 384 (432, 108) 174.4, 169.3, (432, 216) 305, 291, but (288, 36) 87.4, 87.6, (648, 108) 232, 238; 64 (512, 128) 212, 210,
//   but (512, 50) 137, 139; 96 (432, 27) 92.5, 89.7, (432, 54) 131.9, 123.6, (864, 54) 254, 236, but (432, 12) 66.8, 67.5, (576, 54) 158, 165;
//   192 (480, 36) 110, 105, (960, 36) 181, 170, (960, 108) 391, 357, but (768, 108) 312, 323 (shapes of three waves have a second round
//   of workgroups from 768 on); 32 (512, 35) 116, 105, (480, 15) 75.9, 74.9, but (512, 9) 67.8, 70.0, (1024, 35) 174, 180; 160 (480, 45) 130, 117.
// Where the walks of the heads differ the long ones are alone at the end and the gain is larger: 64, 96-token tiles, seven heads of 27, 72
// and 3 (504) 89.5, 75.7; 384, two of 108 and 216 159, 141, three 201, 186; 32-token, twelve of 49 and 9 (768) 104, 93; 192, eight of 30 and 3
// (480) 79.6, 68.4; 128, the same 134, 116; 305, 280; (512) 120, 97; 117, 102; 256-token, five of 96 and 24 (480) 162, 157; but 192, sixteen of
// 60 and 18 (960) 161, 167.  At 128, tiles of 96 tokens' multiples, up to two workgroups a CU, walks of 20 to 31 and shorter ones, both kernels:
// sixty drawn launches 0.87 to 0.97 of the time of two groups of three waves, 0.91 in the mean.  Drawn launches that this rule changes, gradients alone,
// with it over without, the largest in brackets: 64 0.89 (181, 1.01), 128 0.90 (119, 0.99); tiles of 128 tokens' multiples 0.95 at either.
template <int D>
bool four_groups_of_one(const BwdArgs &a, uint64_t waves, uint32_t units)
{
    const uint64_t cus = sta::compute_units();
    const uint32_t P = a.p.P;
    const bool three = P % 96 == 0 && P % 128 != 0, one = P % 64 != 0 && P % 96 != 0;       // waves of the other shapes
    if (waves <= (D == 64 && three ? 2 * cus : cus)) return true;
    if (waves > 4 * cus) return false;
    const bool equal = units == walk_of_rank(a, a.p.heads - 1);
    if (D == 64) {
        if (three) return units >= 30;
        if (one) return units >= (waves <= 2 * cus ? 15 : 30);
        return units >= 36 && waves <= (P % 128 == 0 ? 3 : 2) * cus;
    }
    if (three) return units >= 20 && (waves <= 2 * cus || (equal && waves > 3 * cus));
    return waves <= 2 * cus && units >= (one ? 15 : 64);
}

// One wave alone (tiles of 32 tokens' multiples): one buffer for each operand where two would make a long walk wait for a place.  A CU holds four
// waves with two buffers at head dimension 128, eight with one; at 64 nine (64 waves a head of 35 sub-blocks: 2304 110, 2368 122 us, with one
// 109, 112) and sixteen.  Where all are resident with two, a wave waits longer for the one buffer that it has just emptied (gradients alone, two
// buffers, one: 128 1.086 of the time just below 1024 waves, 0.857 just beyond; 64 1.005, 0.910), and where walks differ that is so as
// long as the long ones are, over half the longest: 128, 1260 waves of 105 and 7 sub-blocks 214, 237, 1728 of 63 and 3 150, 164.  Many short walks take
// the places as well: from 1.25 times the even share on.  Nor, at 64, where one begins its second round and two has just filled
// two (4097 to 4608 waves: up to 1.027).  1082 drawn launches, time over that of two buffers everywhere: equal walks 0.977 (64) and 0.924 (128),
// at most 1.002, different ones 0.988 and 0.963, 8 of 353 beyond 1.01 and 1.032 at most (of 300 later ones three, 1050 waves of 50 to 90 sub-blocks at 128 1.058); by the number of
// waves alone, from 2048 and 1025 on, 66 of 353 and 1.123.
template <int D>
bool one_buffer_alone(const BwdArgs &a, uint64_t waves, uint32_t units)
{
    const uint64_t cus = sta::compute_units(), resident = (D == 64 ? 9 : 4) * cus, per_head = (uint64_t)a.B * (a.p.N / 32);
    uint64_t all = 0, long_walks = 0;
    for (uint32_t r = 0; r < a.p.heads; ++r) {
        all += per_head * walk_of_rank(a, r);
        if (2 * walk_of_rank(a, r) > units) long_walks += per_head;
    }
    if (D == 64 && long_walks > 16 * cus && waves <= 18 * cus) return false;
    return long_walks > resident || 4 * all > 5 * resident * units;
}

template <int D>
hipError_t dispatch_dq(const BwdArgs &a)
{
    const uint64_t waves = (uint64_t)a.B * a.p.heads * (a.p.N / 32), fits = (uint64_t)sta::compute_units() * (D == 128 ? 8 : 12);
    const uint32_t P = a.p.P;
    const uint32_t units = longest_walk(a);
    const uint64_t cus = sta::compute_units();
    const bool two_for_64 = D == 64 && P % 64 == 0 && P % 128 != 0 && P % 96 != 0 && units >= 32;
    const uint64_t places = two_for_64 ? 16 * cus : fits;
    bool two = 2 * waves <= places && units >= 16;
    // Where the walks of the heads differ, the long ones are alone at the end, and two groups halve them: where the longest is 1.8 times a
    // place's share of all walks or more (entry point, us, by the number of waves and so; head dimension 64: 96x96 in 64-token tiles, nine
    // heads of 288, 18 and 6 sub-blocks 342, 270; 12x48x48 in 384-token tiles, four of 36, 108, 12 and 864 1270, 971 (with dK/dV below);
    // 8x40x48 in 128-token tiles, six of 480, 36 and 12 487, 438; 128: the same nine 540, 442; the same six 780, 750; 12x32x32 in
    // 256-token tiles, four of 384 and 72 594, 558).  Shapes of three waves, and of four at head
    // dimension 128, in launches that do not have two groups whatever their walks: from two times on, those of three only where the waves of
    // the walks over half the longest are 0.4 of the places or less.  Short of that two groups are 0.8 % ahead in the mean of 222 launches, but
    // up to 12 % behind (one against two: 192-token tiles, 64, 14 heads of 180, 150, 90 and 18, 2.03 times, 289, 301; 288-token tiles, 128, six
    // of 162 and 27, 2.03 times, 358, 376; 384-token tiles, 128, twelve of 120, 36 and 24, 1.86 times, 326, 335).
    // A CU holds six waves of the shapes of three at head dimension 128 (9x40x40,
    // six heads of 162, 18 and 6, 2.0 times in eighths, 1.5 in sixths 467, 480; 151 launches of up to 1024 waves less than 1.8 times in sixths: one
    // group 0 to 10 % ahead).
    if (units >= 64 && units != walk_of_rank(a, a.p.heads - 1)) {
        uint64_t all = 0;
        for (uint32_t r = 0; r < a.p.heads; ++r) all += walk_of_rank(a, r);
        all *= (uint64_t)a.B * (a.p.N / 32);
        const bool three = P % 96 == 0 && P % 128 != 0;
        const uint64_t held = D == 128 && three ? 6 * cus : places;
        if (two || !(three || (D == 128 && P % 128 == 0))) {
            two = 18 * all <= 10 * held * units;
        } else {
            uint64_t long_heads = 0;
            for (uint32_t r = 0; r < a.p.heads; ++r) long_heads += 2 * walk_of_rank(a, r) > units;
            two = 2 * all <= held * units && (!three || 10 * long_heads * a.B * (a.p.N / 32) <= 4 * held);
        }
    }
    if (P % 128 != 0 && !(sta::dma_aligned(a.k) && sta::dma_aligned(a.v))) return launch_dq<D, 1, 1, false>(a);
    if (eight_groups(D, waves, units)) return launch_dq<D, 1, 8>(a);
    // (four groups: two buffers for each operand where every workgroup is resident with them, see the kernel)
    if (four_groups_of_one<D>(a, waves, units)) return waves <= (D == 64 ? 2 : 1) * cus ? launch_dq<D, 1, 4, true, false>(a) : launch_dq<D, 1, 4>(a);
    if (P % 96 == 0 && P % 128 != 0) return two ? launch_dq<D, 3, 2>(a) : launch_dq<D, 3, 1>(a);
    if (P % 64 != 0) return one_buffer_alone<D>(a, waves, units) ? launch_dq<D, 1, 1, true, true>(a) : launch_dq<D, 1, 1>(a);
    if (two) return launch_dq<D, 2, 2>(a);
    return P % 128 == 0 ? launch_dq<D, 4, 1>(a) : launch_dq<D, 2, 1>(a);
}

// dK/dV.  Entry point in us; waves of 32 keys and sub-blocks per walk in brackets.
// Four walk groups of one wave each while few of them share a CU, against two groups of two waves: head dimension 64, 64x64 image
// at 3x3, two heads (256, 18) 21.1, 25.2, eight (1024, 18) 35.2, 34.3; at 5x5, eight (1024, 50) 70, 80; 12x24x24 in 384-token tiles,
// two (432, 108) 83, 89; 9x40x40 in 192-token tiles, two (900, 54) 82, 97, four (1800, 54) 126, 129; 128,
// 8x32x32 in 128-token tiles, one (256, 36) 46, 60, two (512, 36) 65, 61; 64x64 at 5x5, five (640, 50) 101, 110; 9x40x40, three (1350,
// 54) 199, 185; training steps 64-token tiles (800, 90) 260, 259, 192 (960, 72) 261, 258, 320 (900, 180) 455, 413.  Against the shapes of 96- and 32-token tiles: 10x30x56, 64, 3x3x3, four slices (2100, 81) 185, 221, eight (4200, 81)
// 341, 378, ten (5250, 81) 430, 418; 128, two (1050, 81) 227, 285, three (1575, 81) 329, 339, 1x3x3, two (1050, 27) 98, 98; 32x64 in
// 32-token tiles, 128, four (256, 9) 24.4, 25.4, eight (512, 9) 32.8, 31.0, at 5x5 (512, 25) 62, 79.
// Beyond that two groups of two waves where the launch is still small or the walk long, against two or four waves: 64, 384-token
// tiles, six heads (1296, 108) 142, 156, eight (1728, 108) 187, 175; 128-token tiles, eight (2048, 36) 89, 91, 24 (6144, 36) 205, 220,
// 256-token tiles, 28 (10080, 120) 951, 914; 64x64, 3x3, 16 (2048, 18) 53, 53, 32 (4096, 18) 88, 85; 192-token tiles, 16 (7200, 54) 355,
// 384; 128, 128-token tiles, six (1536, 36) 128, 137, 24 (6144, 36) 379, 382; 192-token tiles, eight (3600, 54) 360, 408, 24 (10800, 54)
// 1019, 1010; 320-token tiles, eight (4000, 90) 605, 694, 24 (12000, 90) 1744, 1715.
// Long walks: how many waves of columns go to four groups of one wave, which cut them in four, where `solo` do whatever the walk.  A key
// tile's walk over the queries varies inside a head (a window of five along eight tiles keeps the inner ones for up to eight), the longest
// ends a launch of a round or two, and the groups by two leave it twice as long.  Training steps, before and with this rule, us;
// waves, longest walk of a query tile:
// - multiples of 128 tokens, head dimension 64, up to three workgroups a CU: (648, 108) 141, 135, (768, 96) 135, 132, (576, 72) 107, 102,
//   (720, 108), walks up to 1.8 times the mean, 186, 155, (672, 60) 108, 101; not short ones ((768, 32) 75.7, 76.0);
// - the same at 128, up to two, where the longest is 1.3 times the mean of all query walks or more: (448, 140) 1.6 times 253, 232,
//   (336, 180) 321, 276, (360, 60) 147, 133, two heads of 108 and 216 304, 253; below that (480, 240) 336, 343, (432, 72) 131, 135, and with
//   a third workgroup (576, 120) 1.6 times 281, 294;
// - multiples of 32 alone (32, 160, 224), up to three: 64 (768, 35) 89.7, 81.0, (672, 147) 216, 195, (588, 63) 110, 100; 128 (588, 147)
//   450, 402, (768, 35) 158, 147, but (640, 40) 147, 151; up to four from 1.5 times on: 64 (840, 75) of several windows 139, 121, (900, 150)
//   201, 188; 128 (784, 126) 449, 406; not (64, (800, 100) of equal walks 164, 174; 128 (1008, 42) 180, 189, (840, 45) 194, 197).
// The other tiles: see solo's own lines.
// Short walks of key tiles that are nearly even gain nothing at 128 where more than a few share a CU: multiples of 32 alone below 100 sub-blocks
// and 1.2 times the mean (gradients alone, without and with four groups, (750, 50) 99, 106, (728, 56) 107, 112, (540, 90) 163, 166; of 350 drawn
// launches beyond 512 waves 22 are such, 1.03 of the time in the mean, the others 0.88), multiples of 128 below 84 and 1.5 times beyond 352
// waves ((512, 48) 67, 70, (432, 48) 58, 60; of 250 drawn 14 are such, 0.95 to 1.04, the others 0.91).
// Drawn launches with and without this rule, gradients alone: 64 multiples of 32 alone 0.84 (46, 0.96 at most), of 128 0.89 (79, 0.96).
uint64_t single_waves_by_walk(const BwdArgs &a, int D, uint64_t waves, uint32_t units, uint64_t solo)
{
    const uint64_t cus = sta::compute_units();
    const uint32_t P = a.p.P;
    const bool whole = P % 128 == 0, one = P % 64 != 0 && P % 96 != 0;
    const bool few = one && waves <= 3 * cus;
    if (few && D == 64) return units >= 32 ? 3 * cus : solo;
    if (whole && D == 64) return units >= 48 ? 3 * cus : solo;
    if (!(few ? units >= 48 : one ? units >= (D == 64 ? 40 : 60) : whole && waves <= 2 * cus && units >= 48)) return solo;
    const uint64_t longest = longest_key_walk(a);
    uint64_t all = 0;
    for (uint32_t r = 0; r < a.p.heads; ++r) all += walk_of_rank(a, r);
    auto uneven = [&](int tenths) { return 10 * longest * a.p.heads >= tenths * all; };
    if (few) return longest >= 100 || uneven(12) ? 3 * cus : solo;
    if (whole) return uneven(longest < 84 && 8 * waves > 11 * cus ? 15 : 13) ? 2 * cus : solo;
    return uneven(15) ? 4 * cus : solo;
}

template <int D>
hipError_t dispatch_dkv(const BwdArgs &a)
{
    const uint64_t cus = sta::compute_units(), waves = (uint64_t)a.B * a.p.heads * (a.p.N / 32);
    const uint32_t P = a.p.P, units = longest_walk(a);
    if (P % 128 != 0 && !(sta::dma_aligned(a.q) && sta::dma_aligned(a.d_o))) {
        if constexpr (D == 128) return launch_dkv_pairs<1, 1, false>(a);
        else return launch_dkv<64, 1, 1, 1, false>(a);
    }
    uint64_t solo = D == 64 ? 2 * cus : cus;            // up to so many waves
    if (P % 64 == 0 && P % 128 != 0 && units >= 48) solo = (D == 64 ? 8 : 3) * cus;
    if (P % 64 != 0 && P % 96 == 0) solo = (D == 64 ? 18 : 6) * cus;
    if (P % 64 != 0 && P % 96 != 0 && units >= 24) solo = 2 * cus;
    if (eight_groups(D, waves, units)) return launch_dkv<D, 1, 8>(a);
    if (waves > solo && waves <= 4 * cus) solo = single_waves_by_walk(a, D, waves, units, solo);
    if (waves <= solo) return launch_dkv<D, 1, 4>(a);
    if (P % 64 != 0) {
        if constexpr (D == 128) return P % 96 == 0 ? launch_dkv_pairs<3, 2>(a) : launch_dkv_pairs<1, 1>(a);
        else return P % 96 == 0 ? launch_dkv<64, 3, 1>(a) : waves <= 4 * cus ? launch_dkv<64, 1, 2>(a) : launch_dkv<64, 1, 1>(a);
    }
    uint64_t by_walk = waves;                           // waves, those of a head with half the longest walk counted half
    if (D == 128 || units >= 64) {
        uint64_t all_units = 0;
        for (uint32_t r = 0; r < a.p.heads; ++r) all_units += walk_of_rank(a, r);
        by_walk = (uint64_t)a.B * (a.p.N / 32) * all_units / units;
    }
    // One round of six pairs, at least four fifths full: half a wave's products per wave fill a CU where whole ones leave it half
    // empty in the same time (training steps, two groups, six pairs: 30x24x32, two heads of 128, whole grid (1440, 720) 1589, 1495;
    // 6x16x16, 31 heads (1488, 48) 219, 212; 6x24x24, 14 heads (1512, 108) 402, 393; 12x24x24, seven (1512, 216) 728, 713).  Not where the
    // walks of the heads differ: the long ones are one round by themselves ((1296, 72) 239, 253), nor where those of the key tiles do by
    // more than 4 : 3, for the same reason (6x32x32, seven heads at 1x3x3, walks up to 1.8 times the 108 of a query tile 427, 477; 30x24x32,
    // two at 3x3x3, up to 2.2 times 324 1179, 1464; at 4 : 3, 1x3x3, 427, 422).
    // 64-token tiles and the like, short walks: two pairs, of which a CU holds three workgroups, where the two workgroups it holds of the
    // groups below begin a second round (training steps, groups, pairs: (1008, 18) 111, 112; (1200, 18) 131, 128; (1404, 36) 142, 132;
    // (1512, 30) 192, 184; (1584, 12) 130, 126; (1632, 6) 112, 105; but (1440, 144) 431, 453).  Waves count by the walks of their
    // heads, as the long ones fill the chip (140 slices of 16x24, 4 and 12 sub-blocks, 1680 waves that count 1288: 130, 122; 70 of
    // 32x24, 6 to 24: 151, 144; by their number the groups had them).  Not where the longest walk, which two groups halve, is more than
    // 2.2 times a place's even share of all (32x48, 25 heads, 6 to 24, up to 32 of a key tile 127, 131; 40x40, 20 heads 120, 126).
    if constexpr (D == 128) {
        const uint64_t longest = longest_key_walk(a), all = by_walk * units;                // sub-blocks; of all items, doubled
        const bool equal = units == walk_of_rank(a, a.p.heads - 1);
        if (P % 384 == 0 && waves <= 6 * cus && 5 * waves >= 24 * cus && equal && 3 * longest <= 4 * units) return launch_dkv_pairs<6, 1>(a);
        // groups also for one round or so of four waves whose longest walk is 1.8 times a place's share of all or more: they halve it
        // (four waves, two groups: 12x32x40, four heads at 1x3x3 (1920, 108) 599, 523; 6x48x40, seven (2520, 108) 684, 651; 4x40x40 in
        // 256-token tiles, nine of 40 and 120 sub-blocks (1800) 472, 427; but 18x24x48, three, 1.4 times (1944, 324) 1298, 1332)
        if (P % 128 == 0 && waves <= 10 * cus && 40 * cus * longest > 9 * all) return launch_dkv<128, 2, 2>(a);
        const bool small = units < 32 ? by_walk <= 8 * cus : units < 48 && 2 * waves <= 13 * cus;
        if (P % 128 != 0 && waves > 4 * cus && small && (longest < 32 || 30 * cus * longest <= 11 * all)) return launch_dkv_pairs<2, 1>(a);
    }
    // (at head dimension 64 by their walks: 12x32x32 in 384-token tiles, six heads of 384, 108 and 36 411, 365; 12x48x48, four of 36, 108, 12
    // and 864 1260, 1113; but not on 128-token tiles, whose line is at four rounds of the chip and more: by walks -15 to +10 %, 4x72x8, 160 heads
    // of 72, 24 and 8 326, 358)
    if (P == 128) return waves <= 24 * cus ? launch_dkv<D, 2, 2>(a) : launch_dkv<D, 4, 1, D == 64 ? 2 : 1>(a);
    if (P % 128 == 0) return (D == 64 ? by_walk : waves) <= 6 * cus ? launch_dkv<D, 2, 2>(a) : launch_dkv<D, 4, 1, D == 64 ? 2 : 1>(a);
    return by_walk <= 8 * cus || (units >= 32 && (D == 64 || waves <= 32 * cus)) ? launch_dkv<D, 2, 2>(a) : launch_dkv<D, 2, 1>(a);
}

}  // namespace

namespace sta {

bool backward_supported(int P, int D) { return (D == 64 || D == 128) && P > 0 && P % kSub == 0; }

hipError_t launch_backward(const void *q, const void *k, const void *v, const void *o, const void *d_o, const float *lse,
                           float *stats, size_t stat_rows, void *d_q, void *d_k, void *d_v, int B, int D, const FwdParams &p,
                           const WindowTable &win, const HeadOrder &order, hipStream_t stream, LaunchNote *note)
{
    if (!backward_supported((int)p.P, D)) return hipErrorInvalidValue;
    const BwdArgs a = {static_cast<const bf16_raw *>(q), static_cast<const bf16_raw *>(k), static_cast<const bf16_raw *>(v),
                       static_cast<const bf16_raw *>(o), static_cast<const bf16_raw *>(d_o), lse, stats, stats + stat_rows,
                       static_cast<bf16_raw *>(d_q), static_cast<bf16_raw *>(d_k), static_cast<bf16_raw *>(d_v), B, D, p, win, order,
                       stream, note};
    const hipError_t e = D == 64 ? dispatch_dq<64>(a) : dispatch_dq<128>(a);
    if (e != hipSuccess) return e;
    return D == 64 ? dispatch_dkv<64>(a) : dispatch_dkv<128>(a);
}

}  // namespace sta

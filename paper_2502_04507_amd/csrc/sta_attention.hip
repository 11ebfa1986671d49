// Sliding Tile Attention forward kernels for gfx950 (MI355X).
//
// What is computed: Eq. 1 of the paper (S = QK^T/sqrt(d), A = softmax(S + M),
// O = AV) where M keeps, for each query tile, exactly the key tiles inside the
// clamped tile window of the appendix algorithm "Mask Definition of 3D STA".
// Tokens arrive in tile order, so each kept (query tile, key tile) pair is a
// fully dense block and no element-level mask exists anywhere in this file.
//
// Formulation.  The kernel works on the TRANSPOSED score block
// S^T = K Q^T (keys along the MFMA M dimension, queries along N), so that one
// lane owns one query column: its running max / sum are per-lane scalars and
// the only cross-lane traffic in the softmax is one exchange between the two
// 32-lane halves of a wave.  The output is accumulated transposed as well,
// O^T += V^T P^T, which lets P^T go from the S^T accumulators straight into the
// B operand of the second MFMA with no data movement: the MFMA contraction
// index is only a summation index, so the keys are fed in the order the
// accumulator layout holds them and V^T is stored in LDS in that same order.
//
// MFMA of the general kernel: v_mfma_f32_32x32x16_bf16.  Operand layout (lane l, lo = l%32, hb = l/32):
//   A (32 x 16): row lo,  k = 8*hb .. 8*hb+7
//   B (16 x 32): col lo,  k = 8*hb .. 8*hb+7
//   C (32 x 32): col lo,  row = 8*g + 4*hb + t for register r = 4*g + t.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sta_device_util.h"
#include "sta_geometry.h"
#include "sta_internal.h"
#include "sta_staged.h"

namespace {

// Position inside a group of 16 keys at which key `k16` (0..15) is stored in the
// transposed V buffer: the accumulator of S^T holds, for half hb, keys
// {4*hb + t} and {8 + 4*hb + t}; they are made adjacent so one 16-byte LDS read
// yields the 8 keys a lane feeds to the PV MFMA.
__device__ __forceinline__ int vt_pos(int k16)
{
    const int a = k16 >> 3, hb = (k16 >> 2) & 1, t = k16 & 3;
    return 8 * hb + 4 * a + t;
}

template <int D, int NW, int NQ, int KB>
struct FwdCfg {
    static constexpr int kThreads = NW * 64;
    static constexpr int kQB = NW * NQ * 32;          // queries per workgroup
    static constexpr int kKStride = D + 8;            // elements; 16 B pad => conflict-free b128 reads
    static constexpr int kVStride = KB + 8;           // elements (keys) per d row of V^T
    static constexpr int kKElems = KB * kKStride;
    static constexpr int kVElems = D * kVStride;
    static constexpr int kChunks = KB * D / 8;        // 16-byte chunks per K (or V) sub-block
    static constexpr int kChunksPerThread = kChunks / kThreads;
    static_assert(kChunks % kThreads == 0, "sub-block must split evenly over the workgroup");
    static_assert(KB % 32 == 0 && D % 32 == 0, "MFMA tiling");
};

// Token-granular sliding window (appendix algorithm "Mask Definition of 3D NATTEN") along one axis for a query
// tile: the window centre of query x is x clamped into [half, L-1-half] (upper clamp first), its keys are the 2*half+1
// positions around the centre.  c0 / c1: centres of the tile's first / last token (the centre is monotone in x).
struct TokenWindowAxis {
    int half, c0, c1;
    __device__ __forceinline__ void init(int L, int T, int W, int q_tile)
    {
        half = (W < 2 * L ? W : 2 * L) / 2;
        c0 = centre(L, q_tile * T);
        c1 = centre(L, q_tile * T + T - 1);
    }
    __device__ __forceinline__ int centre(int L, int x) const
    {
        const int c = x < (L - 1 - half) ? x : (L - 1 - half);
        return c > half ? c : half;
    }
    // key tiles that at least one query of the tile keeps
    __device__ __forceinline__ StaAxisRange touched(int L, int T) const
    {
        const int lo = c0 - half > 0 ? c0 - half : 0, hi = c1 + half < L - 1 ? c1 + half : L - 1;
        return StaAxisRange{lo / T, hi / T};
    }
    // every query of the tile keeps every key of key tile kt
    __device__ __forceinline__ bool all_kept(int T, int kt) const { return c1 - half <= kt * T && kt * T + T - 1 <= c0 + half; }
};

// TW: token-granular sliding window instead of the STA mask (win then holds the window in tokens); used to
// measure what blocks that are only partly kept cost on the same data.
template <int D, int NW, int NQ, int KB, bool TW = false>
__global__ __launch_bounds__(NW * 64) void sta_fwd_kernel(const bf16_raw *__restrict__ q,
                                                          const bf16_raw *__restrict__ k,
                                                          const bf16_raw *__restrict__ v,
                                                          bf16_raw *__restrict__ o, sta::FwdParams p,
                                                          sta::WindowTable win)
{
    using C = FwdCfg<D, NW, NQ, KB>;
    constexpr int MB = KB / 32;       // 32-key blocks per sub-block
    constexpr int KS = D / 16;        // MFMA k-steps over the head dim
    constexpr int DB = D / 32;        // 32-row blocks of O^T

    __shared__ __attribute__((aligned(16))) bf16_raw Ks[C::kKElems];
    __shared__ __attribute__((aligned(16))) bf16_raw Vt[C::kVElems];
    // TW: coordinates of every token of a tile relative to the tile's origin, packed (t << 20 | h << 10 | w)
    __shared__ __attribute__((aligned(16))) uint32_t intra[TW ? sta::kMaxTokenWindowTile : 4];

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int lo = lane & 31;
    const int hb = lane >> 5;

    const uint32_t qblock = blockIdx.x;                       // index of this QB-query block inside the head
    const uint32_t bh_local = blockIdx.y;                     // b * heads + h_local
    const uint32_t h_local = bh_local % p.heads;
    const uint32_t b = bh_local / p.heads;
    const size_t bh = (size_t)b * p.H + p.head_base + h_local;
    const uint32_t q_tile = (qblock * C::kQB) / p.P;

    StaBox box;
    TokenWindowAxis ax_t, ax_h, ax_w;
    // per lane and query block: first kept key coordinate and (kept keys - 1) along each axis
    int q_lo[NQ][3];
    uint32_t q_span[3] = {0, 0, 0};
    if constexpr (TW) {
        const uint32_t tq_w = q_tile % p.n_w, tq_h = (q_tile / p.n_w) % p.n_h, tq_t = q_tile / (p.n_w * p.n_h);
        ax_t.init(p.n_t * p.T_t, p.T_t, win.w[h_local][0], tq_t);
        ax_h.init(p.n_h * p.T_h, p.T_h, win.w[h_local][1], tq_h);
        ax_w.init(p.n_w * p.T_w, p.T_w, win.w[h_local][2], tq_w);
        box.t = ax_t.touched(p.n_t * p.T_t, p.T_t);
        box.h = ax_h.touched(p.n_h * p.T_h, p.T_h);
        box.w = ax_w.touched(p.n_w * p.T_w, p.T_w);
        for (uint32_t i = tid; i < p.P; i += C::kThreads) {
            const uint32_t iw = i % p.T_w, ih = (i / p.T_w) % p.T_h, it = i / (p.T_w * p.T_h);
            intra[i] = (it << 20) | (ih << 10) | iw;
        }
        q_span[0] = 2 * ax_t.half; q_span[1] = 2 * ax_h.half; q_span[2] = 2 * ax_w.half;
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq) {
            const uint32_t i = (qblock * C::kQB + wave * NQ * 32 + nq * 32 + lo) % p.P;
            const uint32_t iw = i % p.T_w, ih = (i / p.T_w) % p.T_h, it = i / (p.T_w * p.T_h);
            q_lo[nq][0] = ax_t.centre(p.n_t * p.T_t, tq_t * p.T_t + it) - ax_t.half;
            q_lo[nq][1] = ax_h.centre(p.n_h * p.T_h, tq_h * p.T_h + ih) - ax_h.half;
            q_lo[nq][2] = ax_w.centre(p.n_w * p.T_w, tq_w * p.T_w + iw) - ax_w.half;
        }
    } else {
        box = sta_key_tile_box_of(p.n_t, p.n_h, p.n_w, win.w[h_local][0], win.w[h_local][1], win.w[h_local][2], q_tile);
    }

    const bf16_raw *qh = q + (bh * p.N + (size_t)qblock * C::kQB + (size_t)wave * NQ * 32) * D;
    const bf16_raw *kh = k + bh * p.N * D;
    const bf16_raw *vh = v + bh * p.N * D;

    // Q fragments stay in registers for the whole kernel (B operand of S^T = K Q^T).
    bf16x8 Qr[NQ][KS];
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            Qr[nq][ks] = *reinterpret_cast<const bf16x8 *>(qh + (size_t)(nq * 32 + lo) * D + ks * 16 + hb * 8);

    floatx16 Oacc[NQ][DB];
    float m_run[NQ], l_run[NQ];
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        m_run[nq] = -INFINITY;
        l_run[nq] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) Oacc[nq][db][r] = 0.f;
    }

    const int sub_per_tile = p.P / KB;
    const int n_iter = box.count() * sub_per_tile;

    // Iteration state: (kt_t, kt_h, kt_w, sub-block) walked in ascending tile id order.
    int it_t = box.t.lo, it_h = box.h.lo, it_w = box.w.lo, it_s = 0;
    auto key_base = [&]() -> size_t {
        const size_t kt = ((size_t)it_t * p.n_h + it_h) * p.n_w + it_w;
        return (kt * p.P + (size_t)it_s * KB) * D;
    };
    auto advance = [&]() {
        if (++it_s == sub_per_tile) {
            it_s = 0;
            if (++it_w > box.w.hi) {
                it_w = box.w.lo;
                if (++it_h > box.h.hi) { it_h = box.h.lo; ++it_t; }
            }
        }
    };

    uint4 kreg[C::kChunksPerThread], vreg[C::kChunksPerThread];
    auto fetch = [&](size_t base) {
#pragma unroll
        for (int i = 0; i < C::kChunksPerThread; ++i) {
            const int ci = tid + i * C::kThreads;
            kreg[i] = *reinterpret_cast<const uint4 *>(kh + base + (size_t)ci * 8);
            vreg[i] = *reinterpret_cast<const uint4 *>(vh + base + (size_t)ci * 8);
        }
    };

    fetch(key_base());

    for (int iter = 0; iter < n_iter; ++iter) {
        __syncthreads();                       // everyone is done reading the previous sub-block
#pragma unroll
        for (int i = 0; i < C::kChunksPerThread; ++i) {
            const int ci = tid + i * C::kThreads;
            const int row = ci / (D / 8);      // key inside the sub-block
            const int c = ci % (D / 8);        // 8-element chunk along d
            *reinterpret_cast<uint4 *>(&Ks[row * C::kKStride + c * 8]) = kreg[i];
            const int col = (row & ~15) + vt_pos(row & 15);
            const bf16_raw *ve = reinterpret_cast<const bf16_raw *>(&vreg[i]);
#pragma unroll
            for (int e = 0; e < 8; ++e) Vt[(c * 8 + e) * C::kVStride + col] = ve[e];
        }
        __syncthreads();
        // TW: this sub-block's key tile and position in it, before the walk moves on
        const int cur_t = it_t, cur_h = it_h, cur_w = it_w, cur_s = it_s;
        advance();
        if (iter + 1 < n_iter) fetch(key_base());   // next sub-block in flight during the math

        // ---- S^T = K Q^T -------------------------------------------------------
        floatx16 S[NQ][MB];
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int r = 0; r < 16; ++r) S[nq][mb][r] = 0.f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&Ks[(mb * 32 + lo) * C::kKStride + ks * 16 + hb * 8]);
#pragma unroll
                for (int nq = 0; nq < NQ; ++nq) S[nq][mb] = mfma_32x32x16(a, Qr[nq][ks], S[nq][mb]);
            }

        // ---- TW: scores of keys outside the query's window become -inf; blocks kept in full skip the test
        if constexpr (TW) {
            const bool whole = ax_t.all_kept(p.T_t, cur_t) && ax_h.all_kept(p.T_h, cur_h) && ax_w.all_kept(p.T_w, cur_w);
            if (!whole) {
                const int o_t = cur_t * p.T_t, o_h = cur_h * p.T_h, o_w = cur_w * p.T_w;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        // registers 4*g .. 4*g+3  <->  keys 8*g + 4*hb + 0..3 of this 32-key block
                        const uint4 c4 = *reinterpret_cast<const uint4 *>(&intra[cur_s * KB + mb * 32 + 8 * g + 4 * hb]);
                        const uint32_t cs[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int kt = o_t + (int)(cs[t] >> 20), kh_ = o_h + (int)((cs[t] >> 10) & 1023), kw = o_w + (int)(cs[t] & 1023);
#pragma unroll
                            for (int nq = 0; nq < NQ; ++nq) {
                                const bool keep = (uint32_t)(kt - q_lo[nq][0]) <= q_span[0] && (uint32_t)(kh_ - q_lo[nq][1]) <= q_span[1] &&
                                                  (uint32_t)(kw - q_lo[nq][2]) <= q_span[2];
                                S[nq][mb][4 * g + t] = keep ? S[nq][mb][4 * g + t] : -INFINITY;
                            }
                        }
                    }
            }
        }

        // ---- online softmax (one query column per lane) -------------------------
        bf16x8 Pb[NQ][MB][2];
#pragma unroll
        for (int nq = 0; nq < NQ; ++nq) {
            float mx = S[nq][0][0];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S[nq][mb][r]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run[nq], mx);
            // TW: a query may have met masked keys only so far; the offset then stays at 0 so that no inf - inf appears
            const float m_off = (TW && m_new == -INFINITY) ? 0.f : m_new;
            const float alpha = exp2f((m_run[nq] - m_off) * p.scale_log2e);
            const float mneg = -m_off * p.scale_log2e;
            m_run[nq] = m_new;
            float psum = 0.f;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        // register 8*j + e  <->  key 16*j + 8*(e/4) + 4*hb + e%4 of this 32-key block
                        const float pe = exp2f(fmaf(S[nq][mb][8 * j + e], p.scale_log2e, mneg));
                        const __bf16 pb = static_cast<__bf16>(pe);
                        Pb[nq][mb][j][e] = pb;
                        psum += static_cast<float>(pb);
                    }
                }
            l_run[nq] = l_run[nq] * alpha + psum;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) Oacc[nq][db][r] *= alpha;
        }

        // ---- O^T += V^T P^T ----------------------------------------------------
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&Vt[(db * 32 + lo) * C::kVStride + (mb * 2 + j) * 16 + hb * 8]);
#pragma unroll
                    for (int nq = 0; nq < NQ; ++nq) Oacc[nq][db] = mfma_32x32x16(a, Pb[nq][mb][j], Oacc[nq][db]);
                }
    }

    // ---- finalize: O = O / l, bf16, tiled layout ----------------------------------
    bf16_raw *oh = o + (bh * p.N + (size_t)qblock * C::kQB + (size_t)wave * NQ * 32) * D;
#pragma unroll
    for (int nq = 0; nq < NQ; ++nq) {
        const float l_tot = l_run[nq] + __shfl_xor(l_run[nq], 32);
        const float inv = 1.f / l_tot;
        // sum_j exp(s_j * scale) = 2^(m * scale_log2e) * l  =>  ln = m * scale_log2e * ln 2 + ln l
        if (p.lse != nullptr && hb == 0)
            p.lse[bh * p.N + (size_t)qblock * C::kQB + (size_t)wave * NQ * 32 + nq * 32 + lo] =
                m_run[nq] * p.scale_log2e * 0.6931471805599453f + __logf(l_tot);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4 ov;
#pragma unroll
                for (int t = 0; t < 4; ++t) ov[t] = static_cast<__bf16>(Oacc[nq][db][4 * g + t] * inv);
                // rows of O^T are channels: d = 32*db + 8*g + 4*hb + t
                *reinterpret_cast<bf16x4 *>(oh + (size_t)(nq * 32 + lo) * D + db * 32 + g * 8 + hb * 4) = ov;
            }
    }
}


// Work splitting below one query block.  The last workgroups of a launch would run on a mostly idle chip (the
// item count is rarely a multiple of the number of workgroups the chip holds).  The host therefore turns the
// items from `split_first` on into `split_parts` workgroups each; part j walks the sub-blocks
// [n*j/parts, n*(j+1)/parts) of the item's key walk and leaves its unnormalised accumulator, exponent offset and
// row sum in the workspace, and sta_fwd_combine_kernel merges the parts of an item in a fixed order.
// Workspace layout, per part (index = workgroup id - split_first): float O[QB][D], float m[QB], float l[QB].
template <int D>
__host__ __device__ __forceinline__ size_t split_part_floats(int QB) { return (size_t)QB * (D + 2); }

// Work items.  The hardware deals workgroup ids round-robin over the 8 XCDs (each with its own L2) and, inside an XCD, starts
// them in increasing order.  The launch's items, taken head after head in scheduling order, are dealt to the XCDs in chunks of
// about an eighth of a head: each XCD carries one eighth of every head whatever the per-head windows are (load balance: with
// mixed per-head windows this halved the launch time), its resident workgroups are neighbouring query blocks of one head (shared
// K/V in L2), and where a head has only a few items no XCD gets one more of every head than the others (eighteen 384-token items
// a head, 28 heads, 1x2x3: 249 us with exact eighths of every head, which gave two XCDs three rounds of workgroups where two are
// needed, 193 in chunks; fifteen of 25 items 281, 219).  The last round of chunks divides what is left evenly (see Deal): whole
// layers, us, with a last round of whole chunks, which some XCDs get and others do not, and evenly: seven heads of 6x16x24 in
// 384-token tiles, head dimension 64, 1x2x3 (252 items: 35 on the fullest XCD's 32 CUs, 32) 43.0, 32.0; 15 of 6x40x40 in 128-token
// tiles, 3x3x3 297, 284; 24 of 30x48x80, 3x3x3 12.29, 11.92 ms.  Heads are visited in descending cost order, so the tail of the
// launch is made of cheap items.
// Inside a head the query tiles are scheduled by pairs of tile rows (h), then w, then the row of the pair, then t fastest, so that
// the ~32 tiles resident on an XCD at one time form a compact 3-D block, (all t) x (2 h) x (about 3 w), and share key tiles along
// all three axes (measured: reads past L2 9.8 -> 6.4 GB per launch against plain tile-id order, 12.81 -> 12.74 ms).
// Every division by a launch constant is prepared by the host: found by division in the kernel, the item, its box and the start
// of the walk took 7500 cycles of a workgroup that has 24,000 cycles of work to do, a 64-token image tile at window 3x3; now 2000,
// most of it waiting for the kernel arguments.
struct GroupItem {
    size_t bh;
    uint32_t qblock;
    StaBox box;
};
__device__ __forceinline__ GroupItem group_item_of(uint32_t id, const sta::FwdParams &p, const sta::FwdPlan &plan)
{
    GroupItem it;
    const uint32_t linear = sta::dealt_item(id, plan.deal);
    const uint32_t rank = fast_div(linear, plan.per_head), pos = linear - rank * plan.per_head.d;
    const uint32_t head_rank = fast_div(rank, plan.batch);                  // batch entries of one head are adjacent
    const sta::FwdPlan::Head head = plan.head[head_rank];
    const uint32_t sched = fast_div(pos, plan.per_tile), sub = pos - sched * plan.per_tile.d;
    const uint32_t hp = fast_div(sched, plan.pair_items), rem = sched - hp * plan.pair_items.d;
    const uint32_t col = fast_div(rem, plan.n_t), t = rem - col * plan.n_t.d;
    const bool two_rows = 2 * hp + 1 < p.n_h;
    const uint32_t w = two_rows ? col >> 1 : col, h = 2 * hp + (two_rows ? col & 1 : 0);
    it.qblock = ((t * p.n_h + h) * p.n_w + w) * plan.per_tile.d + sub;
    it.bh = (size_t)(rank - head_rank * plan.batch.d) * p.H + p.head_base + head.h;
    it.box.t = sta_axis_range(p.n_t, head.w[0], t);
    it.box.h = sta_axis_range(p.n_h, head.w[1], h);
    it.box.w = sta_axis_range(p.n_w, head.w[2], w);
    return it;
}

// ---------------------------------------------------------------------------
// The key-group kernel: head dimension 64 at every tile size, head dimension 128 where the tile is not a multiple of 128
// tokens and in small launches of those that are.  A workgroup is QW waves of 32 queries (one query block) times KG key groups: the groups share the queries and
// take one KG-th of the walk each, with LDS stages of their own, and their partial results are merged through LDS at the
// end.  KG = 1 where the launch fills the chip; KG = 2 or 4 makes more waves of few queries, for launches that would leave
// it idle.
//
// v_mfma_f32_16x16x32_bf16.  A lane holds column c16 = lane & 15 of a 16x16 result (a query) and its rows 4*g4 .. 4*g4+3
// (g4 = lane >> 4); a wave's 32 queries are two blocks of 16 and every K and V fragment read from LDS feeds both.  The
// score accumulators start at minus the exponent offset (Sinit).  Row sums are a matrix product too, with an operand of
// ones: v_dot2_f32_bf16 runs on the matrix pipe as well and eight of them take longer than the two matrix instructions.
// The LDS layouts (Staged for V, StagedRows for K) leave five operand addresses per wave; the stage is part of the read instructions
// where the loop is unrolled over the stages (the offset stays), an addition to each address otherwise.
//
// What bounds it.  Head dimension 64: the vector issue port.  A unit (32 keys) is 18 matrix instructions (288 cycles of the matrix
// pipe, 8 of the port each) next to 41 vector instructions, 16 of them exponentials (9 cycles; the others 4): 205 ns a SIMD and unit for the
// instructions alone, at 1.8 to 2.1 GHz, measured 233 on the 30x48x80 grid (24 heads, 384-token tiles, window 3x3x3), where the matrix pipe is
// busy 68 % of the cycles.  Seven vector instructions more (the stage in the addresses, the operand of ones made in every unit) made that
// 243.  41 % on 128 heads of a 64x64 image in 8x8 tiles (18 units per item, 78 % of an item's cycles; 99 -> 96 us); LDS bank
// conflicts only where the results leave (16 to 64 per wave).
// The grid: 6.97-7.15 ms with the 12-wave kernel on v_mfma_f32_32x32x16_bf16 that was here before, 6.68-6.83 with QW = 4
// (QW = 12: 7.5, QW = 2: 7.3; row sums by v_dot2: 7.2), 6.53-6.63 with two units per stage (UPS, 64 keys per barrier).  The
// images: 105-109 us before, 98-100.  (Figures from before the loop was unrolled: 6.94 -> 6.69 ms a layer since.)  Head dimension 128, 96-token tiles (10x30x56, 10 slices, windows 3x3x3 and 2x4x3): 2390 us
// with the register-staged kernel that served it before, 294-299 us, 290 since a move of the offset touches no score (below).
// FOLLOW: the offset is the running maximum in every unit.  Otherwise it is the maximum of an item's first unit, and the
// largest probabilities of a row are rounded to bf16 like any other; at the running maximum the largest is exactly 1 and has
// no rounding error.  Against 64 bits (2-norm of the outputs, 96-token tiles, window 3x3x3, N(0,1)): 2.32e-3 with the fixed
// offset, 2.17e-3 following, 2.24e-3 with the register-staged kernel.  Following costs 15 %
// (260 -> 299 us; 290 with the offset in the exponent's fused multiply-add, which also ended the spills of the three-wave shapes at
// head dimension 128, 12 to 32 bytes; 24 slices, 1x3x3 229 -> 222, 30 of head dimension 64 420 -> 411), so it is done on the tiles whose kernel has always done it: no multiple of 128 tokens at head dimension
// 128, of 64 at 64.
// ONEV: two stages of K and one of V, for 26 KB of LDS a group at head dimension 128 instead of 34.  A step is: K of the unit has landed
// (barrier); V of the unit is requested, and K of the next; scores and exponentials; V has landed (barrier); its product.  The first barrier
// comes when everyone has read the V before, the second when everyone has read the K before.  Six workgroups of two waves a CU, three waves
// a SIMD, where two stages allow four; the rule and both sides are at launch_groups.
// A third LDS stage (DMA two units ahead, waited for by count behind a bare s_barrier, which __syncthreads() does not
// allow: it waits for every outstanding DMA) changes nothing at four waves per SIMD and costs occupancy on small tiles:
// 6.77 against 6.73 ms, 108 against 98 us.
// ---------------------------------------------------------------------------
template <int D, int QW, int KG, int WPE, bool FOLLOW, int UPS, bool ONEV>
__global__ __attribute__((amdgpu_flat_work_group_size(QW * KG * 64, QW * KG * 64), amdgpu_waves_per_eu(WPE)))
void sta_fwd_group_kernel(const bf16_raw *__restrict__ q,
                                                                         const bf16_raw *__restrict__ k,
                                                                         const bf16_raw *__restrict__ v,
                                                                         bf16_raw *__restrict__ o, sta::FwdParams p,
                                                                         sta::FwdPlan plan)
{
    using L = Staged<D>;                                    // V; K is read by rows only
    using R = StagedRows<D>;
    constexpr int KS = L::KS, CB = L::CB;
    constexpr int NQ = 2;                                   // 16-query blocks per wave
    constexpr int WQ = 16 * NQ;                             // queries per wave
    constexpr int QB = QW * WQ;                             // queries per workgroup
    constexpr int UNIT_B = R::Tile + L::Tile;               // 32 keys: K, then V
    constexpr int STAGE_B = UPS * UNIT_B;                   // what a barrier makes available
    // LDS of one key group: two stages, or (ONEV) two stages of K and one of V
    constexpr int GROUP_B = ONEV ? 2 * R::Tile + L::Tile : 2 * STAGE_B;
    constexpr int K_STAGE_B = ONEV ? R::Tile : STAGE_B;     // from K of a stage to K of the other
    constexpr int V_AT = ONEV ? 2 * R::Tile : R::Tile;      // V of the first stage
    static_assert(!ONEV || (FOLLOW && UPS == 1 && L::Groups % QW == 0));
    static_assert(UPS == 1 || KG == 1, "shares of a walk are counted in single units");
    constexpr int OPS = 2 * L::Groups;                      // DMA instructions per unit
    constexpr int WAVE_OPS = (OPS + QW - 1) / QW;           // at most this many per wave
    constexpr int WAVE_OUT = WQ * L::RowB;                  // a wave's output rows
    constexpr int WAVE_PART = (CB * NQ + 1) * 1024;         // a wave's accumulators, offsets and row sums in fp32
    constexpr int MERGE_B = (KG / 2) * QW * WAVE_PART;
    constexpr int LPR = L::RowB / 16;                       // 16-byte chunks per row
    constexpr int SMEM = KG * GROUP_B > QW * WAVE_OUT ? (KG * GROUP_B > MERGE_B ? KG * GROUP_B : MERGE_B)
                                                      : (QW * WAVE_OUT > MERGE_B ? QW * WAVE_OUT : MERGE_B);
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];
    __shared__ uint32_t redo_of[QW * KG];

    const GroupItem item = group_item_of(blockIdx.x, p, plan);
    const uint32_t qblock = item.qblock;
    const size_t bh = item.bh;
    const StaBox box = item.box;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / QW, qw = wave % QW;               // key group, and which queries of the workgroup
    const int lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;

    const size_t my_row = bh * p.N + (size_t)qblock * QB + (size_t)qw * WQ;
    const char *kh = reinterpret_cast<const char *>(k + bh * p.N * D);
    const char *vh = reinterpret_cast<const char *>(v + bh * p.N * D);

    // ---- this group's share of the walk, in units of 32 keys
    BoxWalk walk;
    walk.start(box, p.n_h, p.n_w, p.P);
    const int n_all = box.count() * walk.sub_per_tile;
    const int u_lo = KG == 1 ? 0 : n_all * kg / KG;
    const int n_units = KG == 1 ? n_all : n_all * (kg + 1) / KG - u_lo;
    const int n_steps = (n_all + KG - 1) / KG;              // the largest share of any group
    auto to_share = [&]() __attribute__((always_inline)) {
        if constexpr (KG > 1) {
            const uint32_t tiles = fast_div((uint32_t)u_lo, plan.sub_per_tile);
            walk.skip(tiles, (uint32_t)u_lo - tiles * plan.sub_per_tile.d);
        }
    };
    to_share();

    // ---- DMA: instruction j of a unit brings 1 KB of K or V; wave qw of the group issues j = qw, qw + QW, ..
    const uint32_t k_lane_off = R::dma_lane_offset(lane), v_lane_off = L::dma_lane_offset(lane);
    // operand: K or V of the 32 keys from row, all of it (ONEV)
    auto issue_operand = [&](const char *head, uint32_t lane_off, uint32_t row, char *dst, int group_bytes) __attribute__((always_inline)) {
        asm volatile("" : "+v"(lane_off));
#pragma unroll
        for (int i = 0; i < L::Groups / QW; ++i) {
            const int j = qw + i * QW;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(head + (size_t)(row + L::GroupRows * j) * L::RowB + lane_off),
                                             STA_LDS_PTR(dst + j * group_bytes), 16, 0, 0);
        }
    };
    int issued = 0;                                         // units requested so far (ONEV: their K)
    uint32_t v_row = 0;                                     // ONEV: the unit whose K was requested last
    bool more = false;                                      // ONEV: a unit's K has been requested behind the V that is waited for
    auto issue_next = [&]() __attribute__((always_inline)) {
        if (issued >= n_units) return;
        if constexpr (ONEV) {
            v_row = walk.next_row;
            issue_operand(kh, k_lane_off, v_row, smem + kg * GROUP_B + (issued & 1) * K_STAGE_B, R::Group);
            walk.advance();
            ++issued;
            return;
        }
        uint32_t koff = k_lane_off, voff = v_lane_off;
        asm volatile("" : "+v"(koff), "+v"(voff));          // keep the lane offsets 32-bit next to a scalar base
        char *stage = smem + kg * GROUP_B + (issued / UPS & 1) * STAGE_B;
#pragma unroll
        for (int su = 0; su < UPS; ++su) {
            const uint32_t row = walk.next_row;
            walk.advance();
#pragma unroll
            for (int i = 0; i < WAVE_OPS; ++i) {
                const int j = qw + i * QW;
                if (OPS % QW == 0 || j < OPS) {
                    const bool is_v = j >= L::Groups;
                    const int group = j % L::Groups;
                    const char *src = (is_v ? vh : kh) + (size_t)(row + L::GroupRows * group) * L::RowB;
                    char *dst = stage + su * UNIT_B + (is_v ? R::Tile + group * L::Group : group * R::Group);
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + (is_v ? voff : koff)),
                                                     STA_LDS_PTR(dst), 16, 0, 0);
                }
            }
        }
        issued += UPS;
    };
    issue_next();

    // ---- operand read addresses (stage 0 of the group) and resident Q fragments
    const uint32_t group_addr = (uint32_t)(uintptr_t)smem + (uint32_t)(kg * GROUP_B);
    const uint32_t row_addr = R::address(group_addr, lane);
    uint32_t tr_addr[4];
    L::transposed_addresses(group_addr + V_AT, lane, tr_addr);
    bf16x8 Qr[NQ][KS];
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            Qr[qb][ks] = *reinterpret_cast<const bf16x8 *>(q + (my_row + 16 * qb + c16) * D + ks * 32 + g4 * 8);

    floatx4 Oacc[CB][NQ];                                   // channel 16*cb + 4*g4 + i of query 16*qb + c16
    // Offset of the lane's queries.  Fixed: the scores start at minus the offset (Sinit).  Following: they start at 0 and the offset
    // (off, rounded, in base 2) enters the exponent by a fused multiply-add, so that a move changes one register and no score.
    floatx4 Sinit[FOLLOW ? 1 : NQ];
    float m_run[NQ], off[NQ];
    floatx4 l_acc[NQ];                                      // row sums (a product with ones: all registers hold the same)
    auto reset = [&](float m) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
            if constexpr (!FOLLOW) Sinit[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
            off[qb] = 0.f;
            l_acc[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
            m_run[qb] = m;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) Oacc[cb][qb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
    };
    reset(0.f);
    const float c = p.scale_log2e;
    bf16x8 ones;                                            // operand of the row sums
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = static_cast<__bf16>(1.0f);
    if constexpr (!FOLLOW && UPS == 1) asm volatile("" : "+v"(ones));   // kept in registers, where there are enough, not made anew in every unit
    if constexpr (QW * KG == 12) {                          // static priorities against the age order, as in the kernel below
        if (wave >= 8) __builtin_amdgcn_s_setprio(2);
        else if (wave >= 4) __builtin_amdgcn_s_setprio(1);
    }

    // ONEV: V of the unit has landed for everyone.  Every wave of the workgroup passes here once a step.
    auto v_landed = [&]() __attribute__((always_inline)) {
        if (more) wait_dma<L::Groups / QW>();               // the next unit's K may be on its way
        else wait_dma<0>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    constexpr int kPlain = 0, kFollow = 1, kFirst = 2, kCareful = 3;
    // One unit of 32 keys whose K begins at LDS offset OFF + at (relative to the group's first stage).
    auto unit_at = [&](auto track_c, auto off_c, uint32_t at, float grow_above) __attribute__((always_inline)) {
        // kFirst: set the offsets; kFollow: move them with the scores.  kCareful: the same on scores that do not start at
        // minus the offset: they lose nothing to an old offset that was far below them (keys masked by a lowest value).
        constexpr int TRACK = decltype(track_c)::value, OFF = decltype(off_c)::value;
        uint32_t tr_at[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) tr_at[m] = tr_addr[m] + (ONEV ? 0u : at);
        floatx4 S[2][NQ];                                   // [key block][query block]
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb) S[kb][qb] = FOLLOW || TRACK == kCareful ? floatx4{0.f, 0.f, 0.f, 0.f} : Sinit[FOLLOW ? 0 : qb];
        rows_times_resident<D, OFF>(row_addr + at, Qr, S);   // K Q^T minus the offset
        if constexpr (TRACK != kPlain) {
            float mq[NQ];
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb) {
                mq[qb] = max3(S[0][qb][0], S[0][qb][1], S[0][qb][2]);
                mq[qb] = max3(mq[qb], S[0][qb][3], S[1][qb][0]);
                mq[qb] = max3(mq[qb], S[1][qb][1], S[1][qb][2]);
                mq[qb] = fmaxf(mq[qb], S[1][qb][3]);
            }
            if constexpr (TRACK == kFirst) {
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) {
                    const float row_max = quad_lane_max(mq[qb]);
                    m_run[qb] = row_max == -INFINITY ? 0.f : row_max;
                    if constexpr (FOLLOW) {
                        off[qb] = m_run[qb] * c;
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) Sinit[qb][r] = -m_run[qb];
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int r = 0; r < 4; ++r) S[kb][qb][r] -= m_run[qb];
                    }
                }
            } else if constexpr (TRACK == kCareful) {
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) {
                    const float row_max = quad_lane_max(mq[qb]);
                    const bool grown = row_max > m_run[qb] + grow_above;
                    if (__builtin_amdgcn_ballot_w64(grown) != 0) {
                        const float alpha = grown ? __builtin_amdgcn_exp2f((m_run[qb] - row_max) * c) : 1.f;
                        m_run[qb] = grown ? row_max : m_run[qb];
                        l_acc[qb] *= alpha;
                        const float alpha_settled = settled_after_transcendental(alpha);
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) scale_in_place(Oacc[cb][qb], alpha_settled);
                    }
                    const float offset = m_run[qb] == -INFINITY ? 0.f : m_run[qb];
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int r = 0; r < 4; ++r) S[kb][qb][r] -= offset;
                }
            } else {
                // a query block at a time: that halves the accumulators scaled where only one of them has grown
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) {
                    if (__builtin_amdgcn_ballot_w64(mq[qb] > m_run[qb]) == 0) continue;
                    const float m_new = fmaxf(m_run[qb], quad_lane_max(mq[qb]));      // the same in the four lanes of a query
                    float off_new = m_new * c;
                    asm volatile("" : "+v"(off_new));       // one rounded number in all its uses
                    const float alpha = __builtin_amdgcn_exp2f(off[qb] - off_new);
                    m_run[qb] = m_new;
                    off[qb] = off_new;
                    l_acc[qb] *= alpha;
                    // the old offset was so far below that the scores behind it are lost: an infinite row sum asks for the
                    // careful pass (it stays infinite; row_sums reads register 0)
                    l_acc[qb][0] = alpha == 0.f ? INFINITY : l_acc[qb][0];
                    const float alpha_settled = settled_after_transcendental(alpha);
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) scale_in_place(Oacc[cb][qb], alpha_settled);
                }
            }
        }
        StagedTransposedProduct<D, OFF> v_t;
        if constexpr (!ONEV) {
            v_t.prefetch(tr_at);
            __builtin_amdgcn_sched_barrier(0);              // the exponentials stay behind these reads
        }
        // probabilities, rounded to bf16, packed as the B operand of the PV product of their query block
        bf16x8 Pb[NQ];
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    auto exponent = [&](float x) { return FOLLOW && TRACK != kCareful ? fmaf(x, c, -off[qb]) : x * c; };
                    const float p0 = __builtin_amdgcn_exp2f(exponent(S[kb][qb][e]));
                    const float p1 = __builtin_amdgcn_exp2f(exponent(S[kb][qb][e + 1]));
                    bf16x2 pp;
                    pp[0] = static_cast<__bf16>(p0);
                    pp[1] = static_cast<__bf16>(p1);
                    Pb[qb][4 * kb + e] = pp[0];
                    Pb[qb][4 * kb + e + 1] = pp[1];
                }
        if constexpr (ONEV) {
            __builtin_amdgcn_sched_barrier(0);
            v_landed();
            v_t.prefetch(tr_at);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) l_acc[qb] = mfma_16x16x32(ones, Pb[qb], l_acc[qb]);       // sums the rounded values
        v_t.run(tr_at, Pb, Oacc);                           // O^T += V^T P^T
    };

    // One pass over the group's units; the first has been requested.  CAREFUL: every unit in the careful form, with the
    // offset moved when a score exceeds it by more than 2^8 in the exponent (FOLLOW: by anything).
    auto run_pass = [&](auto careful_c) __attribute__((always_inline)) {
        constexpr bool CAREFUL = decltype(careful_c)::value;
        constexpr int REST = CAREFUL ? kCareful : FOLLOW ? kFollow : kPlain;
        const float bound = FOLLOW || !CAREFUL ? 0.f : __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(8.0f / c)));
        auto next_stage = [&](int u) __attribute__((always_inline)) {
            // this wave's DMA for the stage must have landed, and everyone's; the other stage is free again
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if constexpr (QW > 1) __builtin_amdgcn_s_barrier();          // the stages of a single wave are its own
            asm volatile("" ::: "memory");
            if constexpr (ONEV) {
                // V of this unit, whose place everyone has read; then the next K
                if (u < n_units) issue_operand(vh, v_lane_off, v_row, smem + kg * GROUP_B + V_AT, L::Group);
                more = issued < n_units;
            }
            issue_next();
        };
        using Rest = std::integral_constant<int, REST>;
        using Stage0 = std::integral_constant<int, 0>;
        using Stage1 = std::integral_constant<int, STAGE_B>;
        auto stage_at = [&](auto first_c, auto stage_c, uint32_t at, int u) __attribute__((always_inline)) {
            next_stage(u);
            if (KG == 1 || u < n_units) unit_at(first_c, stage_c, at, bound);
            else if constexpr (ONEV) v_landed();
            if constexpr (UPS == 2) unit_at(Rest{}, std::integral_constant<int, decltype(stage_c)::value + UNIT_B>{}, at, bound);
        };
        if constexpr (!CAREFUL) stage_at(std::integral_constant<int, kFirst>{}, Stage0{}, 0u, 0);
        // The stage is part of the read instructions, not an addition to each of five addresses.  (Added in the careful pass, and where
        // the offset follows: there the unrolled loop copies the accumulators from one half to the other, 29 registers of scratch.)
        if constexpr (!CAREFUL && !FOLLOW) {
#pragma unroll 1
            for (int u = UPS; u < n_steps; u += 2 * UPS) {
                stage_at(Rest{}, Stage1{}, 0u, u);
                if (u + UPS < n_steps) stage_at(Rest{}, Stage0{}, 0u, u + UPS);
            }
        } else {
#pragma unroll 1
            for (int u = CAREFUL ? 0 : UPS; u < n_steps; u += UPS) stage_at(Rest{}, Stage0{}, (uint32_t)((u / UPS & 1) * K_STAGE_B), u);
        }
    };
    float l_tot[NQ];
    auto row_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) l_tot[qb] = l_acc[qb][0];
    };
    run_pass(std::false_type{});
    row_sums();
    // Done again: row sums beyond 2^96 (infinite where an offset has jumped) and below 2^-64, which only a group has whose
    // first keys all score minus infinity (its offset is 0 then).
    constexpr float kRedoAbove = 79228162514264337593543950336.f, kRedoBelow = 5.42101086242752217e-20f;
    // Accumulators that have left the range; those of key groups from 2^125 on, so that the sum of four stays in it.
    constexpr uint32_t kRedoBits = KG == 1 ? 0x7f800000u : 0x7e000000u;
    // The sum of their absolute values is at least their largest and not a number where one of them is not; it is tested on the
    // bit pattern, which a NaN passes.  (That the sum leaves the range before any of them costs a second pass, no result.)
    float o_sum[4] = {0.f, 0.f, 0.f, 0.f};
    bool redo = false;
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
        redo = redo || !(l_tot[qb] < kRedoAbove) || ((KG == 1 || n_units > 0) && l_tot[qb] < kRedoBelow);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) o_sum[r] += __builtin_fabsf(Oacc[cb][qb][r]);
    }
    const uint32_t o_bits = __float_as_uint((o_sum[0] + o_sum[1]) + (o_sum[2] + o_sum[3])) & 0x7fffffffu;
    // Every wave leaves its answer in LDS and sees everyone's behind one barrier, which also ends all reads of the stages.
    // (__syncthreads_or took 0.55 us of a 64-token item's 11, with the maximum over the bit patterns that was formed here.)
    const bool wave_redo = __builtin_amdgcn_ballot_w64(redo || o_bits >= kRedoBits) != 0;
    if (lane == 0) redo_of[wave] = wave_redo;
    __syncthreads();
    const uint32_t others = lane < QW * KG ? redo_of[lane] : 0u;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(others != 0) != 0, 0)) {
        reset(-INFINITY);
        walk.start(box, p.n_h, p.n_w, p.P);
        to_share();
        issued = 0;
        issue_next();
        run_pass(std::true_type{});
        row_sums();
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) off[qb] = m_run[qb] * c;
        __syncthreads();
    }

    // ---- merge of the key groups: the upper half of the remaining groups hands its accumulators, offsets and row sums
    // to the lower half through LDS until one is left, always in the same order
    // (a group without units or with scores of minus infinity only: an offset below every other, finite so that two such
    // groups can be merged)
    float m2[NQ];                                           // offsets in base-2 units
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) m2[qb] = (KG > 1 && n_units == 0) ? -3.0e38f : fmaxf(FOLLOW ? off[qb] : m_run[qb] * c, -3.0e38f);
    if constexpr (KG > 1) {
#pragma unroll
        for (int n = KG; n > 1; n = (n + 1) / 2) {
            const int half = (n + 1) / 2;                   // groups half .. n-1 give, groups 0 .. n-1-half take
            if (n != KG) __syncthreads();                   // the previous round has been read
            if (kg >= half && kg < n) {
                char *to = smem + ((kg - half) * QW + qw) * WAVE_PART + lane * 16;
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) *reinterpret_cast<floatx4 *>(to + (qb * CB + cb) * 1024) = Oacc[cb][qb];
                *reinterpret_cast<floatx4 *>(to + NQ * CB * 1024) = floatx4{m2[0], m2[1], l_tot[0], l_tot[1]};
            }
            __syncthreads();
            if (kg + half < n) {
                const char *from = smem + (kg * QW + qw) * WAVE_PART + lane * 16;
                const floatx4 ml = *reinterpret_cast<const floatx4 *>(from + NQ * CB * 1024);
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) {
                    const float m_new = fmaxf(m2[qb], ml[qb]);
                    const float wa = __builtin_amdgcn_exp2f(m2[qb] - m_new), wb = __builtin_amdgcn_exp2f(ml[qb] - m_new);
                    m2[qb] = m_new;
                    l_tot[qb] = l_tot[qb] * wa + ml[NQ + qb] * wb;
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        const floatx4 x = *reinterpret_cast<const floatx4 *>(from + (qb * CB + cb) * 1024);
#pragma unroll
                        for (int r = 0; r < 4; ++r) Oacc[cb][qb][r] = Oacc[cb][qb][r] * wa + x[r] * wb;
                    }
                }
            }
        }
        __syncthreads();
        if (kg != 0) return;
    }

    // ---- finalize (the first group): rows through LDS, whole rows to memory with streaming stores
    if (p.lse != nullptr && g4 == 0) {
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) p.lse[my_row + 16 * qb + c16] = m2[qb] * 0.6931471805599453f + __logf(l_tot[qb]);
    }
    char *rows = smem + qw * WAVE_OUT;
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
        const float inv = 1.f / l_tot[qb];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            bf16x4 ov;
#pragma unroll
            for (int t = 0; t < 4; ++t) ov[t] = static_cast<__bf16>(Oacc[cb][qb][t] * inv);
            const int chunk = 2 * cb + (g4 >> 1);
            *reinterpret_cast<bf16x4 *>(rows + (16 * qb + c16) * L::RowB + ((chunk ^ (c16 & (LPR - 1))) << 4) + 8 * (g4 & 1)) = ov;
        }
    }
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    char *out = reinterpret_cast<char *>(o + my_row * D);
#pragma unroll
    for (int i = 0; i < WAVE_OUT / 1024; ++i) {
        const int r = L::GroupRows * i + lane / LPR, cpos = lane % LPR;
        const u32x4 x = *reinterpret_cast<const u32x4 *>(rows + r * L::RowB + ((cpos ^ (r & (LPR - 1))) << 4));
        __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(out + (size_t)r * L::RowB + (cpos << 4)));
    }
}

// ---------------------------------------------------------------------------
// The small launches' kernel ("solo"): a workgroup is KG waves that share NQ blocks of 16 queries and take one KG-th of the walk
// each, with LDS of their own.  No barrier until the end, so that the waves drift apart and one computes where another waits; and
// a wave's requests need no second stage: K of the next unit is requested as soon as K of this one has been read, V likewise,
// each waited for by count (requests complete in order).  At the end every wave leaves its accumulators, offsets and row sums in
// its LDS, and all of them merge one share of the channels each, in a fixed order: two barriers, whatever KG is.
//
// What bounds it: the latencies of one wave's unit where there are few waves (1200 cycles a unit at one wave per SIMD in the kernel
// above, which had all its waves in the same phase behind one barrier per unit), the 64 bytes per cycle that a CU takes from L2 where
// there are many (8 KB a unit at head dimension 64, for 32 queries; hence NQ = 4, 64 queries, where the walk is long), and the fixed
// part of a launch, about 6 us: arguments, Q and the first K from memory, the merge, the way out.  In us, the kernel above and this
// one: 4x12x24 in 96-token tiles, one head, 64 16.6, 9.1, 128 23.6, 13.1; 12x24x24 in 384-token tiles, one head, 64 24.2, 14.4, 128
// 35.0, 23.1; 18x24x24, one head of 64 24.4, 19.5; 10x30x56 in 96-token tiles, 64, three heads 84, 62.
//
// The scores start at 0 and the offset enters the exponent by a fused multiply-add (one instruction per score, as the
// multiplication it replaces): six registers less than scores that start at minus the offset.
// ---------------------------------------------------------------------------
template <int D, int NQ, int KG, int WPE, bool FOLLOW>
__global__ __attribute__((amdgpu_flat_work_group_size(KG * 64, KG * 64), amdgpu_waves_per_eu(WPE)))
void sta_fwd_solo_kernel(const bf16_raw *__restrict__ q, const bf16_raw *__restrict__ k, const bf16_raw *__restrict__ v,
                         bf16_raw *__restrict__ o, sta::FwdParams p, sta::FwdPlan plan)
{
    using L = Staged<D>;                                    // V; K is read by rows only
    using R = StagedRows<D>;
    constexpr int KS = L::KS, CB = L::CB;
    constexpr int QB = 16 * NQ;                             // queries of the workgroup
    constexpr int GROUPS = L::Groups;                       // DMA instructions per operand of a unit
    constexpr int SLICES = CB * NQ;                         // 16x16 blocks of an accumulator, 1 KB each
    constexpr int UNIT_B = R::Tile + L::Tile;
    constexpr int REGION = UNIT_B > SLICES * 1024 ? UNIT_B : SLICES * 1024;    // LDS of a wave: K, then V; at the end its accumulators
    constexpr int PER_WAVE = SLICES / KG;                   // of them that a wave merges
    static_assert(SLICES % KG == 0 && CB % PER_WAVE == 0, "merge");
    constexpr int STATS = KG * REGION;                      // offset and row sum of every group's queries
    constexpr int FLAGS = STATS + KG * QB * 8;
    constexpr int OUT = (FLAGS + KG * 4 + 15) / 16 * 16;
    __shared__ __attribute__((aligned(1024))) char smem[OUT + QB * L::RowB];

    const GroupItem item = group_item_of(blockIdx.x, p, plan);
    const size_t bh = item.bh;
    const StaBox box = item.box;
    const int tid = threadIdx.x;
    const int kg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, c16 = lane & 15, g4 = lane >> 4;
    const size_t my_row = bh * p.N + (size_t)item.qblock * QB;
    const char *kh = reinterpret_cast<const char *>(k + bh * p.N * D);
    const char *vh = reinterpret_cast<const char *>(v + bh * p.N * D);

    BoxWalk walk;
    int n_units;
    auto start_walk = [&]() __attribute__((always_inline)) {
        walk.start(box, p.n_h, p.n_w, p.P);
        const int n_all = box.count() * walk.sub_per_tile;
        const int lo = n_all * kg / KG;
        n_units = n_all * (kg + 1) / KG - lo;
        const uint32_t tiles = fast_div((uint32_t)lo, plan.sub_per_tile);
        walk.skip(tiles, (uint32_t)lo - tiles * plan.sub_per_tile.d);
    };
    start_walk();

    char *region = smem + kg * REGION;
    const uint32_t k_lane_off = R::dma_lane_offset(lane), v_lane_off = L::dma_lane_offset(lane);
    auto issue_k = [&](uint32_t row) __attribute__((always_inline)) {
        uint32_t off = k_lane_off;
        asm volatile("" : "+v"(off));                       // keep the lane offset 32-bit next to a scalar base
#pragma unroll
        for (int i = 0; i < GROUPS; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(kh + (size_t)(row + L::GroupRows * i) * L::RowB + off),
                                             STA_LDS_PTR(region + i * R::Group), 16, 0, 0);
    };
    auto issue_v = [&](uint32_t row) __attribute__((always_inline)) {
        uint32_t off = v_lane_off;
        asm volatile("" : "+v"(off));
#pragma unroll
        for (int i = 0; i < GROUPS; ++i)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(vh + (size_t)(row + L::GroupRows * i) * L::RowB + off),
                                             STA_LDS_PTR(region + R::Tile + i * L::Group), 16, 0, 0);
    };
    if (n_units > 0) {
        issue_k(walk.next_row);
        issue_v(walk.next_row);
    }

    const uint32_t region_addr = (uint32_t)(uintptr_t)smem + (uint32_t)(kg * REGION);
    const uint32_t row_addr = R::address(region_addr, lane);
    uint32_t tr_addr[4];
    L::transposed_addresses(region_addr + R::Tile, lane, tr_addr);
    bf16x8 Qr[NQ][KS];
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            Qr[qb][ks] = *reinterpret_cast<const bf16x8 *>(q + (my_row + 16 * qb + c16) * D + ks * 32 + g4 * 8);

    floatx4 Oacc[CB][NQ];                                   // channel 16*cb + 4*g4 + i of query 16*qb + c16
    float m_run[NQ], off[NQ];                               // largest score, in its own units and (rounded) in base 2
    floatx4 l_acc[NQ];                                      // row sums
    auto reset = [&](float m) __attribute__((always_inline)) {
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
            l_acc[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
            m_run[qb] = m;
            off[qb] = 0.f;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) Oacc[cb][qb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
    };
    reset(0.f);
    const float c = p.scale_log2e;

    auto run_pass = [&](auto careful_c) __attribute__((always_inline)) {
        constexpr bool CAREFUL = decltype(careful_c)::value;
        const float bound = FOLLOW || !CAREFUL ? 0.f : __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(8.0f / c)));
#pragma unroll 1
        for (int u = 0; u < n_units; ++u) {
            const bool more = u + 1 < n_units;
            wait_dma<GROUPS>();                             // K of this unit; its V has been requested behind it
            floatx4 S[2][NQ];                               // [key block][query block]
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) S[kb][qb] = floatx4{0.f, 0.f, 0.f, 0.f};
            rows_times_resident<D, 0>(row_addr, Qr, S);     // K Q^T
            walk.advance();
            if (more) issue_k(walk.next_row);
            if (CAREFUL || FOLLOW || u == 0) {
                float mq[NQ];
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) {
                    mq[qb] = max3(S[0][qb][0], S[0][qb][1], S[0][qb][2]);
                    mq[qb] = max3(mq[qb], S[0][qb][3], S[1][qb][0]);
                    mq[qb] = max3(mq[qb], S[1][qb][1], S[1][qb][2]);
                    mq[qb] = fmaxf(mq[qb], S[1][qb][3]);
                }
                if constexpr (CAREFUL) {
#pragma unroll
                    for (int qb = 0; qb < NQ; ++qb) {
                        const float row_max = quad_lane_max(mq[qb]);
                        const bool grown = row_max > m_run[qb] + bound;
                        if (__builtin_amdgcn_ballot_w64(grown) != 0) {
                            const float alpha = grown ? __builtin_amdgcn_exp2f((m_run[qb] - row_max) * c) : 1.f;
                            m_run[qb] = grown ? row_max : m_run[qb];
                            l_acc[qb] *= alpha;
                            const float alpha_settled = settled_after_transcendental(alpha);
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb) scale_in_place(Oacc[cb][qb], alpha_settled);
                        }
                        // subtracted, exactly 0 for the largest score: c times a lowest number and its rounding are far apart
                        const float offset = m_run[qb] == -INFINITY ? 0.f : m_run[qb];
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int r = 0; r < 4; ++r) S[kb][qb][r] -= offset;
                    }
                } else if constexpr (!FOLLOW) {
#pragma unroll
                    for (int qb = 0; qb < NQ; ++qb) {
                        const float row_max = quad_lane_max(mq[qb]);
                        m_run[qb] = row_max == -INFINITY ? 0.f : row_max;
                        off[qb] = m_run[qb] * c;
                    }
                } else {
                    const bool first = u == 0;              // sets the offset, which is 0 until then
#pragma unroll
                    for (int qb = 0; qb < NQ; ++qb) {
                        if (!first && __builtin_amdgcn_ballot_w64(mq[qb] > m_run[qb]) == 0) continue;
                        const float row_max = quad_lane_max(mq[qb]);
                        const float m_new = first ? (row_max == -INFINITY ? 0.f : row_max) : fmaxf(m_run[qb], row_max);
                        float off_new = m_new * c;
                        asm volatile("" : "+v"(off_new));   // one rounded number in all its uses
                        const float alpha = first ? 1.f : __builtin_amdgcn_exp2f(off[qb] - off_new);
                        m_run[qb] = m_new;
                        off[qb] = off_new;
                        l_acc[qb] *= alpha;
                        // an offset that jumped so far that what lay behind it is lost: an infinite row sum asks for the careful pass
                        l_acc[qb][0] = alpha == 0.f ? INFINITY : l_acc[qb][0];
                        const float alpha_settled = settled_after_transcendental(alpha);
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) scale_in_place(Oacc[cb][qb], alpha_settled);
                    }
                }
            }
            bf16x8 Pb[NQ];
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = CAREFUL ? S[kb][qb][e] * c : fmaf(S[kb][qb][e], c, -off[qb]);
                        Pb[qb][4 * kb + e] = static_cast<__bf16>(__builtin_amdgcn_exp2f(x));
                    }
            bf16x8 ones;
#pragma unroll
            for (int e = 0; e < 8; ++e) ones[e] = static_cast<__bf16>(1.0f);
            if (more) wait_dma<GROUPS>();                   // V of this unit; the next unit's K has been requested behind it
            else wait_dma<0>();
            StagedTransposedProduct<D, 0> v_t;
            v_t.prefetch(tr_addr);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb) l_acc[qb] = mfma_16x16x32(ones, Pb[qb], l_acc[qb]);       // sums the rounded values
            v_t.run(tr_addr, Pb, Oacc);                     // O^T += V^T P^T
            if (more) issue_v(walk.next_row);
        }
    };

    // (In the first pass c times the scores is exact inside the fused multiply-add and the offset rounded: what is between them is a
    // factor common to a row's probabilities and its sum, which shows as an extreme row sum where it is extreme.)
    // Row sums and accumulators of this wave to LDS; what asks for the careful pass is as in the kernel above.
    constexpr float kRedoAbove = 79228162514264337593543950336.f, kRedoBelow = 5.42101086242752217e-20f;
    // 2^123, 2^124, 2^125: the sum of all groups stays in range
    constexpr uint32_t kRedoBits = KG > 8 ? 0x7d000000u : KG > 4 ? 0x7d800000u : 0x7e000000u;
    auto leave_partial = [&](bool careful) __attribute__((always_inline)) {
        float o_sum[4] = {0.f, 0.f, 0.f, 0.f};
        bool redo = false;
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
            redo = redo || !(l_acc[qb][0] < kRedoAbove) || (n_units > 0 && l_acc[qb][0] < kRedoBelow);
            const float m2 = n_units == 0 ? -3.0e38f : fmaxf(careful ? m_run[qb] * c : off[qb], -3.0e38f);
            if (g4 == 0) *reinterpret_cast<float2 *>(smem + STATS + (kg * QB + 16 * qb + c16) * 8) = make_float2(m2, l_acc[qb][0]);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
                for (int r = 0; r < 4; ++r) o_sum[r] += __builtin_fabsf(Oacc[cb][qb][r]);
                *reinterpret_cast<floatx4 *>(region + (qb * CB + cb) * 1024 + lane * 16) = Oacc[cb][qb];
            }
        }
        const uint32_t o_bits = __float_as_uint((o_sum[0] + o_sum[1]) + (o_sum[2] + o_sum[3])) & 0x7fffffffu;
        const uint64_t any = __builtin_amdgcn_ballot_w64(redo || o_bits >= kRedoBits);
        if (lane == 0) *reinterpret_cast<uint32_t *>(smem + FLAGS + 4 * kg) = any != 0;
    };
    run_pass(std::false_type{});
    leave_partial(false);
    __syncthreads();
    const uint32_t flag = lane < KG ? *reinterpret_cast<const uint32_t *>(smem + FLAGS + 4 * lane) : 0u;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(flag != 0) != 0, 0)) {
        __syncthreads();                                    // everyone has seen the flags and is about to start again
        reset(-INFINITY);
        start_walk();
        if (n_units > 0) {
            issue_k(walk.next_row);
            issue_v(walk.next_row);
        }
        run_pass(std::true_type{});
        leave_partial(true);
        __syncthreads();
    }

    // ---- merge: every wave sums the groups' parts of its slices of the accumulators, in ascending order
    const int first = kg * PER_WAVE, qb = first / CB;
    const float2 *stats = reinterpret_cast<const float2 *>(smem + STATS) + 16 * qb + c16;
    float m = -INFINITY, l = 0.f, weight[KG];
#pragma unroll
    for (int g = 0; g < KG; ++g) m = fmaxf(m, stats[g * QB].x);
#pragma unroll
    for (int g = 0; g < KG; ++g) {
        weight[g] = __builtin_amdgcn_exp2f(stats[g * QB].x - m);
        l += stats[g * QB].y * weight[g];
    }
    const float inv = 1.f / l;
#pragma unroll
    for (int j = 0; j < PER_WAVE; ++j) {
        const int cb = first % CB + j;
        floatx4 sum = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            const floatx4 x = *reinterpret_cast<const floatx4 *>(smem + g * REGION + (first + j) * 1024 + lane * 16);
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[r] = fmaf(x[r], weight[g], sum[r]);
        }
        bf16x4 ov;
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = static_cast<__bf16>(sum[r] * inv);
        *reinterpret_cast<bf16x4 *>(smem + OUT + (16 * qb + c16) * L::RowB + (16 * cb + 4 * g4) * 2) = ov;
    }
    if (p.lse != nullptr && first % CB == 0 && g4 == 0) p.lse[my_row + 16 * qb + c16] = m * 0.6931471805599453f + __logf(l);
    __syncthreads();
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    char *out = reinterpret_cast<char *>(o + my_row * D);
    for (int i = tid * 16; i < QB * L::RowB; i += KG * 64 * 16)
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4 *>(smem + OUT + i), reinterpret_cast<u32x4 *>(out + i));
}

// Head dimension 128, tiles of 128 tokens' multiples: one kernel without key groups, 32-key sub-blocks.  On this chip the run
// time on real data follows the energy of the instruction stream (the package sits at its power limit and lowers
// the clock), and the 16x16x32 shape is the cheaper one per flop: it reads and writes 4 accumulator registers per
// 16 Kflop where 32x32x16 moves 16 per 32 Kflop.  Measured with nothing but matrix instructions on N(0,1) operands:
// 1969 TFLOP/s against 1783 at two waves per SIMD (both 2440-2450 on constant operands), 1901 against 1443 at the
// three waves per SIMD this kernel runs with (2412 against 1839 on constant operands).
// Layout: a lane holds column c16 = lane & 15 of a 16x16 result (a query) and rows 4*g4 .. 4*g4+3 (g4 = lane >> 4);
// of an operand it holds row/column c16 and the k-chunk 8*g4 .. 8*g4+7.  A wave's 32 queries are two query blocks;
// every K and V fragment read from LDS feeds both.
// LDS layout of a staged sub-block: groups of 4 rows (1 KB, what one DMA instruction fills), the groups
// kKGroup = 1024 + 64 bytes apart for K and kVGroup = 1024 + 32 bytes apart for V; inside a group the 16-byte chunk c
// of row j (0..3) sits at position c ^ j for K and c ^ (j << 2) for V.  A row is 256 bytes = all 64 banks, so the
// rows of a group start at the same bank and it is the XOR that keeps them apart, while the padding turns
// consecutive groups by 16 (K) or 8 (V) banks.  Measured with the bank-conflict counter, both reads are free of
// conflicts:
//  - a 16-byte read is served 16 lanes at a time, and those are not 16 consecutive lanes but lanes 0-7 together
//    with lanes 24-31 (then 8-15 with 16-23, and the same in the upper half): rows 0..7 at chunk x, rows 8..15 at
//    chunk x ^ 1.  Four groups of four rows, each group in its own 64 bytes of the 256;
//  - a transposing 8-byte read is served 32 lanes at a time: 8 consecutive rows, two neighbouring chunks of each.
//    The rows of a group take different quarters of the 256 bytes, the second group the other 32 bytes of each.
// The point of this layout over a plain XOR swizzle of whole rows: the k-step of a K read (64 bytes) and the odd
// channel blocks of a V read (32 bytes) are offsets that go into the instruction, and the XOR touches only two
// address bits of V.  Per sub-block that leaves five address computations where a whole-row swizzle needs
// thirteen, and on this chip every vector instruction saved is energy, hence time.
constexpr int kKGroup = 1024 + 64, kVGroup = 1024 + 32;

template <int NW, int KB, int STAGES, int MINB>
__global__ __launch_bounds__(NW * 64, MINB) void sta_fwd_x32_kernel(const bf16_raw *__restrict__ q,
                                                                 const bf16_raw *__restrict__ k,
                                                                 const bf16_raw *__restrict__ v,
                                                                 bf16_raw *__restrict__ o, sta::FwdParams p,
                                                                 sta::FwdPlan plan)
{
    constexpr int D = 128;
    static_assert(KB == 32, "keys per sub-block");
    constexpr int QB = NW * 32;                    // queries per workgroup: one 32-query block per wave
    constexpr int KS = D / 32;                     // k-steps of 32 channels in S^T = K Q^T
    constexpr int CB = D / 16;                     // 16-channel blocks of O^T
    constexpr int ROWB = D * 2;                    // bytes per key row in LDS
    constexpr int GROUPS = KB / 4;                 // 4-row groups of a sub-block = DMA instructions per operand
    constexpr int K_BYTES = GROUPS * kKGroup, V_BYTES = GROUPS * kVGroup;
    constexpr int STAGE_BYTES = K_BYTES + V_BYTES; // K then V
    constexpr int INSTR = GROUPS;
    constexpr int WANT_LOADERS = NW < 4 ? NW : (NW < 8 ? 4 : 8);
    constexpr int LOADERS = WANT_LOADERS < INSTR ? WANT_LOADERS : INSTR;     // waves 0 .. LOADERS-1 issue the DMA
    constexpr int LOADS = INSTR / LOADERS;         // ... this many instructions per operand each
    constexpr int RPI = 1024 / ROWB;               // key rows per DMA instruction (4 or 8)
    constexpr int IPB = 16 / RPI;                  // DMA instructions per block of 16 rows
    constexpr int LPR = ROWB / 16;                 // lanes (16-byte chunks) per row
    static_assert(KB % 32 == 0 && INSTR % LOADERS == 0 && LOADS >= 1 && LOADERS <= NW && LOADERS % IPB == 0,
                  "sub-block shape");
    static_assert(STAGES == 2, "LDS stages");

    // the K/V stages; at the end every wave passes its 32 output rows (32 * ROWB bytes) through the same memory
    constexpr int OUT_BYTES = QB * ROWB;
    __shared__ __attribute__((aligned(1024))) char smem[STAGES * STAGE_BYTES > OUT_BYTES ? STAGES * STAGE_BYTES : OUT_BYTES];

    // ---- work item (see group_item_of), possibly one part of a split item
    uint32_t item_id = blockIdx.x, part = 0;
    const bool is_part = blockIdx.x >= p.split_first;
    if (is_part) {
        const uint32_t idx = blockIdx.x - p.split_first;
        item_id = p.split_first + idx / p.split_parts;
        part = idx - (item_id - p.split_first) * p.split_parts;
    }
    const GroupItem item = group_item_of(item_id, p, plan);
    const uint32_t qblock = item.qblock;
    const size_t bh = item.bh;
    const StaBox box = item.box;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int c16 = lane & 15;                     // column of a 16x16 result this lane holds (a query)
    const int g4 = lane >> 4;                      // its rows 4*g4 .. 4*g4+3; k-chunk 8*g4 .. 8*g4+7 of an operand

    const bf16_raw *qh = q + (bh * p.N + (size_t)qblock * QB + (size_t)wave * 32) * D;
    const char *kh = reinterpret_cast<const char *>(k + bh * p.N * D);
    const char *vh = reinterpret_cast<const char *>(v + bh * p.N * D);

    // ---- DMA loads.  Each wave-wide 16 B/lane instruction fills 1 KB of LDS = one group of 4 key rows (a lane's
    // LDS slot is fixed by the hardware: base + 16*lane), so the XOR is applied on the global side: the lane
    // fetches the logical chunk that belongs at its slot.  Loading wave w takes the groups LOADS*w .. +LOADS-1.
    // A lane's offset inside its group is the same for all its instructions and the rest of the address is
    // wave-uniform: one 32-bit lane offset per operand on top of a scalar base, no vector arithmetic per load.
    static_assert(RPI == 4 && LPR == 16, "a DMA instruction fills one group of four rows");
    const uint32_t k_lane_off = (uint32_t)((lane >> 4) * ROWB + (((lane & 15) ^ (lane >> 4)) << 4));
    const uint32_t v_lane_off = (uint32_t)((lane >> 4) * ROWB + (((lane & 15) ^ ((lane >> 4) << 2)) << 4));
    auto issue_loads = [&](int stage, size_t key_byte_base) {
        char *sdst = smem + stage * STAGE_BYTES;                           // only waves < LOADERS get here
        uint32_t koff = k_lane_off, voff = v_lane_off;
        asm volatile("" : "+v"(koff), "+v"(voff));      // keep the lane offsets 32-bit next to a scalar base
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int group = LOADS * wave + i;
            const size_t gbase = key_byte_base + (size_t)group * (4 * ROWB);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(kh + gbase + koff),
                                             STA_LDS_PTR(sdst + group * kKGroup), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(vh + gbase + voff),
                                             STA_LDS_PTR(sdst + K_BYTES + group * kVGroup), 16, 0, 0);
        }
    };

    // ---- per-lane constants of the operand reads (stage 0; the other is in the read instructions, added in the careful pass)
    // K (A operand of S^T = K Q^T, 16 keys x 32 channels): key row 16*kb + c16 = row c16 & 3 of group 4*kb + (c16 >> 2),
    // logical chunk 4*ks + g4.  The XOR reaches only the two low bits of the chunk, so kb and ks are immediates.
    const uint32_t smem_addr = (uint32_t)(uintptr_t)smem;
    const uint32_t k_base = smem_addr + (uint32_t)((c16 >> 2) * kKGroup + (c16 & 3) * ROWB + ((g4 ^ (c16 & 3)) << 4));
    // V (A operand of O^T += V^T P^T, 16 channels x 32 keys) through the transposing read: within each block of 16
    // lanes, lane 4*j4 + s4 supplies 4 channels (4*s4..4*s4+3 of the block's 16) of key row 4*g4 + j4 = row j4 of
    // group g4; lane i then receives channel i of those four rows.  The second read of a pair takes the rows 16
    // (four groups) further down.  Logical chunk 2*cb + (s4 >> 1): the XOR with j4 << 2 reaches the two high bits
    // of the chunk = cb >> 1, one address per value of it; cb & 1 is 32 bytes in the instruction.
    const int j4 = (lane & 15) >> 2, s4 = lane & 3;
    uint32_t v_addr[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
        v_addr[m] = smem_addr + (uint32_t)(K_BYTES + g4 * kVGroup + j4 * ROWB + ((((m ^ j4) << 2) | (s4 >> 1)) << 4) + 8 * (s4 & 1));

    // ---- Q fragments (B operand of S^T: query 16*qb + c16, channels 32*ks + 8*g4 ..), resident in registers.
    // Multiplied by scale * log2(e) here, once, and rounded to bf16 again, they would make the matrix product deliver
    // base-2 exponents and save the 16 multiplications per lane and sub-block.  That was 4.5 % faster (11.43 against
    // 11.95 ms at 115,200 tokens, window 3x3x3), but the second rounding of Q puts a relative error of up to 2^-9 on every
    // term of a score: with scores of a few tens the probabilities are off by a percent and the output error leaves the
    // 2e-2 bound (0.07 on the growing-maximum test).
    bf16x8 Qr[2][KS];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            Qr[qb][ks] = *reinterpret_cast<const bf16x8 *>(qh + (size_t)(16 * qb + c16) * D + ks * 32 + g4 * 8);

    // O^T accumulators: Oacc[cb][qb][i] = channel 16*cb + 4*g4 + i of query 16*qb + c16
    floatx4 Oacc[CB][2];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) Oacc[cb][qb] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Offset m per query, in the units of the scores (raw dot products).  The score
    // accumulators START at -m (Sinit, the value replicated over the four registers of an accumulator), so what the
    // matrix instructions deliver is s - m and the exponential needs one multiplication by scale * log2(e) per
    // element instead of a fused multiply-add plus bookkeeping.  m is 0 while the first sub-block's scores are formed, which
    // then set it, and never decreases afterwards.
    float m_run[2] = {0.f, 0.f};
    floatx4 Sinit[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
    // Row sums, a matrix product with an operand of ones (all registers of a lane hold the sum of its query).  Two matrix instructions a
    // sub-block where eight v_dot2 had to go through the matrix pipe as well: 10,748 -> 10,649 us, and 10,116 -> 9784 over the whole grid.
    floatx4 l_acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};

    const int sub_per_tile = p.P / KB;
    const int n_all = box.count() * sub_per_tile;           // sub-blocks of the whole item
    // (the 64-bit divisions are done in vector registers; the results are wave-uniform and go back to scalar ones)
    const int iter_lo = is_part ? __builtin_amdgcn_readfirstlane((int)((long long)n_all * part / p.split_parts)) : 0;
    const int n_iter = (is_part ? __builtin_amdgcn_readfirstlane((int)((long long)n_all * (part + 1) / p.split_parts)) : n_all) - iter_lo;
    // Order in which the key tiles of the box are visited.  Along each axis the box [lo, hi] holds e = hi-lo+1
    // consecutive tiles, hence exactly one tile of every residue class mod e; the walk takes them in the order
    // of that residue (k mod e = 0, 1, ..), i.e. it starts inside the box and wraps from hi to lo.  Query tiles
    // that are neighbours along an axis have boxes shifted by one tile: with this order they reach each key
    // tile they share at the SAME step of their walks, so workgroups resident on an XCD at one time read the
    // same K/V tiles at about the same time and find them in that XCD's L2.  (Walking every box from its own lo
    // makes neighbours read a shared tile at different steps; the L2 is far too small to keep it that long.)
    const int e_t = box.t.hi - box.t.lo + 1, e_h = box.h.hi - box.h.lo + 1, e_w = box.w.hi - box.w.lo + 1;
    const int start_t = box.t.lo + (e_t - box.t.lo % e_t) % e_t;
    const int start_h = box.h.lo + (e_h - box.h.lo % e_h) % e_h;
    const int start_w = box.w.lo + (e_w - box.w.lo % e_w) % e_w;
    int it_t, it_h, it_w, it_s;
    int left_h, left_w;                     // tiles still to visit in the current h-cycle / w-cycle
    auto row_start = [&]() -> size_t {      // byte offset of key tile (it_t, it_h, it_w) inside the head
        const size_t kt = ((size_t)it_t * p.n_h + it_h) * p.n_w + it_w;
        return kt * p.P * ROWB;
    };
    size_t next_base;
    auto start_walk = [&]() __attribute__((always_inline)) {
        it_t = start_t; it_h = start_h; it_w = start_w;
        left_h = e_h; left_w = e_w;
        // a part starts iter_lo sub-blocks into the walk: whole tiles first, then sub-blocks inside the tile
        for (int skip = iter_lo / sub_per_tile; skip > 0; --skip) {
            if (++it_w > box.w.hi) it_w = box.w.lo;
            if (--left_w == 0) {
                left_w = e_w;
                it_w = start_w;
                if (++it_h > box.h.hi) it_h = box.h.lo;
                if (--left_h == 0) {
                    left_h = e_h;
                    it_h = start_h;
                    if (++it_t > box.t.hi) it_t = box.t.lo;
                }
            }
        }
        it_s = iter_lo % sub_per_tile;
        next_base = row_start() + (size_t)it_s * KB * ROWB;
    };
    auto advance = [&]() __attribute__((always_inline)) {
        next_base += (size_t)KB * ROWB;
        if (++it_s == sub_per_tile) {
            it_s = 0;
            if (++it_w > box.w.hi) it_w = box.w.lo;
            if (--left_w == 0) {
                left_w = e_w;
                it_w = start_w;
                if (++it_h > box.h.hi) it_h = box.h.lo;
                if (--left_h == 0) {
                    left_h = e_h;
                    it_h = start_h;
                    if (++it_t > box.t.hi) it_t = box.t.lo;
                }
            }
            next_base = row_start();
        }
    };

    // The SIMD's arbiter prefers its oldest wave, and a wave whose next instruction is an MFMA waiting for the
    // matrix pipe holds the vector issue port meanwhile: the softmax arithmetic of the younger waves of a SIMD
    // then waits behind the older waves' matrix phases.  Static priorities against the age order (waves w, w+4,
    // w+8 share a SIMD) even this out.  Measured in one call: 12.41 -> 12.22 ms, and 9.50 -> 9.24 ms on constant
    // inputs, where the clock does not move.
    if constexpr (NW == 12) {
        if (wave >= 8) __builtin_amdgcn_s_setprio(2);
        else if (wave >= 4) __builtin_amdgcn_s_setprio(1);
    }

    // ---- pipeline: up to STAGES-1 sub-blocks are in flight.  (it_t, it_h, it_w, it_s) always names the next
    // sub-block to request; `issued` counts the requests made so far.
    int issued;
    auto issue_next = [&]() __attribute__((always_inline)) {
        if (issued < n_iter) {
            if (wave < LOADERS) issue_loads(issued % STAGES, next_base);
            advance();
            ++issued;
        }
    };
    auto start_pipeline = [&]() __attribute__((always_inline)) {
        start_walk();
        issued = 0;
#pragma unroll
        for (int s = 0; s < STAGES - 1; ++s) issue_next();
    };
    start_pipeline();

    // One sub-block.  OFF and lds_off: where its stage begins.  In the first pass the loop is unrolled over the two stages and the
    // stage is part of the read instructions (OFF), which saves an addition per operand address: 43 vector instructions where
    // there were 53, with the row sums below.  The careful loop, which rarely runs, adds it at run time (lds_off).
    // us, before and after both changes, 384-token tiles: 24 heads of 30x48x80, 3x3x3 10,834, 10,649, 1x3x3 3964, 3823; two heads
    // over the whole grid 10,250, 9784; 12 heads of 12x48x48, 1x3x3 474, 461; 128-token tiles, 24 heads of 8x64x64, 3x3x3 1129, 1088.
    const float c = p.scale_log2e;
    constexpr int kPlain = 0, kFirst = 1, kCareful = 2;
    using Stage0 = std::integral_constant<int, 0>;
    using Stage1 = std::integral_constant<int, STAGE_BYTES>;
    auto sub_block_at = [&](auto track_c, auto off_c, uint32_t lds_off, float grow_above) __attribute__((always_inline)) {
        // kFirst: set the offsets.  kCareful: follow the growth of the scores, which start at zero here: those of keys behind
        // masked ones (scores of the lowest numbers) are lost in accumulators that start at minus such an offset.
        constexpr int TRACK = decltype(track_c)::value, OFF = decltype(off_c)::value;
        const uint32_t kb_ = k_base + lds_off;
        uint32_t vb_[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) vb_[m] = v_addr[m] + lds_off;
        // ---- S^T = K Q^T: four 16x16 blocks (two key blocks x two query blocks), four k-steps of 32 channels each.
        // K-operand reads are issued by hand, one key block ahead of the MFMAs.
        floatx4 S[2][2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) S[kb][qb] = TRACK == kCareful ? floatx4{0.f, 0.f, 0.f, 0.f} : Sinit[qb];
        auto k_read = [&](auto kbc, auto ksc) {
            return ds_read_b128_at<OFF + decltype(kbc)::value * 4 * kKGroup + decltype(ksc)::value * 64>(kb_);
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        using I3 = std::integral_constant<int, 3>;
        // six reads in flight at most; the second key block's last two fragments reuse the registers of the first's
        bf16x8 a0 = k_read(I0{}, I0{}), a1 = k_read(I0{}, I1{}), a2 = k_read(I0{}, I2{}), a3 = k_read(I0{}, I3{});
        bf16x8 b0 = k_read(I1{}, I0{}), b1 = k_read(I1{}, I1{});
        // The query blocks are taken 0, 1, 1, 0, ..: from one matrix instruction to the next only one operand
        // changes (measured on N(0,1) operands: a percent more flops at the power limit than changing both).
        lds_wait2<4>(a0, a1);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) S[0][qb] = mfma_16x16x32(a0, Qr[qb][0], S[0][qb]);
#pragma unroll
        for (int qb = 1; qb >= 0; --qb) S[0][qb] = mfma_16x16x32(a1, Qr[qb][1], S[0][qb]);
        __builtin_amdgcn_sched_barrier(0);   // keep each MFMA group ahead of the next group's reads and wait
        bf16x8 b2 = k_read(I1{}, I2{}), b3 = k_read(I1{}, I3{});
        lds_wait2<4>(a2, a3);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) S[0][qb] = mfma_16x16x32(a2, Qr[qb][2], S[0][qb]);
#pragma unroll
        for (int qb = 1; qb >= 0; --qb) S[0][qb] = mfma_16x16x32(a3, Qr[qb][3], S[0][qb]);
        __builtin_amdgcn_sched_barrier(0);
        lds_wait2<2>(b0, b1);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) S[1][qb] = mfma_16x16x32(b0, Qr[qb][0], S[1][qb]);
#pragma unroll
        for (int qb = 1; qb >= 0; --qb) S[1][qb] = mfma_16x16x32(b1, Qr[qb][1], S[1][qb]);
        __builtin_amdgcn_sched_barrier(0);
        lds_wait2<0>(b2, b3);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) S[1][qb] = mfma_16x16x32(b2, Qr[qb][2], S[1][qb]);
#pragma unroll
        for (int qb = 1; qb >= 0; --qb) S[1][qb] = mfma_16x16x32(b3, Qr[qb][3], S[1][qb]);
        __builtin_amdgcn_sched_barrier(0);
        // ---- online softmax.  A lane holds, for each of its two queries, 8 of the 32 scores (keys 4*g4 + i of both
        // key blocks); the other 24 sit in the lanes 16, 32 and 48 further on.  In the careful loop the offset only moves
        // when a score exceeds it by more than 2^8 in the exponent (grow_above, in the units of the scores).
        if constexpr (TRACK != kPlain) {
            float mq[2];
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                mq[qb] = max3(S[0][qb][0], S[0][qb][1], S[0][qb][2]);
                mq[qb] = max3(mq[qb], S[0][qb][3], S[1][qb][0]);
                mq[qb] = max3(mq[qb], S[1][qb][1], S[1][qb][2]);
                mq[qb] = quad_lane_max(fmaxf(mq[qb], S[1][qb][3]));
            }
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                float offset;
                if constexpr (TRACK == kFirst) {
                    m_run[qb] = offset = mq[qb] == -INFINITY ? 0.f : mq[qb];
#pragma unroll
                    for (int r = 0; r < 4; ++r) Sinit[qb][r] = -offset;
                } else {
                    const bool grown = mq[qb] > m_run[qb] + grow_above;           // the same in the four lanes of a query
                    if (__builtin_amdgcn_ballot_w64(grown) != 0) {
                        const float alpha = grown ? __builtin_amdgcn_exp2f((m_run[qb] - mq[qb]) * c) : 1.f;
                        m_run[qb] = grown ? mq[qb] : m_run[qb];
                        l_acc[qb] *= alpha;
                        // in place: written as plain multiplications the register allocator gives the scaled accumulators
                        // new registers and then copies all 64 on the path that does NOT rescale
                        // (the compiler does not see into the assembly: the wait state that a vector instruction needs before
                        // it reads the result of a transcendental one is given by hand)
                        const float alpha_settled = settled_after_transcendental(alpha);
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) scale_in_place(Oacc[cb][qb], alpha_settled);
                    }
                    offset = m_run[qb] == -INFINITY ? 0.f : m_run[qb];
                }
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) S[kb][qb][r] -= offset;
            }
        }
        // first group of V-operand reads (channel blocks 0..3) goes out once the offsets are settled (no
        // earlier: their sixteen registers would be live across the rescaling branch); the exponentials hide its latency
        shortx4 va[2][4][2];
        static_for<0, 4>([&](auto i) {
            constexpr int cb = decltype(i)::value;
            va[0][cb][0] = ds_read_tr16<OFF + (cb & 1) * 32>(vb_[cb >> 1]);
            va[0][cb][1] = ds_read_tr16<OFF + (cb & 1) * 32 + 4 * kVGroup>(vb_[cb >> 1]);
        });
        __builtin_amdgcn_sched_barrier(0);       // the exponentials stay behind these reads
        // probabilities, rounded to bf16, packed as the B operand of the PV product of their query block: k index
        // 8*g4 + i of that product is key 4*g4 + i of the first key block (i < 4) or of the second (i >= 4)
        bf16x8 Pb[2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                    const float p0 = __builtin_amdgcn_exp2f(S[kb][qb][e] * c);
                    const float p1 = __builtin_amdgcn_exp2f(S[kb][qb][e + 1] * c);
                    bf16x2 pp;
                    pp[0] = static_cast<__bf16>(p0);
                    pp[1] = static_cast<__bf16>(p1);
                    Pb[qb][4 * kb + e] = pp[0];
                    Pb[qb][4 * kb + e + 1] = pp[1];
                }
        }
        bf16x8 ones;
#pragma unroll
        for (int e = 0; e < 8; ++e) ones[e] = static_cast<__bf16>(1.0f);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) l_acc[qb] = mfma_16x16x32(ones, Pb[qb], l_acc[qb]);       // sums the rounded values

        // ---- O^T += V^T P^T: one k-step covers the 32 keys; eight channel blocks x two query blocks.  The transposing
        // reads are issued by hand, four channel blocks ahead of the MFMAs that consume them.
        static_for<0, 2>([&](auto gi) {
            constexpr int g = decltype(gi)::value;
            if constexpr (g == 0) {
                static_for<0, 4>([&](auto i) {
                    constexpr int cb = 4 + decltype(i)::value;
                    va[1][cb - 4][0] = ds_read_tr16<OFF + (cb & 1) * 32>(vb_[cb >> 1]);
                    va[1][cb - 4][1] = ds_read_tr16<OFF + (cb & 1) * 32 + 4 * kVGroup>(vb_[cb >> 1]);
                });
                pv_wait<8>(va[0]);
            } else {
                pv_wait<0>(va[1]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                typedef short shortx8 __attribute__((ext_vector_type(8)));
                const shortx8 v01 = __builtin_shufflevector(va[g][i][0], va[g][i][1], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int qb = (i & 1) ^ t;      // 0, 1, 1, 0, ..: one operand changes at a time
                    Oacc[4 * g + i][qb] = mfma_16x16x32(__builtin_bit_cast(bf16x8, v01), Pb[qb], Oacc[4 * g + i][qb]);
                }
            }
            if constexpr (g == 0) __builtin_amdgcn_sched_barrier(0);   // the second group's wait stays behind these MFMAs
        });
    };

    const uint32_t bound_bits = __builtin_amdgcn_readfirstlane(__float_as_uint(8.0f / c));
    auto next_sub_block = [&]() __attribute__((always_inline)) {
        // this wave's DMA for this sub-block must have landed (the only requests outstanding)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();   // ... and everyone's; the stage read in the previous iteration is free again
        issue_next();      // refills the other stage
    };
    // The first sub-block of an item sets the offsets (row maxima of its 32 keys).  After that the common case needs
    // no offset to move: probabilities, row sums and accumulators are fp32 or bf16 numbers with 8 exponent bits,
    // whose relative precision does not depend on their size, so an offset that turns out too low costs nothing
    // until the sums near the end of that range.  The remaining sub-blocks therefore run WITHOUT following the
    // maximum (ten vector instructions and a branch less per sub-block), and the row sums are looked at once at the
    // end: if one of them is beyond 2^96 or not a number, or an accumulator has left the range, the workgroup does the
    // whole item again with the careful loop, which re-bases whenever a score exceeds the offset by more than 2^8 in
    // the exponent.  (Its scores start at zero and the offset is subtracted behind the product; with the offset in the
    // accumulators as well it cost 36 bytes of scratch: 24 heads of 30x48x80, window 1x1x1 755 -> 728 us.)  (2^96 leaves 66 in the exponent of e between the first keys' maximum and the largest score before
    // the second pass is needed, and room for |V| up to 2^32 in the accumulators.)
    next_sub_block();
    sub_block_at(std::integral_constant<int, kFirst>{}, Stage0{}, 0u, 0.f);
#pragma unroll 1
    for (int iter = 1; iter < n_iter; iter += 2) {
        next_sub_block();
        sub_block_at(std::integral_constant<int, kPlain>{}, Stage1{}, 0u, 0.f);
        if (iter + 1 < n_iter) {
            next_sub_block();
            sub_block_at(std::integral_constant<int, kPlain>{}, Stage0{}, 0u, 0.f);
        }
    }
    float l_tot[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) l_tot[qb] = l_acc[qb][0];
    // 2^96; and 2^-64, below which only rows are whose first keys all score minus infinity (their offset is 0 then)
    constexpr float kRedoAbove = 79228162514264337593543950336.f, kRedoBelow = 5.42101086242752217e-20f;
    // The accumulators too: with |V| beyond 2^32 they can leave the range before the row sums reach the bound.  The
    // test is on the bit patterns (largest exponent field), so that it sees a NaN (infinity minus infinity) as well.
    uint32_t o_max = 0;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int r = 0; r < 4; ++r) o_max = max(o_max, __float_as_uint(Oacc[cb][qb][r]) & 0x7fffffffu);
    // (With finite inputs a row sum is never a NaN: a probability that overflows is +infinity, and so is the sum.
    // The barrier inside also ends every wave's reads of the stages.)
    if (__builtin_expect(__syncthreads_or(!(l_tot[0] < kRedoAbove && l_tot[1] < kRedoAbove) || l_tot[0] < kRedoBelow ||
                                         l_tot[1] < kRedoBelow || o_max >= 0x7f800000u), 0)) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            m_run[qb] = -INFINITY;
            l_acc[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
            Sinit[qb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) Oacc[cb][qb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        start_pipeline();
#pragma unroll 1
        for (int iter = 0; iter < n_iter; ++iter) {
            next_sub_block();
            // growth threshold: 2^8 in the units of the scores
            sub_block_at(std::integral_constant<int, kCareful>{}, Stage0{}, (uint32_t)((iter & 1) * STAGE_BYTES), __uint_as_float(bound_bits));
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) l_tot[qb] = l_acc[qb][0];
    }

    // ---- finalize -------------------------------------------------------------------
    if (is_part) {
        // unnormalised accumulator, offset and row sum of this part; the combine kernel does the rest
        float *ws = p.split_ws + (size_t)(blockIdx.x - p.split_first) * split_part_floats<D>(QB);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            float *wo = ws + (size_t)(wave * 32 + 16 * qb + c16) * D;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) *reinterpret_cast<floatx4 *>(wo + 16 * cb + 4 * g4) = Oacc[cb][qb];
            if (g4 == 0) {
                ws[(size_t)QB * D + wave * 32 + 16 * qb + c16] = fmaxf(m_run[qb] * c, -3.0e38f);     // the merge takes base-2 units
                ws[(size_t)QB * D + QB + wave * 32 + 16 * qb + c16] = l_tot[qb];
            }
        }
        return;
    }
    bf16_raw *oh = o + (bh * p.N + (size_t)qblock * QB + (size_t)wave * 32) * D;
    // sum_j exp(s_j * scale) = 2^m * l  =>  ln = m * ln 2 + ln l
    if (p.lse != nullptr && g4 == 0) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
            p.lse[bh * p.N + (size_t)qblock * QB + (size_t)wave * 32 + 16 * qb + c16] =
                m_run[qb] * c * 0.6931471805599453f + __logf(l_tot[qb]);
    }
    // The rows go through LDS (each wave its own 32 rows; 16-byte chunk c of row r at position c ^ (r & 15)) and leave
    // as whole rows, 1 KB contiguous per store instruction, with streaming stores.
    __syncthreads();                                   // every wave has finished reading the K/V stages
    char *rows = smem + wave * (32 * ROWB);
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const float inv = 1.f / l_tot[qb];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            bf16x4 ov;
#pragma unroll
            for (int t = 0; t < 4; ++t) ov[t] = static_cast<__bf16>(Oacc[cb][qb][t] * inv);
            const int chunk = 2 * cb + (g4 >> 1);
            *reinterpret_cast<bf16x4 *>(rows + (16 * qb + c16) * ROWB + ((chunk ^ c16) << 4) + 8 * (g4 & 1)) = ov;
        }
    }
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int r = RPI * i + lane / LPR, cpos = lane % LPR;
        const u32x4 x = *reinterpret_cast<const u32x4 *>(rows + r * ROWB + ((cpos ^ (r & (LPR - 1))) << 4));
        __builtin_nontemporal_store(x, reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(oh) + (size_t)r * ROWB + (cpos << 4)));
    }
}

// Merges the parts of every split item.  With m the largest of the parts' offsets (base-2 units):
// O = sum_j 2^(m_j - m) O_j / sum_j 2^(m_j - m) l_j, parts in ascending order.  A wave takes eight query rows, half a wave a row,
// four channels a lane, with four rows' loads in flight.  (One row per wave before: 18,432 workgroups for 48 items of 384 queries in
// two parts, each of which finds its item first: 19 us, now 15, and 9 at best.)
template <int D, int QB>
__global__ __launch_bounds__(256) void sta_fwd_combine_kernel(bf16_raw *__restrict__ o, sta::FwdParams p, sta::FwdPlan plan)
{
    static_assert(D == 128, "four channels per lane");
    constexpr int ROWS = 4;                                    // per lane, two rows apart
    const uint32_t item_id = p.split_first + blockIdx.y;
    const GroupItem item = group_item_of(item_id, p, plan);
    const int lane = threadIdx.x & 63;
    const int row0 = blockIdx.x * 32 + (threadIdx.x >> 6) * 8 + (lane >> 5), channel = 4 * (lane & 31);
    const float *ws = p.split_ws + (size_t)blockIdx.y * p.split_parts * split_part_floats<D>(QB);
    float m[ROWS], l[ROWS];
    floatx4 acc[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        m[r] = -INFINITY;
        l[r] = 0.f;
        acc[r] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    for (uint32_t j = 0; j < p.split_parts; ++j)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) m[r] = fmaxf(m[r], ws[j * split_part_floats<D>(QB) + (size_t)QB * D + row0 + 2 * r]);
    for (uint32_t j = 0; j < p.split_parts; ++j) {
        const float *part = ws + j * split_part_floats<D>(QB);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int row = row0 + 2 * r;
            const floatx4 x = *reinterpret_cast<const floatx4 *>(part + (size_t)row * D + channel);
            const float w = exp2f(part[(size_t)QB * D + row] - m[r]);
            l[r] += w * part[(size_t)QB * D + QB + row];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[r][c] += w * x[c];
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const float inv = 1.f / l[r];
        const size_t out_row = item.bh * p.N + (size_t)item.qblock * QB + row0 + 2 * r;
        bf16x4 ov;
#pragma unroll
        for (int c = 0; c < 4; ++c) ov[c] = static_cast<__bf16>(acc[r][c] * inv);
        __builtin_nontemporal_store(ov, reinterpret_cast<bf16x4 *>(o + out_row * D + channel));
        if (p.lse != nullptr && (lane & 31) == 0) p.lse[out_row] = m[r] * 0.6931471805599453f + __logf(l[r]);
    }
}

// Host side of the work splitting: how many workgroups the chip holds at once.
inline uint32_t resident_workgroups(int minb) { return sta::compute_units() * (uint32_t)minb; }

// What a launch function is called with.
struct FwdArgs {
    const void *q, *k, *v;
    void *o;
    int B;
    const sta::FwdParams &p;
    const sta::WindowTable &win;
    const sta::HeadOrder &order;
    float *split_ws;
    size_t split_ws_floats;
    hipStream_t stream;
    sta::LaunchNote *note;      // not null: the shape is written there and nothing is launched
};

// The plan of a launch of blocks of that many queries.
sta::FwdPlan make_plan(uint32_t queries, const FwdArgs &a)
{
    const sta::FwdParams &p = a.p;
    sta::FwdPlan plan;
    const uint32_t per_head = p.N / queries;
    plan.deal = sta::deal_of(per_head, (uint32_t)a.B * p.heads);
    plan.per_head = sta::fast_div_of(per_head);
    plan.per_tile = sta::fast_div_of(p.P / queries);
    plan.pair_items = sta::fast_div_of(2 * p.n_w * p.n_t);
    plan.n_t = sta::fast_div_of(p.n_t);
    plan.batch = sta::fast_div_of((uint32_t)a.B);
    plan.sub_per_tile = sta::fast_div_of(p.P / kSub);
    for (uint32_t h = 0; h < p.heads; ++h) {
        plan.head[h].h = a.order.h[h];
        for (int i = 0; i < 3; ++i) plan.head[h].w[i] = a.win.w[a.order.h[h]][i];
    }
    return plan;
}

// Units (32 keys) of the walk of a head of the launch; heads by rank, the one with the most key tiles first.
uint32_t walk_of_rank(const FwdArgs &a, uint32_t rank)
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
uint32_t longest_walk(const FwdArgs &a) { return walk_of_rank(a, 0); }

// Heads whose walk is more than so many quarters of the longest.
uint32_t heads_of_long_walks(const FwdArgs &a, uint32_t quarters)
{
    uint32_t n = 1;
    while (n < a.p.heads && 4 * (uint64_t)walk_of_rank(a, n) > (uint64_t)quarters * longest_walk(a)) ++n;
    return n;
}

// Where the walks of the heads differ and the longest is more than 1.4 times an even share of all of the launch's items on so many places
// (the cases at its uses are at 1.45, 1.5 and 3.0): the long ones are what the launch waits for, and its last items, the short ones, are not.
// They differ where the mean is less than nine tenths of the longest.  us, 384-token tiles, twelve waves a workgroup and four, by mean over
// longest: 0.73 (18x40x40, 324, 324 and 540 units, 0.88 rounds) 585, 449, 0.80 123, 113, 0.88 261, 244; 0.90 99, 107 and 355, 369, 0.93 217,
// 225, 0.94 134, 141 and, cut into parts, 164, 160.  (756 launches of up to one round: 0.86 of the time on
// average, 24 from 0.9 on 1.01.)
bool waits_for_long_walks(const FwdArgs &a, uint64_t items, uint64_t places)
{
    const uint64_t longest = longest_walk(a);
    uint64_t all = 0;
    for (uint32_t r = 0; r < a.p.heads; ++r) all += walk_of_rank(a, r);
    return 10 * all < 9 * a.p.heads * longest && 5 * longest * places * a.p.heads > 7 * all * items;
}

// Items of qb queries beyond the last full round of workgroups are cut into parts that fill the chip once: how many parts
// each of them gets, 1 where they are left whole (no workspace, more than half a round, walks too short).  They are the last ids,
// all of which name an item, so that the parts never need more than one resident set of the workspace.  (While ids without an
// item stood among them and took slots, launches with few items in a round of chunks were left whole: whole layers, us, whole and
// in parts, nine heads of 12x24x40 in 384-token tiles, 1x3x3 279, 219, 1x3x5 428, 301; 13 of 6x48x80, 1x3x3 604, 546; 19 of
// 18x24x24, 3x3x3 1124, 938.)
uint32_t parts_of_tail(const FwdArgs &a, uint32_t items, uint32_t capacity, int qb)
{
    const sta::FwdParams &p = a.p;
    const uint32_t tail = items % capacity;
    if (a.split_ws == nullptr || tail == 0 || 2 * tail > capacity) return 1;
    // (12x32x32 in 384-token tiles, twelve heads of 108, 384 and 36 units, 394 us in parts, 367 whole)
    if (items > capacity && waits_for_long_walks(a, items, capacity)) return 1;
    uint32_t parts = capacity / tail;
    // a part should keep at least four sub-blocks of the cheapest item of the launch
    uint32_t min_tiles = 0xffffffffu;
    for (uint32_t h = 0; h < p.heads; ++h) {
        uint32_t tiles = 1;
        const uint32_t n[3] = {p.n_t, p.n_h, p.n_w};
        for (int i = 0; i < 3; ++i) {
            const uint32_t kept = 2 * (a.win.w[h][i] / 2) + 1;
            tiles *= kept < n[i] ? kept : n[i];
        }
        min_tiles = tiles < min_tiles ? tiles : min_tiles;
    }
    const uint32_t min_iters = min_tiles * (p.P / kSub);
    while (parts > 1 && min_iters / parts < 4) --parts;
    return (size_t)tail * parts * split_part_floats<128>(qb) <= a.split_ws_floats ? parts : 1;
}

template <int NW, int KB, int STAGES, int MINB>
hipError_t launch_x32(const FwdArgs &a)
{
    constexpr int D = 128, QB = NW * 32;
    sta::FwdParams p = a.p;
    const sta::FwdPlan plan = make_plan(QB, a);
    const uint32_t items = plan.deal.total, capacity = resident_workgroups(MINB);
    p.split_parts = parts_of_tail(a, items, capacity, QB);
    const uint32_t split_items = p.split_parts > 1 ? items % capacity : 0;
    p.split_first = items - split_items;
    p.split_ws = split_items ? a.split_ws : nullptr;
    dim3 grid(p.split_first + split_items * p.split_parts), block(NW * 64);
    if (a.note) return a.note->add("x32<%d> items %u workgroups %u parts %u of %u", NW, items, grid.x, p.split_parts, split_items);
    const hipError_t e = sta::launch_kernel(
        sta_fwd_x32_kernel<NW, KB, STAGES, MINB>, grid, block, a.stream,
        static_cast<const bf16_raw *>(a.q), static_cast<const bf16_raw *>(a.k), static_cast<const bf16_raw *>(a.v),
        static_cast<bf16_raw *>(a.o), p, plan);
    if (e != hipSuccess || split_items == 0) return e;
    return sta::launch_kernel(sta_fwd_combine_kernel<D, QB>, dim3(QB / 32, split_items), dim3(256), a.stream, static_cast<bf16_raw *>(a.o), p, plan);
}

template <int D, int QW, int KG, int WPE, bool FOLLOW, int UPS = 1, bool ONEV = false>
hipError_t launch_group(const FwdArgs &a)
{
    const sta::FwdPlan plan = make_plan(32 * QW, a);
    if (a.note) return a.note->add("%s<%d,%d,%d,%d,%d> items %u", ONEV ? "group_one_v" : "group", D, QW, KG, (int)FOLLOW, UPS, plan.deal.total);
    return sta::launch_kernel(
        sta_fwd_group_kernel<D, QW, KG, WPE, FOLLOW, UPS, ONEV>, dim3(plan.deal.total), dim3(QW * KG * 64), a.stream,
        static_cast<const bf16_raw *>(a.q), static_cast<const bf16_raw *>(a.k), static_cast<const bf16_raw *>(a.v),
        static_cast<bf16_raw *>(a.o), a.p, plan);
}

template <int D, int NQ, int KG, bool FOLLOW>
hipError_t launch_solo(const FwdArgs &a)
{
    const sta::FwdPlan plan = make_plan(16 * NQ, a);
    if (a.note) return a.note->add("solo<%d,%d,%d,%d> items %u", D, NQ, KG, (int)FOLLOW, plan.deal.total);
    return sta::launch_kernel(
        sta_fwd_solo_kernel<D, NQ, KG, D == 64 && NQ < 4 ? 6 - NQ : 2, FOLLOW>, dim3(plan.deal.total), dim3(KG * 64), a.stream,
        static_cast<const bf16_raw *>(a.q), static_cast<const bf16_raw *>(a.k), static_cast<const bf16_raw *>(a.v),
        static_cast<bf16_raw *>(a.o), a.p, plan);
}

// Shape of the kernel for a launch.
// Small launches, solo: in waves of 32 queries (counted as for the key groups below) and units of the longest walk; us, key-group
// kernel against KG = 8, 4, and where they exist 64 queries per wave with KG = 8, 4.
// Head dimension 64, tiles of 64 tokens' multiples: 128 waves, 18 units 8.4, 8.0, 7.7, 9.5, 9.1; 128, 50 14.5, 9.3, 10.7, 13.0, 15.3;
// 216, 108 24.2, 14.4, 17.9, 19.2, 25.7; 432, 108 24.4, 23.6, 22.3, 20.0, 25.6; 450, 54 15.1, 15.2, 13.9, 13.4, 15.9; 512, 36 11.6, 12.4,
// 11.4, 11.7, 12.2; 648, 108 34.8, 34.0, 31.7, 37.9, 31.0; 768, 36 16.9, 17.4, 15.6, 21.5, 15.6; 1024, 18 10.8, 16.2, 13.2, 18.0, 12.2;
// 1024, 50 22.4, 27.0, 24.4, 26.5, 21.1; 1296, 108 50, 64, 59, 62, 56.  96-token tiles: 144, 36 16.8, 9.6, 10.8; 525, 27 16.8, 16.4,
// 14.0; 1575, 81 84, 68, 62; 2100, 81 82, 88, 79; 3150, 81 109, 126, 114.  32-token tiles: 256, 25 13.2, 8.7, 9.6; 768, 25 16.9, 16.7,
// 14.6; 768, 9 9.5, 12.2, 9.6; 1024, 25 18.3, 20.8, 17.9.
// Head dimension 128: 384-token tiles 216, 108 35.0, 23.1, 25.0; 432, 108 37, 45, 40; 128-token tiles 256, 36 16.6, 12.8, 12.2; 512, 36
// 18, 25, 20; 64-token tiles 128, 50 24.3, 16.0, 18.5; 384, 50 24.9, 29.3, 23.2; 512, 18 14.0, 20.1, 13.8; 640, 50 38, 44, 39; 192-token
// tiles 900, 54 72, 62, 49; 1350, 54 62, 91, 73; 96-token tiles 36, 36 23.6, 13.1, 14.4; 432, 36 24.8, 26.9, 21.4; 525, 27 22.8, 32, 25;
// 32-token tiles 256, 25 25.9, 12.8, 13.1; 512, 25 26.7, 23.3, 17.3; 768, 25 27, 34, 27.
// Key-group kernel.  Waves of queries: as many as the tile allows up to four (three for 96-token multiples), because a K/V unit
// brought into LDS serves them all; five waves leave the four SIMDs uneven (tiles of 320 tokens: 585 us with five waves, 431 with
// two).  Tiles of 192 tokens at head dimension 64 take three, but two where the fullest CU gets fewer waves that way (with key groups:
// no more; us, three and two waves, waves of the fullest CU in brackets: 9x40x40, window 3x3x3, two heads 79 (6), 54 (4); four 118 (9),
// 92 (8); twelve, one group 263 (24), 257 (22); six, one group 133 (12), 157 (12); 6x24x40, 1x3x3, four heads 18.9 (3), 21.8 (4)).
// Two units per stage where four waves of queries share it and there are no key groups: one barrier for 64 keys (12x48x48 in
// 384-token tiles, us, one and two units: three heads 85, 83; six 162, 157; twelve 289, 283).  With two waves or with groups the
// larger stages or the registers cost a wave per SIMD (twelve heads, two groups 305, 362).
// Key groups: the most, of 1, 2 and (384-token tiles and the like at head dimension 128) 4, with which the launch still fits the chip
// at once (16 waves per CU at head dimension 64, 8 at 128) and a group has at least eight units to walk.  Where the longest walk is 64
// units or more, heads count by their walks, because it is the long ones that leave the chip idle (six heads of a 128x112 image, two
// of them over all of it, 242 us counted by heads, 153 by walks; 9x40x40, 1x3x3, 3x5x5 and 1x1x3, six heads 245, 156; but 27 of a 32x48
// image, 8 to 48 units, 17.9, 20.8).  Measured around the line (us; 1, 2, 4 groups), head dimension 64, 384-token tiles, 108 units: 972
// waves 62, 40, 38; 1944 waves 69, 66, 71; 2592 waves 89, 94, 101.  64-token tiles, 18 units: 1024 waves 15.1, 12.6, 14.1; 2048 waves
// 17.3, 17.4, 22.9; 4096 waves 27.5, 30.1, 42.4.  Head dimension 128, 96-token tiles, about 75 units: 525 waves 50, 39, 34; 1050 waves
// 68, 78, 69.
template <int D>
hipError_t launch_groups(const FwdArgs &a)
{
    constexpr uint32_t kFixed = D == 64 ? 64 : 128;         // tiles of its multiples keep the offset of the first unit
    const sta::FwdParams &p = a.p;
    const uint32_t units = longest_walk(a), P = p.P;
    uint64_t heads = p.heads;
    if (units >= 64) {
        uint64_t all_units = 0;
        for (uint32_t r = 0; r < p.heads; ++r) all_units += walk_of_rank(a, r);
        heads = (all_units + units - 1) / units;
    }
    const uint64_t cus = resident_workgroups(1), waves = (uint64_t)a.B * heads * (p.N / 32);

    if (waves <= cus) {
        const bool eight = units >= (D == 64 ? (P % 64 == 0 ? 24 : 16) : P % 64 == 0 ? (P % 128 == 0 ? 48 : 32) : 16);
        if (P % kFixed == 0)
            return eight ? launch_solo<D, 2, 8, false>(a)
                         : launch_solo<D, 2, 4, false>(a);
        return eight ? launch_solo<D, 2, 8, true>(a)
                     : launch_solo<D, 2, 4, true>(a);
    }
    if constexpr (D == 64) {
        // 48 queries for twelve waves where that gives no CU two workgroups (of the workgroups there are, whatever their walks: the LDS holds
        // one at a time) and 64 would leave a third of the chip without one.  us, 64 queries for eight waves against these, waves and units
        // in brackets: (324, 108) 19.6, 17.5; (360, 108) 19.0, 16.6; (324, 324) 40.5, 36.2; (360, 360) 43.5, 40.5; 192-token tiles (300, 54)
        // 13.1, 12.2; not measured below that.  Heads of different walks, more waves than 384 that count fewer: (594, 66 and 18) 16.9, 20.0;
        // (768, 120, 24 and 6) 19.5, 22.1; (576, 192 to 36) 28.4, 30.6.  (Sixteen waves for 32 queries up to 256 waves: 1.0 to 1.5 us slower
        // than eight, at 36 to 128 units.)
        const uint64_t all_waves = (uint64_t)a.B * p.heads * (p.N / 32);
        if (P % 192 == 0 && 8 * waves > 9 * cus && 2 * all_waves <= 3 * cus && units >= 48) return launch_solo<64, 3, 12, false>(a);
        if (P % 64 == 0 && waves <= 2 * cus)
            return units >= 48 ? launch_solo<64, 4, 8, false>(a)
                               : launch_solo<64, 2, 4, false>(a);
        if (P % 64 == 0 && waves <= 4 * cus && units >= 32) return launch_solo<64, 4, 4, false>(a);
        if (P % 64 != 0 && waves <= (P % 96 == 0 ? 8 : units >= 16 ? 3 : 2) * cus)
            return launch_solo<64, 2, 4, true>(a);
    } else if (P % 128 != 0 && waves <= (P % 192 == 0 ? 4 : 2) * cus) {
        return launch_solo<128, 2, 4, true>(a);
    }

    const uint64_t fits = cus * (D == 64 ? 16 : 8);
    const bool two = 2 * waves <= fits && units >= 16;
    auto fullest_cu = [&](uint64_t qw) { return (waves / qw + cus - 1) / cus * qw; };          // waves of queries
    const bool two_for_192 = D == 64 && P % 64 == 0 && (two ? fullest_cu(2) <= fullest_cu(3) : 20 * fullest_cu(2) < 19 * fullest_cu(3));
    if (P % 96 == 0 && P % 128 != 0 && !two_for_192) {
        if constexpr (D == 64) {
            if (P % 64 != 0) return launch_group<64, 3, 1, 3, true>(a);
            return two ? launch_group<64, 3, 2, 3, false>(a)
                       : launch_group<64, 3, 1, 3, false>(a);
        } else {
            return two ? launch_group<128, 3, 2, 3, true>(a)
                       : launch_group<128, 3, 1, 3, true>(a);
        }
    }
    // One LDS stage of V instead of two (head dimension 128): whether n workgroups of qw waves of queries, of which a CU then holds six
    // instead of four, are through in fewer rounds.  Heads of different walks: not where those over half the longest, which run first, are
    // less than a round of four and the longest is 0.9 of a place's even share or more, as a wave that is alone at the end is slower with one
    // stage, nor where those ones end beyond a round of six and within two of four, unless the longest is less than 0.45 shares.  (us, two
    // stages, one; waves, units and heads: 64-token tiles (4320; 60 x 10, 20, 12 and 6 x 30) 78, 102, (3200; 400 x 4, 50 x 4) 417, 520; 32-token
    // tiles (2464; 55 x 8, 9 and 3 x 24) 53, 67, (3840; 96 x 20, 3 x 20) 169, 211; 383 launches that this leaves on two stages: one 2 % slower
    // in the mean, 27 % at most; 1717 on one: 12 % faster.)
    const uint64_t long_waves = (uint64_t)a.B * heads_of_long_walks(a, 2) * (p.N / 32);
    auto one_stage = [&](uint64_t n, uint64_t qw) {
        const uint64_t places = 4 * cus, long_ones = long_waves / qw, longest = units * places;
        auto beyond_six = [&](uint64_t m) { return 2 * m > 3 * places && m <= 2 * places; };
        uint64_t all = 0;                                   // units of all workgroups
        for (uint32_t r = 0; r < p.heads; ++r) all += walk_of_rank(a, r);
        all *= (uint64_t)a.B * (p.N / 32) / qw;
        return n > places && !beyond_six(n) && (long_ones > places || 10 * longest < 9 * all) && !(beyond_six(long_ones) && 20 * longest >= 9 * all);
    };
    if (P % 64 == 0) {
        if constexpr (D == 128) {
            // Two stages of V, four of these workgroups a CU, or one stage, six (three with two groups).  One stage costs a second barrier
            // a unit and waits for V; it pays by its places: more than a round of four, and two groups for up to three workgroups a CU (measured
            // from 576 workgroups of one group on: 25.7, two 23.7).
            // Not from the first round of six to the second of four ((1540, 308 units) 606, 641; (1600, 150) 313, 333; 36 launches up to 1620 4 % on
            // average; (1664) 51, 52; (1750) 372, 394; (1920) 54, 58), and where the walks of the
            // heads differ, two groups of two stages for one to one and a half rounds, as the long walks are alone at the end (96x96, 18 heads
            // of 18, 50 and 288 units 365, one stage 401; nine (by walks 576) 256, in two groups of one stage 194).  us, two stages, one, one and two groups; workgroups
            // of one group in brackets: 64x64, 3x3 (640) 25.9, 26.0, 23.9; (768) 26.4, 26.3, 25.4; (1024) 29.6, 29.6, 33.1; (1280) 42.4, 37.6,
            // 38.7; (1536) 50, 41, 44; (2048) 62, 59, 57; (3072) 86, 80, 87; 128x128, 5x5 (768) 57, 59, 53; (1280) 97, 85, 85; (1536) 113, 92, 98;
            // (2048) 131, 138, 132; (2560) 169, 159, 161; (4096) 249, 242, 257; 10x40x40 in 320-token tiles (750) 168, 177, 156; (1500) 314, 288,
            // 302; (2000) 388, 437, 400; (2500) 529, 488, 498; (4000) 765, 745, 779; 10x24x48 in them, 2x2x4, eight
            // heads (1440, 300 units), two groups of two stages 547, one of one stage 475.
            const uint64_t blocks = waves / 2, places = 4 * cus;
            if (P % 128 != 0) {
                if (two) return launch_group<128, 2, 2, 2, true>(a);
                if (4 * blocks >= 9 * cus && blocks <= 3 * cus && long_waves <= 6 * cus && units >= 16) return launch_group<128, 2, 2, 3, true, 1, true>(a);
                if (units >= 64 && units != walk_of_rank(a, p.heads - 1) && blocks > places && 2 * blocks <= 3 * places)
                    return launch_group<128, 2, 2, 2, true>(a);
                return one_stage(blocks, 2) ? launch_group<128, 2, 1, 3, true, 1, true>(a)
                                            : launch_group<128, 2, 1, 2, true>(a);
            }
            if (4 * waves <= fits && units >= 32) return launch_group<128, 2, 4, 2, false>(a);
            return two ? launch_group<128, 2, 2, 2, false>(a)
                       : launch_group<128, 2, 1, 2, false>(a);
        } else {
            if (two) return launch_group<64, 2, 2, 4, false>(a);
            return P % 128 == 0 ? launch_group<64, 4, 1, 4, false, 2>(a)
                                : launch_group<64, 2, 1, 4, false>(a);
        }
    }
    // other multiples of 32 tokens: one wave of queries, whose LDS stages then limit a CU to four such workgroups at head
    // dimension 128, with or without key groups (525 waves: 59 us, two groups 74)
    if (D == 64 && two) return launch_group<64, 1, 2, 2, true>(a);
    if constexpr (D == 128) {
        // one stage of V here too: six waves a CU instead of four (us, two stages, one; waves, units: 32-token tiles (1536, 9) 25.7, 19.4;
        // (2304, 9) 36.2, 30.6; (3072, 9) 39.1, 35.2; (4608, 9) 61.8, 50.0; (3072, 25) 79, 73; (7680, 25) 203, 176; 160-token tiles (1080, 45)
        // 79.6, 56.9; (1440, 45) 80.4, 59.7)
        if (one_stage(waves, 1)) return launch_group<128, 1, 1, 2, true, 1, true>(a);
    }
    return launch_group<D, 1, 1, D == 64 ? 3 : 1, true>(a);
}

// Test hook: the key-tile list of every (head, query tile) from the same box function.
__global__ void sta_dump_key_tiles_kernel(sta::FwdParams p, sta::WindowTable win, int32_t *counts, int32_t *lists)
{
    const uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= p.heads * p.n_tiles) return;
    const uint32_t h_local = idx / p.n_tiles;
    const uint32_t q_tile = idx % p.n_tiles;
    const StaBox box = sta_key_tile_box_of(p.n_t, p.n_h, p.n_w, win.w[h_local][0], win.w[h_local][1],
                                           win.w[h_local][2], q_tile);
    const size_t row = (size_t)(p.head_base + h_local) * p.n_tiles + q_tile;
    int32_t *out = lists + row * p.n_tiles;
    uint32_t c = 0;
    for (int a = box.t.lo; a <= box.t.hi; ++a)
        for (int bq = box.h.lo; bq <= box.h.hi; ++bq)
            for (int cq = box.w.lo; cq <= box.w.hi; ++cq) out[c++] = (a * (int)p.n_h + bq) * (int)p.n_w + cq;
    counts[row] = (int32_t)c;
    for (; c < p.n_tiles; ++c) out[c] = -1;
}

template <int D, int NW, int NQ, int KB, bool TW = false>
hipError_t launch_cfg(const FwdArgs &a)
{
    using C = FwdCfg<D, NW, NQ, KB>;
    dim3 grid(a.p.N / C::kQB, (uint32_t)a.B * a.p.heads);
    dim3 block(C::kThreads);
    if (a.note) return a.note->add("general<%d,%d,%d>", D, NW, KB);
    return sta::launch_kernel(
        sta_fwd_kernel<D, NW, NQ, KB, TW>, grid, block, a.stream,
        static_cast<const bf16_raw *>(a.q), static_cast<const bf16_raw *>(a.k), static_cast<const bf16_raw *>(a.v),
        static_cast<bf16_raw *>(a.o), a.p, a.win);
}

template <int D, bool TW = false>
hipError_t launch_d(const FwdArgs &a)
{
    const uint32_t P = a.p.P;
    if (P % 128 == 0) return launch_cfg<D, 4, 1, 64, TW>(a);
    if (P % 64 == 0) return launch_cfg<D, 2, 1, 64, TW>(a);
    if (P % 32 == 0) return launch_cfg<D, 1, 1, 32, TW>(a);
    return hipErrorInvalidValue;
}

}  // namespace

namespace sta {

uint32_t compute_units()
{
    static const int cus = []() {
        int dev = 0, n = 0;
        return hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0
                   ? n
                   : 256;
    }();
    return (uint32_t)cus;
}

bool forward_supported(int P, int D) { return (D == 64 || D == 128) && P > 0 && P % 32 == 0; }

size_t forward_split_workspace_bytes(int P, int D)
{
    if (D != 128 || P % 128 != 0) return 0;
    // At most one resident set of workgroups leaves partial results, QB queries x (128 + 2) floats each.  (Twice that, as it has
    // always been: a caller's workspace has to have this size.)
    if (P % 384 == 0) return (size_t)2 * resident_workgroups(1) * 384 * 130 * sizeof(float);
    return (size_t)2 * resident_workgroups(3) * 128 * 130 * sizeof(float);
}

hipError_t launch_forward(const void *q, const void *k, const void *v, void *o, int B, int D, const FwdParams &p,
                          const WindowTable &win, const HeadOrder &order, float *split_ws, size_t split_ws_floats,
                          hipStream_t stream, LaunchNote *note)
{
    if (!forward_supported((int)p.P, D)) return hipErrorInvalidValue;
    const FwdArgs a = {q, k, v, o, B, p, win, order, split_ws, split_ws_floats, stream, note};
    // K or V at an odd address: tiles that have not always been staged by DMA keep to plain loads, which take any address.
    if (p.P % (D == 64 ? 64 : 128) != 0 && !(dma_aligned(k) && dma_aligned(v)))
        return D == 64 ? launch_d<64>(a) : launch_d<128>(a);
    if (D == 64) return launch_groups<64>(a);
    if (p.P % 128 != 0) return launch_groups<128>(a);
    // Tiles of 128 tokens' multiples.  Up to 1280 waves of 32 queries (the chip holds 2048 of the key-group kernel's at this
    // head dimension) the key-group kernel: more and smaller workgroups, and key groups that need no workspace.  Where one is
    // given, items cut into parts are ahead on long walks: then up to 256 waves, up to 512 (four groups) at up to 240 units, up to 1024
    // (two) at up to 128, and any number here at up to 80; from 256 to 320 waves at up to 192 units, from 512 to 614 at up to 112, as fewer
    // items are cut into more parts.  us, parts and key groups; waves, units: 384-token tiles (324, 108) 44.4, 34.4;
    // (432, 108) 47.1, 35.4; (360, 180) 57.0, 51.9; (384, 192) 59.4, 55.2; (432, 216) 65.6, 62.7; (384, 384) 89, 103; (648, 108) 53.8, 52.6;
    // (864, 108) 63.2, 58.7; (576, 192) 72, 85; (960, 192) 101, 105; (1080, 108) 76, 81; 256-token tiles (384, 128) 50.3, 39.6; (400, 200)
    // 63.1, 57.9; (768, 128) 67, 65; (1024, 128) 82, 75; (648, 216) 91, 98; 128-token tiles (480, 108) 48.7, 36.4; (480, 180) 64.5, 55.9; (480,
    // 480) 132, 137; (960, 108) 70.2, 62.4; (720, 144) 71, 72; (576, 200) 77, 91; any of them (288, 144) 49, 43; (288, 216) 56, 60; (300, 180) 53,
    // 51; (528, 120) 51, 54; (576, 120) 54, 56; (576, 108) 49.9, 49.6; (640, 120) 60, 57.
    // Beyond 128 units only where the mean walk is two thirds of the longest or more: the parts of the long ones are shorter than a quarter,
    // and share a CU with fewer ((432, 216 and 24) 55, 60; (400, 200 and 40) 51, 56; (480, 160, 80 and 48) 44, 46; (480, 240 and 200) 72, 69).
    // Measured in us, 12-wave or 4-wave kernel without a workspace, with one, key groups; waves, units:
    // 6x16x24 in 384-token tiles, one head (72, 72) 79, 37, 26; 12x48x48, one head (864, 108) 116, 68, 57; 2x40x40 in 128-token
    // tiles, one head (100, 36) 27, 26, 17, twelve (1200, 36) 37, 54, 34; 16x8x40 in 128-token tiles, four heads (640, 120) 76,
    // 64, 58, eight (1280, 120) 102, 104, 99; 12x32x40 in 256-token tiles, four heads (1920, 216) 255, 255, 280.
    const uint64_t cus = compute_units(), slices = (uint64_t)B * p.heads, waves = slices * (p.N / 32);
    const uint32_t units = longest_walk(a);
    uint64_t all_units = 0;                                 // units of a walk of every head
    for (uint32_t r = 0; r < p.heads; ++r) all_units += walk_of_rank(a, r);
    const bool alike = 3 * all_units >= 2 * (uint64_t)p.heads * units;
    const bool short_walks = waves <= 4 * cus && units <= (waves <= 2 * cus || 5 * waves > 12 * cus ? 128 : 112);
    const bool long_walks = waves <= 2 * cus && units <= (4 * waves > 5 * cus ? 240 : 192) && alike;
    if (waves <= 5 * cus && (split_ws == nullptr || units <= 80 || waves <= cus || short_walks || long_walks))
        return launch_groups<128>(a);
    // A tile of 384 tokens (the paper's 6x8x8) gets one 12-wave workgroup per query tile: every K/V sub-block
    // fetched from L2 then serves 384 queries instead of 128.  Measured at the 115,200-token layer, window
    // 3x3x3: 12.8-13.1 ms against 13.6-13.7 ms for the 4-wave shape in the same session.  Not where the last round of such
    // workgroups would be mostly empty and is not cut into parts: where the rounds are filled by less than four fifths, the only round
    // by less than seven tenths (12x48x48, window
    // 1x3x3, us, 12 waves against 4, rounds in brackets: two heads (0.56) 117, 97; three (0.84) 126, 141; four (1.13) 244, 194 and with
    // parts 180, 184; six (1.69) 237, 262; eight (2.25) 355, 315; eleven (3.09) 477, 436; twelve (3.38) 486, 487; thirteen (3.66) 500, 498;
    // 6x48x48, eleven (1.55) 233, 223; twelve (1.69) 235, 258; 18x48x48, 3x3x3, five (2.11) 1009, 885; six (2.53) 1013, 1011.  From 0.70 to
    // 0.78 of a round, 94 launches of 24 to 432 units a walk: 12 waves ahead by 7 %, 15 at most; 119, 130 at 0.70 and 108 units).
    // Nor where the launch waits for long walks, which the smaller workgroups spread over three times as many CUs (12x48x48, heads of 36,
    // 108, 12 and 864 units, four 803, 482; eight 830, 775).
    // Nor is the second round too empty where the long walks, one to a CU, outlast all others beside them (heads of two lengths, us, 12 waves
    // against 4, rounds of all and of the long ones in brackets: 396 and 36 units (1.41, 0.70) 424, 480; 180, 36 (1.41, 0.70) 209, 225; 240, 36
    // (1.56, 0.78) 298, 313; 336, 72 (1.5, 0.75) 386, 416; 264, 72 (1.5, 0.75) 314, 341; but 36,
    // 12 (1.15, 0.82) 68, 53 and 324, 60, 36 (2.25, 0.70) 470, 433): where the longest is 1.04 times an even share of all or more, and the two
    // rounds are seven tenths full, what counts is the round of those over three quarters of it.
    const uint64_t items = slices * (p.N / 384), rounds = (items + cus - 1) / cus;
    auto full = [&](uint64_t n) { return 10 * n >= (n <= cus ? 7 : 8 * ((n + cus - 1) / cus)) * cus; };
    auto full_of_long_walks = [&]() {
        const uint64_t n = items / p.heads * heads_of_long_walks(a, 3);
        return rounds == 2 && 10 * items >= 14 * cus && 25 * (uint64_t)units * cus * p.heads >= 26 * all_units * items && n <= cus && full(n);
    };
    if (p.P % 384 == 0 && !waits_for_long_walks(a, items, cus) &&
        (parts_of_tail(a, (uint32_t)items, (uint32_t)cus, 384) > 1 || full(items) || full_of_long_walks()))
        return launch_x32<12, 32, 2, 1>(a);
    return launch_x32<4, 32, 2, 3>(a);
}

hipError_t launch_forward_general(const void *q, const void *k, const void *v, void *o, int B, int D, const FwdParams &p,
                                  const WindowTable &win, bool token_window, hipStream_t stream)
{
    if (!forward_supported((int)p.P, D)) return hipErrorInvalidValue;
    const HeadOrder order = {};                             // the general kernel takes the heads as they come
    const FwdArgs a = {q, k, v, o, B, p, win, order, nullptr, 0, stream, nullptr};
    if (token_window) {
        if (p.P > kMaxTokenWindowTile || p.T_t > 1023 || p.T_h > 1023 || p.T_w > 1023) return hipErrorInvalidValue;
        return D == 64 ? launch_d<64, true>(a) : launch_d<128, true>(a);
    }
    return D == 64 ? launch_d<64>(a) : launch_d<128>(a);
}

hipError_t launch_dump_key_tiles(const FwdParams &p, const WindowTable &win, int32_t *counts, int32_t *lists,
                                 hipStream_t stream)
{
    const uint32_t total = p.heads * p.n_tiles;
    return launch_kernel(sta_dump_key_tiles_kernel, dim3((total + 255) / 256), dim3(256), stream, p, win, counts, lists);
}

}  // namespace sta

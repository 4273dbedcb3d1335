// fp32 path on the fp32 matrix instruction, for the steps that hexi_f32x3_fwd() and hexi_f32x3_bwd() (hexi_shapes.h) leave to it, and for rows
// whose values leave the range of the kernels of hexi_f32_bf16x3.hip: the contractions run on
// v_mfma_f32_16x16x4_f32, whose products and sums are ordinary fp32 fused multiply-adds at twice the rate of the
// vector unit's.  Forward, dQ (both q-stationary) and dK/dV (key-stationary, one kernel with dQ; P is recomputed from the
// saved global LSE in both).  No sum is spread over workgroups here, so every output of these kernels has a fixed summation order.
//
// Shape of a workgroup.  A wavefront owns 16 stationary rows (q rows, or keys in the dK/dV kernel): their operand
// fragments and output accumulators live in its registers.  The other operand's rows are streamed through LDS by
// direct global->LDS transfers.  Two shapes:
//   shared (SPLIT = false): 4 wavefronts with 64 stationary rows share 32-row tiles, double-buffered, one workgroup
//     barrier per tile.  Re-reads the stream least.
//   split (SPLIT = true): 8 wavefronts with the SAME 16 stationary rows, each streaming an eighth of the other rows
//     (16 of every 128) through a private piece of LDS without any barrier; their partial results are combined through
//     LDS at the end.  Four times as many workgroups, each on a whole CU, which is what a short shard lacks: 3055 rows
//     of 6 heads are 288 workgroups of 64 rows on 256 CUs (two rounds, the second one nearly empty) but 1146 of 16 rows.
//   split, two a CU (TWO, head_dim 64): the same with one tile buffer instead of two, so that 65 KB (backward: 73) of LDS and 128
//     registers leave room for a second workgroup: 4 wavefronts per SIMD instead of 2 cover each other's LDS reads, vector
//     work and transfers, where with 2 the matrix pipes idle for a quarter of the time.  us, shared / split / two a CU, all
//     keys visible: forward of 1500 rows and keys, 24 heads 168 / 181 / 143; backward of 2048, 8 / 8 heads 254 / 302 / 245,
//     of 1500, 24 / 8 heads 529 / 507 / 411; diagonal: forward of 2048, 24 heads 155 / 179 / 135, backward 666 / 494 / 392.
// What bounds it: the matrix pipes (256 flop / clk / CU, 157 TFLOP/s; a library product reaches 154).  A 16-byte LDS read
// per lane feeds four MFMAs of 32 cycles, so LDS needs a quarter of its rate, and the vector work per 16 x 16 block of
// scores (4 per lane) is ~40 operations against 2048 cycles of MFMA (D = 128).  Measured, executed flops of a launch that
// fills the chip (4096 rows x 4096 keys x 16 heads x 128, shared shape, a size that goes to hexi_f32_bf16x3.hip since): forward 121, dQ 134, dK/dV 134 TFLOP/s.  The plain-FMA
// kernels before these read both operands of every product from LDS element by element and put 64 x nq / nkv rows
// in flight per workgroup: 3055 rows x 12011 keys, 6 / 2 heads, forward + backward 54.8 ms, now 2.77 ms; 1024 rows x 2048
// keys, 4 heads of 64: 1486 us, now 113 us (bound there by launch latency and by 2 wavefronts per SIMD walking 8 blocks each).
//
// v_mfma_f32_16x16x4_f32 layout (lane = 16 g + l): A: row l, contraction slot g; B: column l, slot g; C: column l,
// register r holds row 4 g + r.  The contraction index may be permuted as long as A and B agree:
//   scores (contraction over the head dimension): slot g of MFMA 4 G + j is column 16 G + 4 g + j, so that one
//     128-bit row read serves the four MFMAs of a G;
//   accumulations (contraction over 16 streamed rows): slot g of MFMA r is streamed row 4 g + r, which is how the
//     score registers come out, so register r of the probabilities is the operand as it stands; the other operand,
//     output columns 64 half + 4 l + j of that row, is one 128-bit read for four accumulators (half, j = 0..3).
//     Register r' of accumulator (half, j) is then output column 64 half + 16 g + 4 r' + j of row l.
// LDS tiles are [TK][D] floats with the 16-byte pieces of a row permuted by piece ^ (row & 15): both the row reads
// (16 rows, one piece) and the column reads (one row, 16 pieces) then touch all 64 banks once.
#pragma once
#include "hexi_internal.h"
#include "hexi_mfma.h"
#include "hexi_f32_common.h"

namespace { namespace rows16 {

__device__ __forceinline__ f32x4 mfma16_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ float max_over_groups(float x)      // max over the four lanes l, l + 16, l + 32, l + 48
{
    const unsigned xi = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
    return max_across_halves(max2(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float sum_over_groups(float x)
{
    const unsigned xi = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
    return sum_across_halves(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// P of a score: 2^(s (c_hi + c_lo) + nl_hi + nl_lo).  The low product takes a finite score: one that overflowed to -inf has
// P = 0, also where c_lo is negative or zero (inf - inf, 0 x inf).
__device__ __forceinline__ float prob(float s, float c_hi, float c_lo, float nl_hi, float nl_lo)
{
    return fast_exp2(fmaf(s, c_hi, nl_hi) + fmaf(max2(s, -3.402823466e38f), c_lo, nl_lo));
}

template <int D_, bool SPLIT_, bool TWO_, int NW_ = SPLIT_ ? 8 : 4, int CHAINS_ = 1, bool CLEAR_ = false> struct F32Cfg {
    static constexpr int D = D_, CHAINS = CHAINS_;           // chains of sums of a score: 1 or 4
    static constexpr bool CLEAR = CLEAR_;                  // rows past the end are zeros (SPLIT): no 0 x inf of theirs where the last row is infinite
    static constexpr bool SPLIT = SPLIT_, TWO = TWO_;
    static_assert(D == 64 || D == 128, "head_dim 64 or 128");
    static constexpr bool PRIVATE = SPLIT;                 // the streamed rows of a wavefront are its own
    static constexpr int NW = NW_;                         // wavefronts per workgroup
    static constexpr int S = SPLIT ? NW : 1;               // splits of the streamed rows
    static constexpr int R = NW / S;                       // 16-row blocks of stationary rows
    static constexpr int ROWS = 16 * R;                    // stationary rows per workgroup
    static constexpr int TK = SPLIT ? 16 * S : 32;         // streamed rows per tile
    static constexpr int NBLK = TK / 16 / S;               // 16-row blocks of the tile per wavefront: 1 or 2
    static constexpr int ROW_BYTES = 4 * D, PIECES = D / 4;
    static constexpr int TILE_BYTES = TK * ROW_BYTES;
    static constexpr int XFERS = TILE_BYTES / 1024 / NW;   // transfers per wavefront and tile (its own rows when split)
    // Tile buffers: two, or one where two would not fit (128 KB for K and V) or would leave no room for a second workgroup on the CU
    // (TWO): a wavefront with rows of its own refills its part as soon as it is done with it, and the other wavefronts of the SIMD
    // cover the wait.
    static constexpr int NBUF = SPLIT && (D == 128 || TWO) ? 1 : 2;
    static constexpr int NG = D / 16;                      // 16-column groups of the head dimension
    static constexpr int NH = D / 64;                      // 64-column halves
    static constexpr int PITCH = D + 4;                    // floats per staged output row
    static constexpr int STAGE_FLOATS = NW * 16 * PITCH;   // one 16-row block per wavefront
};

// Byte offset of 16-byte piece `c` of row `row` within a tile.
template <int ROW_BYTES> __device__ __forceinline__ uint32_t piece_off(int row, int c) { return (uint32_t)(row * ROW_BYTES + 16 * (c ^ (row & 15))); }

// The fetching side of a tile: lane parts of the transfers of one wavefront (XFERS of them per tensor and tile).
template <class C> struct TileFetch {
    uint32_t off[C::XFERS];    // byte offset of the lane's piece from the tile's first row
    int row[C::XFERS];         // its row within the tile
    __device__ __forceinline__ TileFetch(int wave, int lane, long long stride_tok)
    {
#pragma unroll
        for (int i = 0; i < C::XFERS; ++i) {
            const int pos = (wave * C::XFERS + i) * 1024 + 16 * lane;
            const int r = pos / C::ROW_BYTES, p = (pos % C::ROW_BYTES) / 16;
            row[i] = r;
            off[i] = 4u * (uint32_t)(r * (int)stride_tok) + 16u * (uint32_t)(p ^ (r & 15));
        }
    }
    // rows [row0, row0 + TK) of `src` (its row 0 is packed row 0 of the tensor's head); rows past `total` re-read the last one
    __device__ __forceinline__ void issue(const float* src, long long stride_tok, int row0, int total, uint32_t lds, int wave) const
    {
        const float* base = src + (long long)row0 * stride_tok;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds + wave * C::XFERS * 1024);
        if (row0 + C::TK <= total) {
#pragma unroll
            for (int i = 0; i < C::XFERS; ++i) lds_dma16_base(base, off[i], __builtin_amdgcn_readfirstlane(dst + i * 1024));
        } else {
#pragma unroll
            for (int i = 0; i < C::XFERS; ++i) {
                uint32_t o = off[i];
                if (row0 + row[i] >= total) o -= 4u * (uint32_t)((row0 + row[i] - (total - 1)) * (int)stride_tok);
                lds_dma16_base(base, o, __builtin_amdgcn_readfirstlane(dst + i * 1024));
            }
        }
    }
};

// The tile this wavefront fetched last has landed, and (when tiles are shared) so have the other wavefronts' parts of it.
template <class C> __device__ __forceinline__ void tile_landed()
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (!C::PRIVATE) __syncthreads();
}

// Of the wavefront's own 16 rows of a tile, which start at row `row0` of `total`, those past the end become zeros.
template <class C> __device__ __forceinline__ void clear_past_end(unsigned char* rows, int row0, int total, int lane)
{
    static_assert(C::SPLIT && C::NBLK == 1, "a wavefront's rows are its own");
    if (row0 + 16 <= total) return;
#pragma unroll
    for (int i = 0; i < 16 * C::ROW_BYTES / 1024; ++i) {
        const int off = 1024 * i + 16 * lane;
        if (row0 + off / C::ROW_BYTES >= total) *reinterpret_cast<f32x4*>(rows + off) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// Row fragments of a stationary tensor: lane (g, l) holds columns 16 G + 4 g .. + 3 of its row in frag[G].
template <int NG> __device__ __forceinline__ void load_rows(f32x4 (&frag)[NG], const float* p, int g)
{
#pragma unroll
    for (int G = 0; G < NG; ++G) frag[G] = *reinterpret_cast<const f32x4*>(p + 16 * G + 4 * g);
#pragma unroll
    for (int G = 0; G < NG; ++G) asm volatile("" ::"v"(frag[G]));     // complete before the first transfer into LDS is issued
}

// Lane parts of the LDS reads.
template <class C> struct LaneAddr {
    uint32_t row[C::NG];     // row read of row l: piece 4 G + g
    uint32_t col[4];         // column read of row 4 g + r: piece l (+ 16 half)
    __device__ __forceinline__ LaneAddr(int g, int l)
    {
#pragma unroll
        for (int G = 0; G < C::NG; ++G) row[G] = piece_off<C::ROW_BYTES>(l, 4 * G + g);
#pragma unroll
        for (int r = 0; r < 4; ++r) col[r] = piece_off<C::ROW_BYTES>(4 * g + r, l);
    }
};
__device__ __forceinline__ f32x4 lds_f4(const unsigned char* p) { return *reinterpret_cast<const f32x4*>(p); }

// out[m = streamed row][n = stationary row] = sum over the head dimension: A from LDS (row reads), B in registers.
// The reads of a step are issued before the MFMAs of the step before it (4 NT MFMAs = 128 NT cycles ahead); left to
// itself the compiler issues them a few dozen cycles before their use.  The summation order over the head dimension is
// the same in all three kernels: the rounding errors of a score and of the LSE it went into then cancel in P.  At head_dim 128, where the LSE may
// come from the split-operand forward instead (hexi_f32_bf16x3.hip), or go to its backward, four chains, one per MFMA of a group, halve the error of
// one and more than make up for what no longer cancels: errors of dq, dk, dv, K scaled by 3, 777 x 1000 x 8/2 heads, one chain in all kernels 1, that
// forward with one chain here 1.5, 1.5, 1.7, with four 0.79, 0.78, 0.81.  Steps that take no kernel of that file keep the one chain
// (hexi_f32_chains(); a backward of 1264 x 108 x 48/24 heads 182 us, with four, and one
// shared workgroup on a CU, 200).
template <class C, int NT> __device__ __forceinline__ void score_block(f32x4 (&out)[NT], const unsigned char* const (&tile)[NT], const LaneAddr<C>& la, const f32x4* const (&frag)[NT])
{
    constexpr int CH = C::CHAINS;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 x[2][NT], sum[CH][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) x[0][t] = lds_f4(tile[t] + la.row[0]);
#pragma unroll
    for (int G = 0; G < C::NG; ++G) {
        if (G + 1 < C::NG) {
#pragma unroll
            for (int t = 0; t < NT; ++t) x[(G + 1) & 1][t] = lds_f4(tile[t] + la.row[G + 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < NT; ++t) sum[j % CH][t] = mfma16_f32(x[G & 1][t][j], frag[t][G][j], G == 0 && j < CH ? zero : sum[j % CH][t]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if constexpr (CH == 4) out[t] = (sum[0][t] + sum[1][t]) + (sum[2][t] + sum[3][t]);
        else out[t] = sum[0][t];
    }
}

// acc[u][4 half + j] += (streamed rows' columns of tile[u])^T x p[u] for NU products.  The first reads are the caller's
// (ColReads::first, issued before the vector work that produces p); the others are issued one step ahead.
template <class C, int NU> struct ColReads {
    f32x4 x[2][C::NH];
    const unsigned char* tile[NU];
    __device__ __forceinline__ void read(const LaneAddr<C>& la, int step)       // step = 4 u + r
    {
#pragma unroll
        for (int h = 0; h < C::NH; ++h) x[step & 1][h] = lds_f4(tile[step / 4] + la.col[step & 3] + 256 * h);
    }
    __device__ __forceinline__ void first(const LaneAddr<C>& la) { read(la, 0); __builtin_amdgcn_sched_barrier(0); }
    __device__ __forceinline__ void run(const LaneAddr<C>& la, f32x4 (*const (&acc)[NU])[4 * C::NH], const f32x4* const (&p)[NU])
    {
#pragma unroll
        for (int st = 0; st < 4 * NU; ++st) {
            if (st + 1 < 4 * NU) read(la, st + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < C::NH; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) (*acc[st / 4])[4 * h + j] = mfma16_f32(x[st & 1][h][j], (*p[st / 4])[st & 3], (*acc[st / 4])[4 * h + j]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// The wavefront's 16 x D accumulator block, times `w` (per row), as rows of a staging area.
template <class C> __device__ __forceinline__ void stage_rows(float* stage, const f32x4 (&acc)[4 * C::NH], int g, int l, float w)
{
#pragma unroll
    for (int h = 0; h < C::NH; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<float4*>(&stage[l * C::PITCH + 64 * h + 16 * g + 4 * r]) =
                make_float4(acc[4 * h][r] * w, acc[4 * h + 1][r] * w, acc[4 * h + 2][r] * w, acc[4 * h + 3][r] * w);
}

template <class C> struct FwdSmem {
    union {
        struct { unsigned char k[C::NBUF][C::TILE_BYTES], v[C::NBUF][C::TILE_BYTES]; } t;
        struct { float stage[C::STAGE_FLOATS], m[C::NW * 16], l[C::NW * 16], w[C::NW * 16], wa[16 * C::R]; } e;
    };
    int kpos[2][C::TK];
};

template <class C> __device__ __forceinline__ void fwd_unit(const FwdArgs& a, const int h, const int q_tile, FwdSmem<C>& sm)
{
    constexpr int D = C::D, NW = C::NW, S = C::S, TK = C::TK, NBLK = C::NBLK;
    constexpr bool SPLIT = C::SPLIT, TWO = C::TWO;
    const AttnGeom& g = a.g;
    auto& kpos = sm.kpos;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave % C::R, sp = wave / C::R;        // row block, split
    const int grp = lane >> 4, l16 = lane & 15;

    const int kvh = g.kv_of_q[h];
    const int row0 = q_tile * C::ROWS;
    const int my_row = row0 + 16 * rb + l16;
    const int my_row_c = my_row < g.lq ? my_row : g.lq - 1;
    const int my_pos = my_row < g.lq ? seg_pos_of_row(g.qs, my_row) : -1;
    const int last_row = (row0 + C::ROWS < g.lq ? row0 + C::ROWS : g.lq) - 1;
    const int n_vis = seg_rows_le(g.ks, seg_pos_of_row(g.qs, last_row));      // visible columns form the prefix [0, n_vis)
    const int n_full = seg_rows_le(g.ks, seg_pos_of_row(g.qs, row0)) / TK;    // tiles no row needs a mask for
    if (n_vis == 0 && a.accumulate) return;               // merging an empty partial is the identity
    const int n_tiles = (n_vis - (SPLIT ? 16 * wave : 0) + TK - 1) / TK;      // of this wavefront: those that hold a visible row

    const float* k = static_cast<const float*>(a.k) + (long long)kvh * g.kv_stride_head;
    const float* v = static_cast<const float*>(a.v) + (long long)kvh * g.kv_stride_head;
    f32x4 qf[C::NG];
    load_rows(qf, static_cast<const float*>(a.q) + (long long)my_row_c * g.q_stride_tok + (long long)h * g.q_stride_head, grp);
    const LaneAddr<C> la(grp, l16);
    const TileFetch<C> fetch(wave, lane, g.kv_stride_tok);
    const uint32_t lds_k = (uint32_t)(uintptr_t)(&sm.t.k[0][0]), lds_v = (uint32_t)(uintptr_t)(&sm.t.v[0][0]);
    const int pos_slot = C::PRIVATE ? (lane < 16 ? 16 * wave + lane : TK) : tid;      // the row whose position this thread looks up
    auto fetch_tile = [&](int t) {
        const int buf = t & 1;
        fetch.issue(k, g.kv_stride_tok, t * TK, g.lc, lds_k + (buf % C::NBUF) * C::TILE_BYTES, wave);
        fetch.issue(v, g.kv_stride_tok, t * TK, g.lc, lds_v + (buf % C::NBUF) * C::TILE_BYTES, wave);
        if (t >= n_full && pos_slot < TK) kpos[buf][pos_slot] = t * TK + pos_slot < g.lc ? seg_pos_of_row(g.ks, t * TK + pos_slot) : 0x7fffffff;
    };

    f32x4 acc[4 * C::NH];
#pragma unroll
    for (int i = 0; i < 4 * C::NH; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    // scores in units of log2: s * scale * log2(e), with the constant carried as two floats
    const float c_hi = g.scale * LOG2E_HI, c_lo = fmaf(g.scale, LOG2E_HI, -c_hi) + g.scale * LOG2E_LO;
    float m_run = -INFINITY, l_run = 0.f;

    if (n_tiles > 0) fetch_tile(0);
    for (int t = 0; t < n_tiles; ++t) {
        tile_landed<C>();         // and everyone is done with the buffer of tile t + 1
        if (C::NBUF == 2 && t + 1 < n_tiles) fetch_tile(t + 1);
        const int buf = t & 1;
        const unsigned char* kt = &sm.t.k[buf % C::NBUF][sp * NBLK * 16 * C::ROW_BYTES];
        const unsigned char* vt = &sm.t.v[buf % C::NBUF][sp * NBLK * 16 * C::ROW_BYTES];
        if constexpr (C::CLEAR) clear_past_end<C>(&sm.t.v[buf % C::NBUF][16 * wave * C::ROW_BYTES], t * TK + 16 * wave, g.lc, lane);
        f32x4 s[NBLK];
        {
            const unsigned char* tiles[NBLK];
            const f32x4* frags[NBLK];
#pragma unroll
            for (int b = 0; b < NBLK; ++b) { tiles[b] = kt + b * 16 * C::ROW_BYTES; frags[b] = qf; }
            score_block<C, NBLK>(s, tiles, la, frags);
        }
        ColReads<C, NBLK> pv;
#pragma unroll
        for (int b = 0; b < NBLK; ++b) pv.tile[b] = vt + b * 16 * C::ROW_BYTES;
        pv.first(la);
        if (t >= n_full) {
#pragma unroll
            for (int b = 0; b < NBLK; ++b) {
                const int4 p4 = *reinterpret_cast<const int4*>(&kpos[buf][16 * (sp * NBLK + b) + 4 * grp]);
                if (p4.x > my_pos) s[b][0] = -INFINITY;
                if (p4.y > my_pos) s[b][1] = -INFINITY;
                if (p4.z > my_pos) s[b][2] = -INFINITY;
                if (p4.w > my_pos) s[b][3] = -INFINITY;
            }
        }
        // running maximum of the row over this wavefront's keys, in raw score units
        float mx = max2(max2(s[0][0], s[0][1]), max2(s[0][2], s[0][3]));
#pragma unroll
        for (int b = 1; b < NBLK; ++b) mx = max2(mx, max2(max2(s[b][0], s[b][1]), max2(s[b][2], s[b][3])));
        mx = max_over_groups(mx);
        if (__any(mx > m_run)) {
            const float m_new = max2(m_run, mx);
            const float x = m_run - m_new;
            const float alpha = m_new == -INFINITY ? 1.f : fast_exp2(fmaf(x, c_hi, x == -INFINITY ? 0.f : x * c_lo));
            l_run *= alpha;
#pragma unroll
            for (int i = 0; i < 4 * C::NH; ++i) acc[i] *= alpha;
            m_run = m_new;
        }
        const float m_use = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = s[b][r] - m_use;
                s[b][r] = fast_exp2(fmaf(x, c_hi, x == -INFINITY ? 0.f : x * c_lo));
                l_run += s[b][r];
            }
        f32x4 (*accs[NBLK])[4 * C::NH];
        const f32x4* ps[NBLK];
#pragma unroll
        for (int b = 0; b < NBLK; ++b) { accs[b] = &acc; ps[b] = &s[b]; }
        pv.run(la, accs, ps);
        if (C::NBUF == 1 && t + 1 < n_tiles) { if (TWO) reads_done(); fetch_tile(t + 1); }
    }

    // Combine the splits and merge with the running (o, lse): weights per (row, split), then a row-contiguous pass.
    l_run = sum_over_groups(l_run);
    __syncthreads();              // the tiles are free
    stage_rows<C>(&sm.e.stage[wave * 16 * C::PITCH], acc, grp, l16, 1.0f);
    if (grp == 0) { sm.e.m[wave * 16 + l16] = m_run; sm.e.l[wave * 16 + l16] = l_run; }
    __syncthreads();
    if (tid < C::ROWS) {          // thread = row of the workgroup (its statistics of split s at s * ROWS + tid)
        float m = -INFINITY;
#pragma unroll
        for (int s = 0; s < S; ++s) m = fmaxf(m, sm.e.m[s * C::ROWS + tid]);
        float l = 0.f, e[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const float ms = sm.e.m[s * C::ROWS + tid];
            const float x = ms - m;
            e[s] = ms == -INFINITY ? 0.f : fast_exp2(fmaf(x, c_hi, x * c_lo));
            l += e[s] * sm.e.l[s * C::ROWS + tid];
        }
        const float lse_part = l > 0.f ? fmaf(m, g.scale, logf(l)) : -INFINITY;
        float wb = l > 0.f ? 1.0f / l : 0.f, wa = 0.f, lse_new = lse_part;
        const int row = row0 + tid;
        if (row < g.lq) {
            float* lp = a.lse + (long long)h * g.lq + row;
            if (a.accumulate) {
                const float la_old = *lp;
                const float mm = fmaxf(la_old, lse_part);
                if (mm == -INFINITY) { wb = 0.f; lse_new = -INFINITY; }
                else {
                    const float ea = expf(la_old - mm), eb = expf(lse_part - mm), inv = 1.0f / (ea + eb);
                    wa = ea * inv;
                    wb *= eb * inv;
                    lse_new = mm + logf(ea + eb);
                }
            }
            *lp = lse_new;
        }
#pragma unroll
        for (int s = 0; s < S; ++s) sm.e.w[s * C::ROWS + tid] = e[s] * wb;
        sm.e.wa[tid] = wa;
    }
    __syncthreads();
    for (int i = tid; i < C::ROWS * C::PIECES; i += 64 * NW) {
        const int r = i / C::PIECES, c = 4 * (i % C::PIECES);
        if (row0 + r >= g.lq) continue;
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s) x += sm.e.w[s * C::ROWS + r] * *reinterpret_cast<const f32x4*>(&sm.e.stage[(s * C::ROWS + r) * C::PITCH + c]);
        f32x4* op = reinterpret_cast<f32x4*>(a.o + ((long long)(row0 + r) * g.nq + h) * D + c);
        if (a.accumulate) x += sm.e.wa[r] * *op;
        *op = x;
    }
}

// dQ: S^T = K Q^T and dP^T = V dO^T per tile, dS^T = P^T (dP^T - Delta), dQ^T += K^T dS^T.
template <class C> struct DqSmem {
    union {
        struct { unsigned char k[C::NBUF][C::TILE_BYTES], v[C::NBUF][C::TILE_BYTES]; } t;
        float stage[C::STAGE_FLOATS];
    };
    int kpos[2][C::TK];
};

template <class C> __device__ __forceinline__ void dq_unit(const BwdArgs& a, const int h, const int q_tile, DqSmem<C>& sm)
{
    constexpr int D = C::D, NW = C::NW, S = C::S, TK = C::TK, NBLK = C::NBLK;
    constexpr bool SPLIT = C::SPLIT, TWO = C::TWO;
    const AttnGeom& g = a.g;
    auto& kpos = sm.kpos;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave % C::R, sp = wave / C::R;
    const int grp = lane >> 4, l16 = lane & 15;
    const int kvh = g.kv_of_q[h];
    const int row0 = q_tile * C::ROWS;
    const int my_row = row0 + 16 * rb + l16;
    const int my_row_c = my_row < g.lq ? my_row : g.lq - 1;
    const int my_pos = my_row < g.lq ? seg_pos_of_row(g.qs, my_row) : -1;
    const int last_row = (row0 + C::ROWS < g.lq ? row0 + C::ROWS : g.lq) - 1;
    const int n_vis = seg_rows_le(g.ks, seg_pos_of_row(g.qs, last_row));
    const int n_full = seg_rows_le(g.ks, seg_pos_of_row(g.qs, row0)) / TK;
    if (n_vis == 0) return;                               // dq_acc unchanged
    const int n_tiles = (n_vis - (SPLIT ? 16 * wave : 0) + TK - 1) / TK;

    const float* k = static_cast<const float*>(a.k) + (long long)kvh * g.kv_stride_head;
    const float* v = static_cast<const float*>(a.v) + (long long)kvh * g.kv_stride_head;
    const float l = a.lse[(long long)h * g.lq + my_row_c];
    const float delta = a.delta[(long long)h * g.lq + my_row_c];
    f32x4 qf[C::NG], gf[C::NG];
    const long long q_off = (long long)my_row_c * g.q_stride_tok + (long long)h * g.q_stride_head;
    load_rows(qf, static_cast<const float*>(a.q) + q_off, grp);
    load_rows(gf, static_cast<const float*>(a.d_o) + q_off, grp);
    const float c_hi = g.scale * LOG2E_HI, c_lo = fmaf(g.scale, LOG2E_HI, -c_hi) + g.scale * LOG2E_LO;
    float nl_hi, nl_lo;
    neg_lse_log2(l, nl_hi, nl_lo);

    const LaneAddr<C> la(grp, l16);
    const TileFetch<C> fetch(wave, lane, g.kv_stride_tok);
    const uint32_t lds_k = (uint32_t)(uintptr_t)(&sm.t.k[0][0]), lds_v = (uint32_t)(uintptr_t)(&sm.t.v[0][0]);
    const int pos_slot = C::PRIVATE ? (lane < 16 ? 16 * wave + lane : TK) : tid;      // the row whose position this thread looks up
    auto fetch_tile = [&](int t) {
        const int buf = t & 1;
        fetch.issue(k, g.kv_stride_tok, t * TK, g.lc, lds_k + (buf % C::NBUF) * C::TILE_BYTES, wave);
        fetch.issue(v, g.kv_stride_tok, t * TK, g.lc, lds_v + (buf % C::NBUF) * C::TILE_BYTES, wave);
        if (t >= n_full && pos_slot < TK) kpos[buf][pos_slot] = t * TK + pos_slot < g.lc ? seg_pos_of_row(g.ks, t * TK + pos_slot) : 0x7fffffff;
    };

    f32x4 acc[4 * C::NH];
#pragma unroll
    for (int i = 0; i < 4 * C::NH; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (n_tiles > 0) fetch_tile(0);
    for (int t = 0; t < n_tiles; ++t) {
        tile_landed<C>();
        if (C::NBUF == 2 && t + 1 < n_tiles) fetch_tile(t + 1);
        const int buf = t & 1;
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            const unsigned char* kt = &sm.t.k[buf % C::NBUF][(sp * NBLK + b) * 16 * C::ROW_BYTES];
            const unsigned char* vt = &sm.t.v[buf % C::NBUF][(sp * NBLK + b) * 16 * C::ROW_BYTES];
            if constexpr (C::CLEAR) clear_past_end<C>(&sm.t.k[buf % C::NBUF][16 * wave * C::ROW_BYTES], t * TK + 16 * wave, g.lc, lane);
            f32x4 sd[2];       // S^T and dP^T of the block: register r is key 4 grp + r
            const unsigned char* const tiles[2] = {kt, vt};
            const f32x4* const frags[2] = {qf, gf};
            score_block<C, 2>(sd, tiles, la, frags);
            ColReads<C, 1> kc;
            kc.tile[0] = kt;
            kc.first(la);
            int4 p4 = make_int4(-1, -1, -1, -1);
            if (t >= n_full) p4 = *reinterpret_cast<const int4*>(&kpos[buf][16 * (sp * NBLK + b) + 4 * grp]);
            const int pv[4] = {p4.x, p4.y, p4.z, p4.w};
            f32x4 ds;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float p = prob(sd[0][r], c_hi, c_lo, nl_hi, nl_lo);
                ds[r] = pv[r] > my_pos ? 0.f : p * (sd[1][r] - delta);
            }
            f32x4 (*const accs[1])[4 * C::NH] = {&acc};
            const f32x4* const ps[1] = {&ds};
            kc.run(la, accs, ps);
        }
        if (C::NBUF == 1 && t + 1 < n_tiles) { if (TWO) reads_done(); fetch_tile(t + 1); }
    }
    __syncthreads();
    stage_rows<C>(&sm.stage[wave * 16 * C::PITCH], acc, grp, l16, g.scale);
    __syncthreads();
    // Added with atomics, consecutive lanes on consecutive floats: chunks of one shard may be in flight on several streams.
    // One addition per element and call, so calls in stream order still have a fixed order.
    for (int i = tid; i < C::ROWS * D; i += 64 * NW) {
        const int r = i / D, c = i % D;
        if (row0 + r >= g.lq) continue;
        float x = sm.stage[r * C::PITCH + c];
#pragma unroll
        for (int s = 1; s < S; ++s) x += sm.stage[(s * C::ROWS + r) * C::PITCH + c];
        global_atomic_add(a.dq + ((long long)(row0 + r) * g.nq + h) * D + c, x);
    }
}

// dK / dV: the stationary rows are keys, the streamed rows q rows (of every q head that reads the kv head, one head
// after the other): S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.  Of those q heads the ones in [h_first, h_end); `atomic`: the result is
// added to dk and dv with atomics.
template <class C> struct DkdvSmem {
    union {
        struct { unsigned char q[C::NBUF][C::TILE_BYTES], g[C::NBUF][C::TILE_BYTES]; } t;
        float stage[C::STAGE_FLOATS];
    };
    __attribute__((aligned(16))) float lse[2][C::PRIVATE ? 64 * C::NW : 64], delta[2][C::PRIVATE ? 64 * C::NW : 64];
    __attribute__((aligned(16))) int qpos[2][C::TK];
};

template <class C> __device__ __forceinline__ void dkdv_unit(const BwdArgs& a, const int kvh, const int kv_tile, DkdvSmem<C>& sm, const int h_first, const int h_end, const bool atomic)
{
    constexpr int D = C::D, NW = C::NW, S = C::S, TM = C::TK, NBLK = C::NBLK;
    constexpr bool SPLIT = C::SPLIT, TWO = C::TWO;
    const AttnGeom& g = a.g;
    constexpr int SET = C::PRIVATE ? 64 : 0;      // row scalars: one set of 64 lanes per wavefront, or one for all
    auto &lse = sm.lse, &delta = sm.delta;
    auto& qpos = sm.qpos;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave % C::R, sp = wave / C::R;
    const int grp = lane >> 4, l16 = lane & 15;
    const int col0 = kv_tile * C::ROWS;
    const int my_col = col0 + 16 * rb + l16;
    const int my_col_c = my_col < g.lc ? my_col : g.lc - 1;
    const int my_kpos = my_col < g.lc ? seg_pos_of_row(g.ks, my_col) : 0x7fffffff;
    const int last_col = (col0 + C::ROWS < g.lc ? col0 + C::ROWS : g.lc) - 1;
    const int row_first = seg_rows_le(g.qs, seg_pos_of_row(g.ks, col0) - 1);         // rows before it see nothing of the tile
    const int row_full = seg_rows_le(g.qs, seg_pos_of_row(g.ks, last_col) - 1);      // rows from it on see all of it
    const int tile0 = row_first / TM, n_qtiles = (g.lq + TM - 1) / TM;
    const int per_head = n_qtiles - tile0;
    const bool key_ragged = col0 + C::ROWS > g.lc;        // padding keys are masked through their position

    f32x4 kf[C::NG], vf[C::NG];
    const long long k_off = (long long)my_col_c * g.kv_stride_tok + (long long)kvh * g.kv_stride_head;
    load_rows(kf, static_cast<const float*>(a.k) + k_off, grp);
    load_rows(vf, static_cast<const float*>(a.v) + k_off, grp);
    const float c_hi = g.scale * LOG2E_HI, c_lo = fmaf(g.scale, LOG2E_HI, -c_hi) + g.scale * LOG2E_LO;
    const LaneAddr<C> la(grp, l16);
    const TileFetch<C> fetch(wave, lane, g.q_stride_tok);
    const uint32_t lds_q = (uint32_t)(uintptr_t)(&sm.t.q[0][0]), lds_g = (uint32_t)(uintptr_t)(&sm.t.g[0][0]);
    auto next_head = [&](int h) { for (++h; h < h_end && g.kv_of_q[h] != kvh; ++h) {} return h; };
    int fetch_h = next_head(h_first - 1), fetch_t = tile0;
    const int pos_slot = C::PRIVATE ? (lane < 16 ? 16 * wave + lane : TM) : tid;
    auto fetch_tile = [&](int buf) {
        const long long off = (long long)fetch_h * g.q_stride_head;
        fetch.issue(static_cast<const float*>(a.q) + off, g.q_stride_tok, fetch_t * TM, g.lq, lds_q + (buf % C::NBUF) * C::TILE_BYTES, wave);
        fetch.issue(static_cast<const float*>(a.d_o) + off, g.q_stride_tok, fetch_t * TM, g.lq, lds_g + (buf % C::NBUF) * C::TILE_BYTES, wave);
        // The rows' LSE and Delta: a 4-byte-per-lane transfer each, by wavefronts 0 and 1 for the tile, or by every
        // wavefront for its own 16 rows.
        const int lrow = C::PRIVATE ? 16 * wave + (lane & 15) : lane;
        const int row = fetch_t * TM + lrow < g.lq ? fetch_t * TM + lrow : g.lq - 1;
        if (C::PRIVATE || wave == 0) lds_dma4(a.lse + (long long)fetch_h * g.lq + row, __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&lse[buf][SET * wave]));
        if (C::PRIVATE || wave == 1) lds_dma4(a.delta + (long long)fetch_h * g.lq + row, __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)&delta[buf][SET * wave]));
        if (pos_slot < TM && (fetch_t * TM < row_full || key_ragged || fetch_t == n_qtiles - 1))
            qpos[buf][pos_slot] = fetch_t * TM + pos_slot < g.lq ? seg_pos_of_row(g.qs, fetch_t * TM + pos_slot) : -1;
        if (++fetch_t == n_qtiles) { fetch_t = tile0; fetch_h = next_head(fetch_h); }
    };

    f32x4 dk[4 * C::NH], dv[4 * C::NH];
#pragma unroll
    for (int i = 0; i < 4 * C::NH; ++i) { dk[i] = f32x4{0.f, 0.f, 0.f, 0.f}; dv[i] = dk[i]; }
    if (per_head > 0) {
        int buf = 0, t = tile0;
        if (fetch_h < h_end) fetch_tile(0);
        for (int h = next_head(h_first - 1); h < h_end;) {
            tile_landed<C>();
            if (C::NBUF == 2 && fetch_h < h_end) fetch_tile(buf ^ 1);
            // (the last tile may hold padding rows, whose position is -1)
            const bool masked = t * TM < row_full || key_ragged || t == n_qtiles - 1;
#pragma unroll
            for (int b = 0; b < NBLK; ++b) {
                const int blk = sp * NBLK + b;
                if (SPLIT && (t * TM + 16 * blk >= g.lq || t * TM + 16 * blk + 16 <= row_first)) continue;      // rows that see nothing
                const unsigned char* qt = &sm.t.q[buf % C::NBUF][blk * 16 * C::ROW_BYTES];
                const unsigned char* gt = &sm.t.g[buf % C::NBUF][blk * 16 * C::ROW_BYTES];
                if constexpr (C::CLEAR) {
                    clear_past_end<C>(&sm.t.q[buf % C::NBUF][16 * wave * C::ROW_BYTES], t * TM + 16 * wave, g.lq, lane);
                    clear_past_end<C>(&sm.t.g[buf % C::NBUF][16 * wave * C::ROW_BYTES], t * TM + 16 * wave, g.lq, lane);
                }
                f32x4 sd[2];       // S and dP of the block: register r is row 4 grp + r
                const unsigned char* const tiles[2] = {qt, gt};
                const f32x4* const frags[2] = {kf, vf};
                score_block<C, 2>(sd, tiles, la, frags);
                ColReads<C, 2> cols;
                cols.tile[0] = gt;
                cols.tile[1] = qt;
                cols.first(la);
                const int sc = (C::PRIVATE ? SET * wave : 16 * blk) + 4 * grp;
                const f32x4 l4 = *reinterpret_cast<const f32x4*>(&lse[buf][sc]);
                const f32x4 dl = *reinterpret_cast<const f32x4*>(&delta[buf][sc]);
                f32x4 p, ds;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float nl_hi, nl_lo;
                    neg_lse_log2(l4[r], nl_hi, nl_lo);
                    p[r] = prob(sd[0][r], c_hi, c_lo, nl_hi, nl_lo);
                }
                if (masked) {
                    const int4 q4 = *reinterpret_cast<const int4*>(&qpos[buf][16 * blk + 4 * grp]);
                    if (my_kpos > q4.x) p[0] = 0.f;
                    if (my_kpos > q4.y) p[1] = 0.f;
                    if (my_kpos > q4.z) p[2] = 0.f;
                    if (my_kpos > q4.w) p[3] = 0.f;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) ds[r] = p[r] * (sd[1][r] - dl[r]);
                f32x4 (*const accs[2])[4 * C::NH] = {&dv, &dk};
                const f32x4* const ps[2] = {&p, &ds};
                cols.run(la, accs, ps);
            }
            if (C::NBUF == 1 && fetch_h < h_end) { if (TWO) reads_done(); fetch_tile(buf ^ 1); }
            buf ^= 1;
            if (++t == n_qtiles) { t = tile0; h = next_head(h); }
        }
    }
    auto write_out = [&](float* out, const f32x4 (&acc)[4 * C::NH], float w) {
        __syncthreads();
        stage_rows<C>(&sm.stage[wave * 16 * C::PITCH], acc, grp, l16, w);
        __syncthreads();
        for (int i = tid; i < C::ROWS * C::PIECES; i += 64 * NW) {
            const int r = i / C::PIECES, c = 4 * (i % C::PIECES);
            if (col0 + r >= g.lc) continue;
            f32x4 x = *reinterpret_cast<const f32x4*>(&sm.stage[r * C::PITCH + c]);
#pragma unroll
            for (int s = 1; s < S; ++s) x += *reinterpret_cast<const f32x4*>(&sm.stage[(s * C::ROWS + r) * C::PITCH + c]);
            f32x4* op = reinterpret_cast<f32x4*>(out + ((long long)(col0 + r) * g.nkv + kvh) * D + c);
            if (atomic) {
#pragma unroll
                for (int e = 0; e < 4; ++e) global_atomic_add(reinterpret_cast<float*>(op) + e, x[e]);
                continue;
            }
            if (a.accumulate) x += *op;
            *op = x;
        }
    };
    write_out(a.dv, dv, 1.0f);
    write_out(a.dk, dk, g.scale);
}

} }  // namespace rows16

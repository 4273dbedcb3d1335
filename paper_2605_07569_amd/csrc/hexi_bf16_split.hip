// bf16 ring step (forward, dQ, dK/dV) for the smallest launches: a workgroup owns 32 stationary rows (q rows of one head; keys of one
// kv head in the dK/dV kernel) and its 8 wavefronts split the streamed rows between them, 32 at a time (block b goes to wavefront
// b % 8).  A wavefront streams its own blocks through a private piece of LDS, without any barrier before the end, where the partial
// results are combined through LDS in a fixed order.
//
// What bounds it: the serial chain of a workgroup, which is 8 times shorter than that of the large workgroups, of which there are too
// few there (1024 rows x 8 heads are 32 workgroups of 256 rows on 256 CUs, and 256 of 32), and, on chains of two to four blocks, its
// start and its end.  Per round of 8 blocks a CU takes 1.1 to 2.1 us: 128 KB through its 64 bytes a clock are 0.85 us alone.  The start:
// the unit's own rows come through LDS, each wavefront fetching a part (16-byte pieces of 32 rows, read by all wavefronts, were 0.7 us);
// the first block sets the softmax reference without rescaling zeros.  The end: every wavefront weighs its own partial result, the
// running values are on their way meanwhile, two barriers instead of three.  These took 512 x 512 x 4 heads x 128 from 9.7 to 8.1 us
// (forward) and from 11.3 to 8.5 us (dQ), 1024 x 1024 x 8 from 12.9 to 11.7 us.  Larger launches take the 64-row workgroups of
// hexi_bf16_quad.hip, then the large ones, which stream less per row: see the rules in hexi_shapes.h.  Measured, us per call
// (head_dim 128, fully visible chunk), large workgroups -> these: 300 rows x 700 keys, 4 / 2 heads: forward 28.3 -> 9.3, dQ
// 36.2 -> 9.8, dK/dV 23.5 -> 12.3.
//
// Operand layouts are those of the large kernels (hexi_mfma.h): scores transposed in the forward and dQ kernels (a lane
// owns a q row), keys across the lanes in the dK/dV kernel; accumulator registers go straight back in as operands, the
// other operand through transposed LDS reads.
#include "hexi_blocks.h"

namespace {

constexpr int NW = 8;          // wavefronts per workgroup

template <int D_> struct SplitCfg : BlockCfg<D_> {
    static constexpr int STAGE_FLOATS = NW * TB * BlockCfg<D_>::PITCH;
    static constexpr int OUT_VECS = TB * D_ / 4 / (64 * NW);      // float4 of the output per thread: 2 or 1
};

// out = sum over ks of (rows of the block at byte `tile` of the wavefront's LDS) x frag(ks); reads three MFMAs ahead.
template <class C, class F> __device__ __forceinline__ f32x16 row_product(const LaneAddr<C>& la, const uint32_t tile, F frag)
{
    bf16x8 x[4], y[4];
    f32x16 out = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) { x[ks] = lds_b128(la.row[ks] + tile); y[ks] = frag(ks); }
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) {
        if (ks + 3 < C::NKS) { x[(ks + 3) & 3] = lds_b128(la.row[ks + 3] + tile); y[(ks + 3) & 3] = frag(ks + 3); }
        __builtin_amdgcn_sched_barrier(0);
        out = mfma32(x[ks & 3], y[ks & 3], out);
        __builtin_amdgcn_sched_barrier(0);
    }
    return out;
}

// acc[db] += (columns of the block at `tile`)^T x p over its 32 rows; p[u] holds rows 16 u .. + 15 in accumulator order.
template <class C> __device__ __forceinline__ void col_product(f32x16 (&acc)[C::NDB], const LaneAddr<C>& la, const uint32_t tile, const bf16x8 (&p)[2])
{
    constexpr int N = 2 * C::NDB;
    bf16x8 x[4];
    auto read = [&](int st) { return lds_tr(la.tr[0][st % C::NDB] + tile + st / C::NDB * 16 * C::ROW_BYTES, la.tr[1][st % C::NDB] + tile + st / C::NDB * 16 * C::ROW_BYTES); };
#pragma unroll
    for (int st = 0; st < 3; ++st) x[st] = read(st);
#pragma unroll
    for (int st = 0; st < N; ++st) {
        if (st + 3 < N) x[(st + 3) & 3] = read(st + 3);
        __builtin_amdgcn_sched_barrier(0);
        const int db = st % C::NDB, u = st / C::NDB;
        acc[db] = mfma32(x[st & 3], p[u], acc[db]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// What the rows of a q tile see of the chunk (prefixes of its keys).
struct Visible {
    int mine;       // keys the lane's row sees (0 for padding rows)
    int n_all;      // keys some row sees
    int n_full;     // 32-key blocks every row sees in full
    __device__ __forceinline__ Visible(const AttnGeom& g, int row0, int l32)
    {
        const int n = rows_le(g.ks, pos_of_row(g.qs, row0 + l32 < g.lq ? row0 + l32 : g.lq - 1));
        n_all = __builtin_amdgcn_readlane(n, 31);
        n_full = __builtin_amdgcn_readlane(n, 0) / TB;
        mine = row0 + l32 < g.lq ? n : 0;
    }
};

// A transposed accumulator (lane = stationary row) as rows of the wavefront's staging area, times w.
template <class C> __device__ __forceinline__ void stage_transposed(float* stage, const f32x16 (&acc)[C::NDB], int l32, int hh, float w)
{
#pragma unroll
    for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int b = 0; b < 4; ++b)
            *reinterpret_cast<float4*>(&stage[l32 * C::PITCH + 32 * db + 8 * b + 4 * hh]) =
                make_float4(acc[db][4 * b] * w, acc[db][4 * b + 1] * w, acc[db][4 * b + 2] * w, acc[db][4 * b + 3] * w);
}

// Sum over the wavefronts of the staged partial results: row r, columns c .. c + 3.
template <class C> __device__ __forceinline__ f32x4 staged_sum(const float* stage, int r, int c)
{
    f32x4 x = *reinterpret_cast<const f32x4*>(&stage[r * C::PITCH + c]);
#pragma unroll
    for (int s = 1; s < NW; ++s) x += *reinterpret_cast<const f32x4*>(&stage[(s * TB + r) * C::PITCH + c]);
    return x;
}

// (at head_dim 64 two workgroups fit a CU if the registers are held to 128)
template <int D>
__global__ void __launch_bounds__(512, D == 64 ? 4 : 2) fwd_split_bf16_kernel(const FwdArgs a, const int n_q_tiles)
{
    using C = SplitCfg<D>;
    const AttnGeom& g = a.g;
    __shared__ __attribute__((aligned(1024))) union {
        struct { unsigned char t[NW][2 * C::TILE_BYTES], q[C::TILE_BYTES]; } b;     // K and V block of each wavefront, the workgroup's Q rows
        struct { float stage[C::STAGE_FLOATS], wa[TB]; } e;
    } sm;
    __shared__ float4 stat[NW][TB];                        // reference, exact sum, sum of the rounded probabilities of each split
    const int tid = threadIdx.x, lane = tid & 63;
    const int sp = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;

    // heads of a q tile side by side, the longest (last) q tiles first
    const int h = blockIdx.x;
    const int row0 = (n_q_tiles - 1 - (int)blockIdx.y) * TB;
    const int kvh = arg_byte(g.kv_of_q, h);
    const uint16_t* k = static_cast<const uint16_t*>(a.k) + (long long)kvh * g.kv_stride_head;
    const uint16_t* v = static_cast<const uint16_t*>(a.v) + (long long)kvh * g.kv_stride_head;
    const uint32_t lds = (uint32_t)(uintptr_t)(&sm.b.t[0][0]) + sp * 2 * C::TILE_BYTES, lds_q = (uint32_t)(uintptr_t)(&sm.b.q[0]);
    fetch_rows<C, TB, NW>(static_cast<const uint16_t*>(a.q) + (long long)h * g.q_stride_head, g.q_stride_tok, row0, g.lq, lds_q, sp, lane);
    const BlockFetch<C> fetch(lane, g.kv_stride_tok);
    auto fetch_k = [&](int b) { fetch.issue(k, g.kv_stride_tok, b * TB, g.lc, lds); };
    auto fetch_v = [&](int b) { fetch.issue(v, g.kv_stride_tok, b * TB, g.lc, lds + C::TILE_BYTES); };

    // the first block is asked for before it is known that some row sees it
    const bool asked = sp * TB < g.lc;
    if (asked) { fetch_k(sp); fetch_v(sp); }
    const Visible vis(g, row0, l32);
    const int n_blocks = (vis.n_all + TB - 1) / TB;
    if (n_blocks == 0 && a.accumulate) {                   // merging an empty partial is the identity
        wait_transfers<0>();
        return;
    }
    const LaneAddr<C> la(lane, lds);
    f32x16 oacc[C::NDB];
#pragma unroll
    for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
    const float c_log2 = g.scale * LOG2E, inv_c_log2 = 1.0f / c_log2;
    float m_run = NEG_BIG, thr_raw = NEG_BIG;
    float ps[4] = {0.f, 0.f, 0.f, 0.f}, psr[4] = {0.f, 0.f, 0.f, 0.f};      // partial sums of the exact and of the rounded probabilities

    // probabilities of block b, rounded to bf16 operand slots
    auto softmax = [&](f32x16& s, int b, bf16x8 (&pf)[2]) __attribute__((always_inline)) {
        if (b >= vis.n_full) {
            keep_branch();
            const int n = vis.mine - b * TB - 4 * hh;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) >= n) s[r] = -INFINITY;
        }
        float mx = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int r = 3; r < 15; r += 2) mx = max3(mx, s[r], s[r + 1]);
        mx = max_across_halves(max2(mx, s[15]));
        if (b == sp) {                                     // nothing to rescale yet
            m_run = fmaxf(NEG_BIG, mx * c_log2);
            thr_raw = (m_run + RESCALE_SLACK) * inv_c_log2;
        } else if (__any(mx > thr_raw)) {                  // running maximum, raised only when a block exceeds it by more than 2^8
            const float m_new = fmaxf(m_run, mx * c_log2);
            const float alpha = fast_exp2(m_run - m_new);
#pragma unroll
            for (int i = 0; i < 4; ++i) { ps[i] *= alpha; psr[i] *= alpha; }
#pragma unroll
            for (int db = 0; db < C::NDB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
            m_run = m_new;
            thr_raw = (m_run + RESCALE_SLACK) * inv_c_log2;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) { p[e] = fast_exp2(fmaf(s[8 * u + e], c_log2, -m_run)); ps[e & 3] += p[e]; }
            pf[u] = pack_bf16x8_sum4(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7], psr);
        }
    };

    if (asked) wait_transfers<2 * C::XFERS>();             // Q has landed
    else wait_transfers<0>();
    block_barrier();
    bf16x8 qf[C::NKS];
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) qf[ks] = lds_b128(la.row[ks] - lds + lds_q);
    for (int b = sp; b < n_blocks; b += NW) {
        const bool more = b + NW < n_blocks;
        wait_transfers<C::XFERS>();                        // K has landed, V may still be in flight
        f32x16 s = row_product<C>(la, 0, [&](int ks) { return qf[ks]; });
        reads_done();
        if (more) fetch_k(b + NW);
        bf16x8 pf[2];
        softmax(s, b, pf);
        if (more) wait_transfers<C::XFERS>();
        else wait_transfers<0>();
        col_product<C>(oacc, la, C::TILE_BYTES, pf);
        reads_done();
        if (more) fetch_v(b + NW);
    }

    // Combine the splits: every wavefront weighs its own partial result, merged with the running (o, lse), then one
    // row-contiguous pass adds them up.  The running values are asked for first (rows past the end read the last one).
    wait_transfers<0>();                                   // (a first block that no row sees)
    f32x4 o_old[C::OUT_VECS];
    float lse_old = -INFINITY;
    if (a.accumulate) {
        lse_old = a.lse[(long long)h * g.lq + (row0 + l32 < g.lq ? row0 + l32 : g.lq - 1)];
#pragma unroll
        for (int j = 0; j < C::OUT_VECS; ++j) {
            const int i = tid + 64 * NW * j, r = row0 + i / (D / 4), c = 4 * (i % (D / 4));
            o_old[j] = *reinterpret_cast<const f32x4*>(a.o + ((long long)(r < g.lq ? r : g.lq - 1) * g.nq + h) * D + c);
        }
    } else {
#pragma unroll
        for (int j = 0; j < C::OUT_VECS; ++j) o_old[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const float l_run = sum_across_halves((ps[0] + ps[1]) + (ps[2] + ps[3]));
    const float lr_run = sum_across_halves((psr[0] + psr[1]) + (psr[2] + psr[3]));
    if (hh == 0) stat[sp][l32] = make_float4(m_run, l_run, lr_run, 0.f);
    __syncthreads();                                       // every wavefront is done with its blocks
    float m = NEG_BIG, l = 0.f, lr = 0.f;
    float4 x[NW];
#pragma unroll
    for (int s = 0; s < NW; ++s) { x[s] = stat[s][l32]; m = fmaxf(m, x[s].x); }
#pragma unroll
    for (int s = 0; s < NW; ++s) {
        const float e = fast_exp2(x[s].x - m);
        l += e * x[s].y;
        lr += e * x[s].z;
    }
    float inv = 0.f, lse_new = -INFINITY, wa = 0.f;
    if (l > 0.f) {
        inv = lr > 0.f ? 1.0f / lr : 0.f;
        lse_new = (m + __log2f(l)) * LN2;
    }
    float wb = inv;
    if (a.accumulate) {
        const float mm = fmaxf(lse_old, lse_new);
        if (mm != -INFINITY) {
            const float ea = __expf(lse_old - mm), eb = __expf(lse_new - mm);
            const float r = 1.0f / (ea + eb);
            wa = ea * r;
            wb = eb * r * inv;
            lse_new = mm + __logf(ea + eb);
        }
    }
    if (sp == 0 && hh == 0) {
        sm.e.wa[l32] = wa;
        if (row0 + l32 < g.lq) a.lse[(long long)h * g.lq + row0 + l32] = lse_new;
    }
    stage_transposed<C>(&sm.e.stage[sp * TB * C::PITCH], oacc, l32, hh, wb * fast_exp2(m_run - m));
    __syncthreads();
#pragma unroll
    for (int j = 0; j < C::OUT_VECS; ++j) {
        const int i = tid + 64 * NW * j, r = i / (D / 4), c = 4 * (i % (D / 4));
        const f32x4 out = sm.e.wa[r] * o_old[j] + staged_sum<C>(sm.e.stage, r, c);
        if (row0 + r < g.lq) *reinterpret_cast<f32x4*>(a.o + ((long long)(row0 + r) * g.nq + h) * D + c) = out;
    }
}

// dQ: dP^T = V dO^T, S^T = K Q^T, dS^T = P^T (dP^T - Delta), dQ^T += K^T dS^T.
template <class C> union DqSmem {
    struct { unsigned char t[NW][2 * C::TILE_BYTES], q[C::TILE_BYTES], g[C::TILE_BYTES]; } b;      // K and V block of each wavefront, the workgroup's rows
    float stage[C::STAGE_FLOATS];
};

template <int D>
__device__ __forceinline__ void dq_unit(const BwdArgs& a, const int h, const int q_tile, DqSmem<SplitCfg<D>>& sm)
{
    using C = SplitCfg<D>;
    const AttnGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int sp = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    const int row0 = q_tile * TB;
    const int kvh = arg_byte(g.kv_of_q, h);
    const int my_row_c = row0 + l32 < g.lq ? row0 + l32 : g.lq - 1;
    const uint16_t* k = static_cast<const uint16_t*>(a.k) + (long long)kvh * g.kv_stride_head;
    const uint16_t* v = static_cast<const uint16_t*>(a.v) + (long long)kvh * g.kv_stride_head;
    const uint32_t lds = (uint32_t)(uintptr_t)(&sm.b.t[0][0]) + sp * 2 * C::TILE_BYTES;
    const uint32_t lds_q = (uint32_t)(uintptr_t)(&sm.b.q[0]), lds_g = (uint32_t)(uintptr_t)(&sm.b.g[0]);
    fetch_rows<C, TB, NW>(static_cast<const uint16_t*>(a.d_o) + (long long)h * g.q_stride_head, g.q_stride_tok, row0, g.lq, lds_g, sp, lane);
    fetch_rows<C, TB, NW>(static_cast<const uint16_t*>(a.q) + (long long)h * g.q_stride_head, g.q_stride_tok, row0, g.lq, lds_q, sp, lane);
    const float lse = a.lse[(long long)h * g.lq + my_row_c];
    const float delta = a.delta[(long long)h * g.lq + my_row_c];
    const BlockFetch<C> fetch(lane, g.kv_stride_tok);
    auto fetch_k = [&](int b) { fetch.issue(k, g.kv_stride_tok, b * TB, g.lc, lds); };
    auto fetch_v = [&](int b) { fetch.issue(v, g.kv_stride_tok, b * TB, g.lc, lds + C::TILE_BYTES); };
    const bool asked = sp * TB < g.lc;
    if (asked) { fetch_v(sp); fetch_k(sp); }
    const Visible vis(g, row0, l32);
    const int n_blocks = (vis.n_all + TB - 1) / TB;
    if (n_blocks == 0) {                                   // dq_acc unchanged
        wait_transfers<0>();
        return;
    }
    const LaneAddr<C> la(lane, lds);
    const float c_log2 = g.scale * LOG2E;
    f32x16 dq[C::NDB];
#pragma unroll
    for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[db][r] = 0.f;
    if (asked) wait_transfers<2 * C::XFERS>();             // Q and dO have landed
    else wait_transfers<0>();
    const float neg_l = lse == -INFINITY ? -INFINITY : -lse * LOG2E;       // a row whose LSE is infinite has P = 0
    // No wait for these inside the loop.  (The compiler waits here for everything in flight, the first K and V included: it does not see
    // the transfers issued behind these two loads.)
    asm volatile("" ::"v"(neg_l), "v"(delta));
    block_barrier();
    bf16x8 qf[C::NKS], gf[C::NKS];
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) { gf[ks] = lds_b128(la.row[ks] - lds + lds_g); qf[ks] = lds_b128(la.row[ks] - lds + lds_q); }

    // dQ^T += K^T dS^T of block b
    auto accumulate = [&](const f32x16& s, const f32x16& dp, int b) __attribute__((always_inline)) {
        float ds[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) ds[r] = fast_exp2(fmaf(s[r], c_log2, neg_l)) * (dp[r] - delta);
        if (b >= vis.n_full) {
            keep_branch();
            const int n = vis.mine - b * TB - 4 * hh;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) >= n) ds[r] = 0.f;
        }
        bf16x8 hi[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) hi[u] = pack_bf16x8(ds[8 * u], ds[8 * u + 1], ds[8 * u + 2], ds[8 * u + 3], ds[8 * u + 4], ds[8 * u + 5], ds[8 * u + 6], ds[8 * u + 7]);
        col_product<C>(dq, la, 0, hi);
        // Blocks with some |bf16(dS)| >= 2 (bit 14 of the pattern) also add the residuals dS - bf16(dS), as two more bf16
        // operands: three bf16 hold 24 bits, so dS reaches the product unrounded (the large kernel adds them in fp32).
        uint32_t big = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const uint4 w = __builtin_bit_cast(uint4, hi[u]);
            big |= w.x | w.y | w.z | w.w;
        }
        if (__any((big & 0x40004000u) != 0u)) {
            bf16x8 part[2] = {hi[0], hi[1]};
#pragma unroll
            for (int n = 0; n < 2; ++n) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) ds[8 * u + e] -= (float)part[u][e];
                    part[u] = pack_bf16x8(ds[8 * u], ds[8 * u + 1], ds[8 * u + 2], ds[8 * u + 3], ds[8 * u + 4], ds[8 * u + 5], ds[8 * u + 6], ds[8 * u + 7]);
                }
                col_product<C>(dq, la, 0, part);
            }
        }
    };
    for (int b = sp; b < n_blocks; b += NW) {
        const bool more = b + NW < n_blocks;
        wait_transfers<C::XFERS>();                        // V has landed, K may still be in flight
        const f32x16 dp = row_product<C>(la, C::TILE_BYTES, [&](int ks) { return gf[ks]; });
        reads_done();
        wait_transfers<0>();
        if (more) fetch_v(b + NW);
        const f32x16 s = row_product<C>(la, 0, [&](int ks) { return qf[ks]; });
        accumulate(s, dp, b);
        reads_done();
        if (more) fetch_k(b + NW);
    }
    wait_transfers<0>();                                   // (a first block that no row sees)
    f32x4 old[C::OUT_VECS];
#pragma unroll
    for (int j = 0; j < C::OUT_VECS; ++j) {                // (rows past the end read the last one)
        const int i = tid + 64 * NW * j, r = row0 + i / (D / 4), c = 4 * (i % (D / 4));
        old[j] = *reinterpret_cast<const f32x4*>(a.dq + ((long long)(r < g.lq ? r : g.lq - 1) * g.nq + h) * D + c);
    }
    __syncthreads();
    stage_transposed<C>(&sm.stage[sp * TB * C::PITCH], dq, l32, hh, g.scale);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < C::OUT_VECS; ++j) {
        const int i = tid + 64 * NW * j, r = i / (D / 4), c = 4 * (i % (D / 4));
        old[j] += staged_sum<C>(sm.stage, r, c);
        if (row0 + r < g.lq) *reinterpret_cast<f32x4*>(a.dq + ((long long)(row0 + r) * g.nq + h) * D + c) = old[j];
    }
}

// dK / dV of 32 keys from the q rows of a run of heads: S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.  The keys'
// own K and V rows stay in LDS at D = 128 (dK and dV take 128 of a wavefront's 256 registers there).
template <class C> union DkdvSmem {
    struct {
        unsigned char t[NW][2 * C::TILE_BYTES];            // Q and dO block of each wavefront
        unsigned char kv[2 * C::TILE_BYTES];               // the workgroup's K and V rows
        float lse[NW][64], delta[NW][64];                  // row scalars of each wavefront's block (32 used; a transfer writes 64)
    } m;
    float stage[C::STAGE_FLOATS];
};

template <int D, bool ATOMIC_DKV>
__device__ __forceinline__ void dkdv_unit(const BwdArgs& a, const HeadRuns& runs, const int run, const int kv_tile, DkdvSmem<SplitCfg<D>>& sm)
{
    using C = SplitCfg<D>;
    const AttnGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    const int col0 = kv_tile * TB;
    const int n_heads = arg_byte(runs.len, run);
    const int kvh = arg_byte(g.kv_of_q, arg_byte(runs.first, run));
    const int my_col = col0 + l32;
    // the rows that see a key are a suffix of the shard: [my_first, lq); no row before row_first sees any of the keys,
    // all rows from row_full on see all of them
    const int first = rows_le(g.qs, pos_of_row(g.ks, my_col < g.lc ? my_col : g.lc - 1) - 1);
    const int my_first = my_col < g.lc ? first : 0x7fffffff;
    const int row_first = __builtin_amdgcn_readlane(first, 0);
    const int row_full = col0 + TB <= g.lc ? __builtin_amdgcn_readlane(first, TB - 1) : 0x7fffffff;
    const int blk0 = row_first / TB;
    const int n_all = row_first < g.lq ? (g.lq + TB - 1) / TB - blk0 : 0;      // blocks of one head

    const uint32_t lds_all = (uint32_t)(uintptr_t)(&sm.m.t[0][0]);
    const uint32_t lds = lds_all + wave * 2 * C::TILE_BYTES;
    const uint32_t lds_kv = (uint32_t)(uintptr_t)(&sm.m.kv[0]);
    const uint32_t lds_lse = (uint32_t)(uintptr_t)(&sm.m.lse[wave][0]), lds_delta = (uint32_t)(uintptr_t)(&sm.m.delta[wave][0]);
    const LaneAddr<C> la(lane, lds);
    const BlockFetch<C> fetch(lane, g.q_stride_tok);
    fetch_rows<C, TB, NW>(static_cast<const uint16_t*>(a.k) + (long long)kvh * g.kv_stride_head, g.kv_stride_tok, col0, g.lc, lds_kv, wave, lane);
    fetch_rows<C, TB, NW>(static_cast<const uint16_t*>(a.v) + (long long)kvh * g.kv_stride_head, g.kv_stride_tok, col0, g.lc, lds_kv + C::TILE_BYTES, wave, lane);
    uint32_t kv_row[C::NKS];
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) kv_row[ks] = la.row[ks] - lds + lds_kv;
    constexpr bool KV_REGS = D == 64;                      // the fragments of K and V fit the registers
    bf16x8 kf[KV_REGS ? C::NKS : 1], vf[KV_REGS ? C::NKS : 1];
    auto k_frag = [&](int ks) { if constexpr (KV_REGS) return kf[ks]; else return lds_b128(kv_row[ks]); };
    auto v_frag = [&](int ks) { if constexpr (KV_REGS) return vf[ks]; else return lds_b128(kv_row[ks] + C::TILE_BYTES); };

    f32x16 dk[C::NDB], dv[C::NDB];
#pragma unroll
    for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dk[db][r] = 0.f; dv[db][r] = 0.f; }
    const float scale_log2 = g.scale * LOG2E;

    // the workgroup's sequence of blocks: those of the first head of the run, then the next head's; this wavefront's
    // first one, and a step of NW
    int h = arg_byte(runs.first, run), t = wave, left = n_heads;
    auto normalise = [&]() { while (left > 0 && t >= n_all) { t -= n_all; h = arg_byte(runs.next, h); --left; } };
    if (n_all == 0) left = 0;
    normalise();
    auto fetch_g = [&](int hd, int row) {
        fetch.issue(static_cast<const uint16_t*>(a.d_o) + (long long)hd * g.q_stride_head, g.q_stride_tok, row, g.lq, lds + C::TILE_BYTES);
        const int r = row + l32 < g.lq ? row + l32 : g.lq - 1;
        lds_dma4(a.lse + (long long)hd * g.lq + r, __builtin_amdgcn_readfirstlane(lds_lse));
        lds_dma4(a.delta + (long long)hd * g.lq + r, __builtin_amdgcn_readfirstlane(lds_delta));
    };
    auto fetch_q = [&](int hd, int row) {
        fetch.issue(static_cast<const uint16_t*>(a.q) + (long long)hd * g.q_stride_head, g.q_stride_tok, row, g.lq, lds);
    };
    if (left > 0) { fetch_g(h, (blk0 + t) * TB); fetch_q(h, (blk0 + t) * TB); }
    // K / V were requested first: whatever is in flight behind them is this wavefront's first block
    if (left > 0) wait_transfers<2 * C::XFERS + 2>();
    else wait_transfers<0>();
    block_barrier();
    if constexpr (KV_REGS) {
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) { kf[ks] = lds_b128(kv_row[ks]); vf[ks] = lds_b128(kv_row[ks] + C::TILE_BYTES); }
    }
    while (left > 0) {
        const int row = (blk0 + t) * TB;
        t += NW;
        normalise();
        const bool more = left > 0;
        const int next_row = (blk0 + t) * TB;
        wait_transfers<C::XFERS>();                    // dO, LSE and Delta have landed, Q may still be in flight
        const f32x16 dp = row_product<C>(la, C::TILE_BYTES, v_frag);
        wait_transfers<0>();
        const f32x16 s = row_product<C>(la, 0, k_frag);
        const bool masked = row < row_full || row + TB > g.lq;
        bf16x8 pf[2], df[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float p[8], ds[8];
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                const int r0 = 16 * u + 8 * rb + 4 * hh;
                const f32x4 l4 = *reinterpret_cast<const f32x4*>(&sm.m.lse[wave][r0]);
                const f32x4 d4 = *reinterpret_cast<const f32x4*>(&sm.m.delta[wave][r0]);
#pragma unroll
                for (int e = 0; e < 4; ++e) p[4 * rb + e] = fast_exp2(fmaf(s[8 * u + 4 * rb + e], scale_log2, l4[e] * -LOG2E));
                if (masked) {      // (a row that sees nothing anywhere, LSE = -inf, is masked in every block)
                    keep_branch();
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (row + r0 + e < my_first || row + r0 + e >= g.lq) p[4 * rb + e] = 0.f;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) ds[4 * rb + e] = p[4 * rb + e] * (dp[8 * u + 4 * rb + e] - d4[e]);
            }
            pf[u] = pack_bf16x8(p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7]);
            df[u] = pack_bf16x8(ds[0], ds[1], ds[2], ds[3], ds[4], ds[5], ds[6], ds[7]);
        }
        col_product<C>(dv, la, C::TILE_BYTES, pf);
        reads_done();
        if (more) fetch_g(h, next_row);
        col_product<C>(dk, la, 0, df);
        reads_done();
        if (more) fetch_q(h, next_row);
    }

    auto write_out = [&](float* out, const f32x16 (&acc)[C::NDB], float w) {
        __syncthreads();
        stage_transposed<C>(&sm.stage[wave * TB * C::PITCH], acc, l32, hh, w);
        __syncthreads();
        if (ATOMIC_DKV) {          // consecutive lanes on consecutive floats
#pragma unroll
            for (int j = 0; j < 4 * C::OUT_VECS; ++j) {
                const int i = tid + 64 * NW * j, r = i / D, c = i % D;
                float x = sm.stage[r * C::PITCH + c];
#pragma unroll
                for (int s = 1; s < NW; ++s) x += sm.stage[(s * TB + r) * C::PITCH + c];
                if (col0 + r < g.lc) global_atomic_add(out + ((long long)(col0 + r) * g.nkv + kvh) * D + c, x);
            }
        } else {
#pragma unroll
            for (int j = 0; j < C::OUT_VECS; ++j) {
                const int i = tid + 64 * NW * j, r = i / (D / 4), c = 4 * (i % (D / 4));
                f32x4 x = staged_sum<C>(sm.stage, r, c);
                if (col0 + r >= g.lc) continue;
                f32x4* op = reinterpret_cast<f32x4*>(out + ((long long)(col0 + r) * g.nkv + kvh) * D + c);
                if (a.accumulate) x += *op;
                *op = x;
            }
        }
    };
    write_out(a.dv, dv, 1.0f);
    write_out(a.dk, dk, g.scale);
}

// One launch for both halves of a backward step: workgroups [0, n_dkdv) are dK / dV units (the longer ones, first), the
// others dQ units.  Within each, heads (runs) side by side and the longest tiles first.
template <int D, bool ATOMIC_DKV>
__global__ void __launch_bounds__(512) bwd_split_bf16_kernel(const BwdArgs a, const HeadRuns runs, const unsigned n_dkdv, const int n_q_tiles)
{
    __shared__ __attribute__((aligned(1024))) union { DkdvSmem<SplitCfg<D>> dkdv; DqSmem<SplitCfg<D>> dq; } sm;
    if (blockIdx.x < n_dkdv) {
        const int tile = uniform((int)(blockIdx.x / (unsigned)runs.n));
        dkdv_unit<D, ATOMIC_DKV>(a, runs, (int)blockIdx.x - tile * runs.n, tile, sm.dkdv);
    } else {
        const unsigned unit = blockIdx.x - n_dkdv;
        const int tile = uniform((int)(unit / (unsigned)a.g.nq));
        dq_unit<D>(a, (int)unit - tile * a.g.nq, n_q_tiles - 1 - tile, sm.dq);
    }
}

}  // namespace

hipError_t hexi_launch_fwd_split_bf16(const FwdArgs& a, hipStream_t s)
{
    const int n_q_tiles = (a.g.lq + TB - 1) / TB;
    const dim3 grid((unsigned)a.g.nq, (unsigned)n_q_tiles);
    if (a.g.d == 128) fwd_split_bf16_kernel<128><<<grid, 512, 0, s>>>(a, n_q_tiles);
    else if (a.g.d == 64) fwd_split_bf16_kernel<64><<<grid, 512, 0, s>>>(a, n_q_tiles);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// dq: with the dQ workgroups; runs: the head runs of the dK / dV workgroups (none: no dK / dV)
hipError_t hexi_launch_bwd_split_bf16(const BwdArgs& a, bool dq, const HeadRuns& runs, bool shared, hipStream_t s)
{
    const int n_q_tiles = dq ? (a.g.lq + TB - 1) / TB : 0;
    // (to keys that no row sees runs would add zeros: 1252 rows x 9572 keys x 8 / 2 heads x 128 in runs of two heads 55 -> 31 us)
    const int n_keys = shared ? hexi_keys_seen(a.g) : a.g.lc;
    const unsigned n_dkdv = (unsigned)((n_keys + TB - 1) / TB) * (unsigned)runs.n;
    const unsigned grid = n_dkdv + (unsigned)n_q_tiles * (unsigned)a.g.nq;
    if (grid == 0) return hipSuccess;
    if (a.g.d == 128) {
        if (shared) bwd_split_bf16_kernel<128, true><<<grid, 512, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
        else bwd_split_bf16_kernel<128, false><<<grid, 512, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
    } else if (a.g.d == 64) {
        if (shared) bwd_split_bf16_kernel<64, true><<<grid, 512, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
        else bwd_split_bf16_kernel<64, false><<<grid, 512, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
    } else return hipErrorInvalidValue;
    return hipGetLastError();
}

// bf16 ring step (forward, dQ, dK/dV) for launches between the smallest (hexi_bf16_split.hip) and those that fill the chip with
// 256-row / 128-key workgroups: a workgroup of four wavefronts, one per SIMD, owns 64 stationary rows, and the wavefronts split the
// streamed rows between them, 32 at a time (block b goes to wavefront b % 4), through private double buffers and without a barrier
// before the end, where the partial results are combined through LDS in a fixed order.
//
// Why this shape.  A wavefront has a SIMD's 512 registers: 64 stationary rows are two independent chains of MFMAs, and every operand
// fragment that it reads from LDS serves both.  Streaming 64 KB per step, a CU's 64 bytes a clock are half the time of its MFMAs
// (with 32 stationary rows per CU twice as much).  Nobody shares a block, so nobody waits for anyone: with two wavefronts to a block
// and a barrier per step, as the 64-row forward and dQ workgroups had before, the two wavefronts of a SIMD ran their MFMAs at the same time
// and their vector work at the same time.  Here the MFMAs, the vector work, the LDS reads and the transfers of one wavefront are laid
// out in one sequence: the scores of the next block beside the probabilities of this one (forward), the second half of a product
// beside the P and dS of the first (backward), the transfers of the block after the next one by one behind MFMAs, scalar work and the
// first fragments of the next block behind the last ones.
// What bounds it: MFMAs are 1024 of 1860 clocks of a forward step, 1536 of 2420 (dQ), 2048 of 3420 (dK / dV; head_dim 128, counted); the
// rest is vector work that does not fit beside them (about 600), transfers (about 300) and the waits at a step's ends; short chains
// add 2.5 to 3.5 us to start and 2 to 4 to finish.  Where the chip is full it is power (1.6 to 1.8 GHz), and the large workgroups, which move
// less through LDS per MFMA, are the better choice.  Measured, us per call, the smaller of the 64-row split and the 256-row workgroups
// before -> these, head_dim 128, fully visible chunk: forward 512 rows x 1024 keys, 24 / 8 heads 17.7 -> 15.7, 4096 x 4096 x 24 / 8 x 64
// 138 -> 130; backward 512 x 1024 x 24 / 8 41 -> 35, 2048 x 2048 x 24 / 8 207 -> 178, 4096 x 4096 x 12 / 3 384 -> 336, 4096 x 4096 x
// 24 / 8 x 64 445 -> 384.
//
// Operand layouts as in hexi_bf16_split.hip; dK and dV are accumulated transposed too (the keys across the lanes).
#include "hexi_blocks.h"

namespace {

constexpr int NW = 4;          // wavefronts per workgroup = splits of the streamed rows
constexpr int ROWS = 64;       // stationary rows per workgroup (every wavefront has all of them)

template <int D_> struct QuadCfg : BlockCfg<D_> {
    using B = BlockCfg<D_>;
    static constexpr int NBUF = 2;                         // buffers per wavefront
    static constexpr int STAGE_FLOATS = NW * ROWS * B::PITCH;
    static constexpr int OUT_VECS = ROWS * D_ / 4 / (64 * NW);      // float4 of the output per thread
};

// What 64 rows see of the chunk.
struct Visible64 {
    int mine[2];    // keys that the lane's rows l32 and 32 + l32 see (0 for padding rows)
    int n_all;      // keys some row sees
    int n_full;     // 32-key blocks every row sees in full
    __device__ __forceinline__ Visible64(const AttnGeom& g, int row0, int lane, int l32)
    {
        const int row = row0 + lane < g.lq ? row0 + lane : g.lq - 1;
        const int n = rows_le(g.ks, pos_of_row(g.qs, row));
        n_all = __builtin_amdgcn_readlane(n, 63);
        n_full = __builtin_amdgcn_readlane(n, 0) / TB;
        const int seen = row0 + lane < g.lq ? n : 0;
        mine[0] = __shfl(seen, l32, 64);
        mine[1] = __shfl(seen, 32 + l32, 64);
    }
};

__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    const bf16x2 t = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, t);
}
__device__ __forceinline__ float add_rounded(uint32_t p, float sum)
{
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), ones, sum, false);
}

template <int D>
__global__ void __launch_bounds__(256, D == 64 ? 2 : 1) fwd_quad_bf16_kernel(const FwdArgs a, const QuadRest rest)
{
    using C = QuadCfg<D>;
    const AttnGeom& g = a.g;
    __shared__ __attribute__((aligned(1024))) union {
        unsigned char t[NW][C::NBUF][2 * C::TILE_BYTES];   // K and V block of each wavefront
        struct { float stage[C::STAGE_FLOATS], wa[ROWS]; } e;
    } sm;
    __shared__ float4 stat[NW][ROWS];                      // reference, exact sum, sum of the rounded probabilities of each split
    const int tid = threadIdx.x, lane = tid & 63;
    const int sp = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;

    // heads of a q tile side by side, the longest (last) q tiles first
    const int h = blockIdx.x;
    const int q_tile = rest.tiles - 1 - (int)blockIdx.y;
    if (!rest.has(h, q_tile)) return;
    const int row0 = q_tile * ROWS;
    const int kvh = arg_byte(g.kv_of_q, h);
    const uint16_t* k = static_cast<const uint16_t*>(a.k) + (long long)kvh * g.kv_stride_head;
    const uint16_t* v = static_cast<const uint16_t*>(a.v) + (long long)kvh * g.kv_stride_head;
    const uint32_t lds = (uint32_t)(uintptr_t)(&sm.t[0][0][0]) + sp * C::NBUF * 2 * C::TILE_BYTES;
    const BlockFetch<C> fetch(lane, g.kv_stride_tok);
    auto fetch_k = [&](int b, int buf) { fetch.issue(k, g.kv_stride_tok, b * TB, g.lc, lds + buf * 2 * C::TILE_BYTES); };
    auto fetch_v = [&](int b, int buf) { fetch.issue(v, g.kv_stride_tok, b * TB, g.lc, lds + buf * 2 * C::TILE_BYTES + C::TILE_BYTES); };

    // What the first scores need is asked for first (K before it is known that some row sees it); everything else is issued beside
    // their MFMAs.  Q comes by way of the second buffer of wavefront 0.
    const uint32_t lds_q = (uint32_t)(uintptr_t)(&sm.t[0][1][0]);
    fetch_rows<C, ROWS, NW>(static_cast<const uint16_t*>(a.q) + (long long)h * g.q_stride_head, g.q_stride_tok, row0, g.lq, lds_q, sp, lane);
    if (sp * TB < g.lc) fetch_k(sp, 0);
    const Visible64 vis(g, row0, lane, l32);
    const int n_blocks = (vis.n_all + TB - 1) / TB;
    if (n_blocks == 0 && a.accumulate) {                   // merging an empty partial is the identity
        wait_transfers<0>();
        return;
    }
    const LaneAddr<C> la(lane, lds);
    f32x16 oacc[2][C::NDB];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int db = 0; db < C::NDB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[r][db][i] = 0.f;
    const float c_log2 = g.scale * LOG2E, inv_c_log2 = 1.0f / c_log2;
    wait_transfers<0>();
    block_barrier();
    bf16x8 qf[2][C::NKS];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) qf[r][ks] = lds_b128(la.row[ks] - lds + lds_q + r * C::TILE_BYTES);
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            if constexpr (D == 128) asm volatile("" : "+a"(qf[r][ks]));
            else pin(qf[r][ks]);
        }
    reads_done();
    block_barrier();                                          // the second buffers are free
    float m_run[2] = {NEG_BIG, NEG_BIG}, thr_raw[2];
    float ps[2][2] = {{0.f, 0.f}, {0.f, 0.f}}, psr[2][2] = {{0.f, 0.f}, {0.f, 0.f}};      // partial sums of the exact and of the rounded probabilities
    uint32_t pw[2][8];                                     // probabilities, two to a word, in operand order

    // two probabilities of row block r: scores 2 i, 2 i + 1
    auto prob2 = [&](const f32x16 (&s)[2], int c) __attribute__((always_inline)) {
        const int r = c >> 3, i = c & 7;
        const float p0 = fast_exp2(fmaf(s[r][2 * i], c_log2, -m_run[r])), p1 = fast_exp2(fmaf(s[r][2 * i + 1], c_log2, -m_run[r]));
        ps[r][0] += p0;
        ps[r][1] += p1;
        pw[r][i] = pack2(p0, p1);
        psr[r][i & 1] = add_rounded(pw[r][i], psr[r][i & 1]);
        asm volatile("" : "+v"(pw[r][i]), "+v"(ps[r][0]), "+v"(ps[r][1]), "+v"(psr[r][i & 1]));     // stays where it stands
    };
    auto p_frag = [&](int r, int u) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, make_uint4(pw[r][4 * u], pw[r][4 * u + 1], pw[r][4 * u + 2], pw[r][4 * u + 3]));
    };
    auto block_max = [&](const f32x16& s) __attribute__((always_inline)) {
        float mx = max3(s[0], s[1], s[2]);
#pragma unroll
        for (int i = 3; i < 15; i += 2) mx = max3(mx, s[i], s[i + 1]);
        return max_across_halves(max2(mx, s[15]));
    };

    // scores of the block at byte `tile`, two MFMAs per K fragment; first() once the first fragments are on their way, between(i)
    // after MFMA i
    auto scores = [&](f32x16 (&out)[2], uint32_t tile, auto&& first, auto&& between) __attribute__((always_inline)) {
        bf16x8 x[4];
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) x[ks] = lds_b128(la.row[ks] + tile);
        __builtin_amdgcn_sched_barrier(0);
        first();
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            if (ks + 3 < C::NKS) x[(ks + 3) & 3] = lds_b128(la.row[ks + 3] + tile);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                out[r] = mfma32(x[ks & 3], qf[r][ks], ks == 0 ? zero : out[r]);
                __builtin_amdgcn_sched_barrier(0);
                between(2 * ks + r);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    auto mask = [&](f32x16 (&s)[2], int b) __attribute__((always_inline)) {
        if (b < vis.n_full) return;
        keep_branch();
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int n = vis.mine[r] - b * TB - 4 * hh;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (8 * (i >> 2) + (i & 3) >= n) s[r][i] = -INFINITY;
        }
    };
    // One block: s its scores, masked and with a reference in m_run; sn receives those of the wavefront's next block.  Its
    // probabilities are formed beside the next block's scores and the second product of the first row block, the next block's
    // maximum beside that of the second.  STEADY: there is a next block, and a whole one after it whose transfers go between the MFMAs too.
    auto step = [&](auto bufc, auto steadyc, f32x16 (&s)[2], f32x16 (&sn)[2], int b) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value;
        constexpr bool STEADY = decltype(steadyc)::value;
        constexpr uint32_t here = buf * 2 * C::TILE_BYTES, there = (buf ^ 1) * 2 * C::TILE_BYTES;
        constexpr int N = C::NDB * 2, SLOTS = 2 * C::NKS;  // MFMAs of a row block in the second product, of both in the scores
        constexpr int LEAD = 4, EARLY = 12;                // pairs of probabilities before the first MFMA, before the second product
        const bool next = STEADY || b + NW < n_blocks, next2 = STEADY || b + 2 * NW < n_blocks;
        const int b2 = b + 2 * NW;
        const uint16_t *k2 = k + (long long)(b2 * TB) * g.kv_stride_tok, *v2 = v + (long long)(b2 * TB) * g.kv_stride_tok;
        bf16x8 x[N];
        auto read = [&](int st) __attribute__((always_inline)) {
            const uint32_t o = here + C::TILE_BYTES + st / C::NDB * 16 * C::ROW_BYTES;
            x[st] = lds_tr(la.tr[0][st % C::NDB] + o, la.tr[1][st % C::NDB] + o);
        };
        if (next) {
            wait_transfers<C::XFERS>();                    // K of the next block has landed, and so has V of this one
            scores(sn, there, [&]() __attribute__((always_inline)) {
                if (!STEADY && next2) fetch_k(b2, buf);    // (K of this buffer went into the scores one step ago)
#pragma unroll
                for (int c = 0; c < LEAD; ++c) prob2(s, c);
            }, [&](int st) __attribute__((always_inline)) {
                for (int c = LEAD + st * (EARLY - LEAD) / SLOTS; c < LEAD + (st + 1) * (EARLY - LEAD) / SLOTS; ++c) prob2(s, c);
                if (STEADY && st % 2 == 0) fetch.one(k2, g.kv_stride_tok, lds + here, st / 2);
                if (st >= SLOTS - N) read(st - (SLOTS - N));
            });
            mask(sn, b + NW);
        } else {
            wait_transfers<0>();
            asm volatile("" : "+v"(m_run[0]), "+v"(m_run[1]));     // (or these would be computed before the branch)
#pragma unroll
            for (int st = 0; st < N; ++st) read(st);
#pragma unroll
            for (int c = 0; c < EARLY; ++c) prob2(s, c);
        }
#pragma unroll
        for (int st = 0; st < N; ++st) {
            oacc[0][st % C::NDB] = mfma32(x[st], p_frag(0, st / C::NDB), oacc[0][st % C::NDB]);
            __builtin_amdgcn_sched_barrier(0);
            for (int c = EARLY + st * (16 - EARLY) / N; c < EARLY + (st + 1) * (16 - EARLY) / N; ++c) prob2(s, c);
            __builtin_amdgcn_sched_barrier(0);
        }
        reads_done();
        if (!STEADY && next2) fetch_v(b2, buf);
        float mx[2] = {sn[0][0], sn[1][0]};
#pragma unroll
        for (int st = 0; st < N; ++st) {
            oacc[1][st % C::NDB] = mfma32(x[st], p_frag(1, st / C::NDB), oacc[1][st % C::NDB]);
            __builtin_amdgcn_sched_barrier(0);
            if (STEADY) fetch.one(v2, g.kv_stride_tok, lds + here + C::TILE_BYTES, st);
#pragma unroll
            for (int i = st * 16 / N; i < (st + 1) * 16 / N; i += 2)
#pragma unroll
                for (int r = 0; r < 2; ++r) mx[r] = max3(mx[r], sn[r][i], sn[r][i + 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!next) return;
        // running maximum, raised only when a block exceeds it by more than 2^8
        mx[0] = max_across_halves(mx[0]);
        mx[1] = max_across_halves(mx[1]);
        if (__any(mx[0] > thr_raw[0] || mx[1] > thr_raw[1])) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const float m_new = fmaxf(m_run[r], mx[r] * c_log2);
                const float alpha = fast_exp2(m_run[r] - m_new);
#pragma unroll
                for (int i = 0; i < 2; ++i) { ps[r][i] *= alpha; psr[r][i] *= alpha; }
#pragma unroll
                for (int db = 0; db < C::NDB; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[r][db][i] *= alpha;
                m_run[r] = m_new;
                thr_raw[r] = (m_run[r] + RESCALE_SLACK) * inv_c_log2;
            }
        }
    };

    f32x16 s0[2], s1[2];
    if (sp < n_blocks) {
        const int n_whole = n_blocks < g.lc / TB ? n_blocks : g.lc / TB;
        if (sp + NW < n_whole) {
            const uint16_t *v0 = v + (long long)(sp * TB) * g.kv_stride_tok, *k1 = k + (long long)((sp + NW) * TB) * g.kv_stride_tok;
            scores(s0, 0, []() {}, [&](int st) __attribute__((always_inline)) {
                if (st < C::XFERS) fetch.one(v0, g.kv_stride_tok, lds + C::TILE_BYTES, st);
                else fetch.one(k1, g.kv_stride_tok, lds + 2 * C::TILE_BYTES, st - C::XFERS);
            });
        } else {
            fetch_v(sp, 0);
            if (sp + NW < n_blocks) fetch_k(sp + NW, 1);
            scores(s0, 0, []() {}, [](int) {});
        }
        if (sp + NW < n_blocks) fetch_v(sp + NW, 1);
        mask(s0, sp);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            m_run[r] = fmaxf(NEG_BIG, block_max(s0[r]) * c_log2);
            thr_raw[r] = (m_run[r] + RESCALE_SLACK) * inv_c_log2;
        }
        // two blocks at a time: the buffer is a compile-time offset of the reads
        using Steady = std::true_type; using Last = std::false_type;
        int b = sp;
        for (; b + 3 * NW < n_whole; b += 2 * NW) {
            step(IC<0>{}, Steady{}, s0, s1, b);
            step(IC<1>{}, Steady{}, s1, s0, b + NW);
        }
        for (; b < n_blocks; b += 2 * NW) {
            step(IC<0>{}, Last{}, s0, s1, b);
            if (b + NW < n_blocks) step(IC<1>{}, Last{}, s1, s0, b + NW);
        }
    }

    // Combine the splits: every wavefront weighs its own partial result, merged with the running (o, lse), then one
    // row-contiguous pass adds them up.
    // The running values are asked for first (rows past the end read the last one).
    wait_transfers<0>();                                   // (a first block that no row sees)
    f32x4 o_old[C::OUT_VECS];
    float lse_old[2] = {-INFINITY, -INFINITY};
    if (a.accumulate) {
#pragma unroll
        for (int r = 0; r < 2; ++r) lse_old[r] = a.lse[(long long)h * g.lq + (row0 + 32 * r + l32 < g.lq ? row0 + 32 * r + l32 : g.lq - 1)];
#pragma unroll
        for (int j = 0; j < C::OUT_VECS; ++j) {
            const int i = tid + 64 * NW * j, r = row0 + i / (D / 4), c = 4 * (i % (D / 4));
            o_old[j] = *reinterpret_cast<const f32x4*>(a.o + ((long long)(r < g.lq ? r : g.lq - 1) * g.nq + h) * D + c);
        }
    } else {
#pragma unroll
        for (int j = 0; j < C::OUT_VECS; ++j) o_old[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float l_run[2], lr_run[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        l_run[r] = sum_across_halves(ps[r][0] + ps[r][1]);
        lr_run[r] = sum_across_halves(psr[r][0] + psr[r][1]);
        if (hh == 0) stat[sp][32 * r + l32] = make_float4(m_run[r], l_run[r], lr_run[r], 0.f);
    }
    __syncthreads();                                       // every wavefront is done with its blocks
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        float m = NEG_BIG, l = 0.f, lr = 0.f;
        float4 x[NW];
#pragma unroll
        for (int s = 0; s < NW; ++s) { x[s] = stat[s][32 * r + l32]; m = fmaxf(m, x[s].x); }
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
            const float mm = fmaxf(lse_old[r], lse_new);
            if (mm != -INFINITY) {
                const float ea = __expf(lse_old[r] - mm), eb = __expf(lse_new - mm);
                const float q = 1.0f / (ea + eb);
                wa = ea * q;
                wb = eb * q * inv;
                lse_new = mm + __logf(ea + eb);
            }
        }
        if (sp == 0 && hh == 0) {
            sm.e.wa[32 * r + l32] = wa;
            if (row0 + 32 * r + l32 < g.lq) a.lse[(long long)h * g.lq + row0 + 32 * r + l32] = lse_new;
        }
        const float w = wb * fast_exp2(m_run[r] - m);
        float* stage = &sm.e.stage[(sp * ROWS + 32 * r) * C::PITCH];
#pragma unroll
        for (int db = 0; db < C::NDB; ++db)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                *reinterpret_cast<float4*>(&stage[l32 * C::PITCH + 32 * db + 8 * b + 4 * hh]) =
                    make_float4(oacc[r][db][4 * b] * w, oacc[r][db][4 * b + 1] * w, oacc[r][db][4 * b + 2] * w, oacc[r][db][4 * b + 3] * w);
    }
    __syncthreads();
    f32x4 out[C::OUT_VECS];
#pragma unroll
    for (int j = 0; j < C::OUT_VECS; ++j) {
        const int i = tid + 64 * NW * j, r = i / (D / 4), c = 4 * (i % (D / 4));
        out[j] = sm.e.wa[r] * o_old[j];
#pragma unroll
        for (int s = 0; s < NW; ++s) out[j] += *reinterpret_cast<const f32x4*>(&sm.e.stage[(s * ROWS + r) * C::PITCH + c]);
    }
#pragma unroll
    for (int j = 0; j < C::OUT_VECS; ++j) {
        const int i = tid + 64 * NW * j, r = i / (D / 4), c = 4 * (i % (D / 4));
        if (row0 + r < g.lq) *reinterpret_cast<f32x4*>(a.o + ((long long)(row0 + r) * g.nq + h) * D + c) = out[j];
    }
}

// acc += x y with acc in accumulation registers, where the backward units keep what they sum over the whole sequence: the vector
// registers are for the scores.  (The compiler, left to choose, moves accumulators between the two kinds in the loop.)  It does not
// see that this is an MFMA: the wait states behind a vector instruction that wrote an operand are part of the statement, and
// acc_settled() comes before anything but another such product reads acc.
__device__ __forceinline__ void mfma_acc(f32x16& acc, const bf16x8& x, const bf16x8& y)
{
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(x), "v"(y));
}
template <int NDB> __device__ __forceinline__ void acc_settled(f32x16 (&acc)[2][NDB])
{
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int db = 0; db < NDB; ++db) asm volatile("" : "+a"(acc[r][db]));
}

// A partial result of every wavefront (transposed accumulators: lane = stationary row), times w, into the staging area.
template <class C> __device__ __forceinline__ void stage64(float* stage, const f32x16 (&acc)[2][C::NDB], int sp, int l32, int hh, float w)
{
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int db = 0; db < C::NDB; ++db)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                *reinterpret_cast<float4*>(&stage[(sp * ROWS + 32 * r + l32) * C::PITCH + 32 * db + 8 * b + 4 * hh]) =
                    make_float4(acc[r][db][4 * b] * w, acc[r][db][4 * b + 1] * w, acc[r][db][4 * b + 2] * w, acc[r][db][4 * b + 3] * w);
}
template <class C> __device__ __forceinline__ f32x4 staged_sum(const float* stage, int r, int c)
{
    f32x4 x = *reinterpret_cast<const f32x4*>(&stage[r * C::PITCH + c]);
#pragma unroll
    for (int s = 1; s < NW; ++s) x += *reinterpret_cast<const f32x4*>(&stage[(s * ROWS + r) * C::PITCH + c]);
    return x;
}

// dQ: S^T = K Q^T, dP^T = V dO^T, dS^T = P^T (dP^T - Delta), dQ^T += K^T dS^T.
template <class C> union QuadDqSmem {
    unsigned char t[NW][C::NBUF][2 * C::TILE_BYTES];       // K and V block of each wavefront
    float stage[C::STAGE_FLOATS];
};

template <int D>
__device__ __forceinline__ void dq_unit(const BwdArgs& a, const int h, const int q_tile, QuadDqSmem<QuadCfg<D>>& sm)
{
    using C = QuadCfg<D>;
    const AttnGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int sp = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    const int row0 = q_tile * ROWS;
    const int kvh = arg_byte(g.kv_of_q, h);
    const uint16_t* k = static_cast<const uint16_t*>(a.k) + (long long)kvh * g.kv_stride_head;
    const uint16_t* v = static_cast<const uint16_t*>(a.v) + (long long)kvh * g.kv_stride_head;
    const uint32_t lds_all = (uint32_t)(uintptr_t)(&sm.t[0][0][0]);
    const uint32_t lds = lds_all + sp * C::NBUF * 2 * C::TILE_BYTES;
    // the unit's own rows, by way of the second buffers of wavefronts 0 (Q) and 1 (dO)
    const uint32_t lds_q = lds_all + 2 * C::TILE_BYTES, lds_g = lds_q + C::NBUF * 2 * C::TILE_BYTES;
    fetch_rows<C, ROWS, NW>(static_cast<const uint16_t*>(a.q) + (long long)h * g.q_stride_head, g.q_stride_tok, row0, g.lq, lds_q, sp, lane);
    fetch_rows<C, ROWS, NW>(static_cast<const uint16_t*>(a.d_o) + (long long)h * g.q_stride_head, g.q_stride_tok, row0, g.lq, lds_g, sp, lane);
    float neg_l[2], delta[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int row = row0 + 32 * r + l32 < g.lq ? row0 + 32 * r + l32 : g.lq - 1;
        neg_l[r] = a.lse[(long long)h * g.lq + row];
        delta[r] = a.delta[(long long)h * g.lq + row];
    }
    const BlockFetch<C> fetch(lane, g.kv_stride_tok);
    auto fetch_k = [&](int b, int buf) { fetch.issue(k, g.kv_stride_tok, b * TB, g.lc, lds + buf * 2 * C::TILE_BYTES); };
    auto fetch_v = [&](int b, int buf) { fetch.issue(v, g.kv_stride_tok, b * TB, g.lc, lds + buf * 2 * C::TILE_BYTES + C::TILE_BYTES); };
    const Visible64 vis(g, row0, lane, l32);
    const int n_blocks = (vis.n_all + TB - 1) / TB;
    if (n_blocks == 0) {                                   // dq_acc unchanged
        wait_transfers<0>();
        return;
    }
    if (sp < n_blocks) { fetch_v(sp, 0); fetch_k(sp, 0); }
    const LaneAddr<C> la(lane, lds);
    const LaneAddr<C> la_q(lane, lds_q);
    const float c_log2 = g.scale * LOG2E;
#pragma unroll
    for (int r = 0; r < 2; ++r) neg_l[r] = neg_l[r] == -INFINITY ? -INFINITY : -neg_l[r] * LOG2E;       // a row whose LSE is infinite has P = 0
    // The compiler waits here for everything in flight, not for these loads alone: it does not see the transfers behind them.  So the first
    // K and V have landed too before the barrier, and the wait in front of that finds nothing left to wait for.
    asm volatile("" ::"v"(neg_l[0]), "v"(neg_l[1]), "v"(delta[0]), "v"(delta[1]));
    f32x16 dq[2][C::NDB];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int db = 0; db < C::NDB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) dq[r][db][i] = 0.f;
    acc_settled<C::NDB>(dq);
    if (sp < n_blocks) wait_transfers<2 * C::XFERS>();
    else wait_transfers<0>();
    block_barrier();
    bf16x8 qf[2][C::NKS], gf[2][C::NKS];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            qf[r][ks] = lds_b128(la_q.row[ks] + r * C::TILE_BYTES);
            gf[r][ks] = lds_b128(la_q.row[ks] + r * C::TILE_BYTES + C::NBUF * 2 * C::TILE_BYTES);
        }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            if constexpr (D == 128) { asm volatile("" : "+a"(qf[r][ks])); asm volatile("" : "+a"(gf[r][ks])); }
            else { pin(qf[r][ks]); pin(gf[r][ks]); }
        }
    reads_done();
    block_barrier();                                          // the second buffers are free
    if (sp + NW < n_blocks) { fetch_v(sp + NW, 1); fetch_k(sp + NW, 1); }

    constexpr int N = 2 * C::NDB;                          // MFMAs of a row block in the third product
    static_assert(N == C::NKS, "one transposed read per MFMA");
    constexpr int AHEAD = 3;
    bf16x8 x[C::NKS];
    f32x16 nd[2];                                          // -Delta of the lane's rows, which dP is accumulated on
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < 16; ++i) { nd[r][i] = -delta[r]; asm volatile("" : "+v"(nd[r][i])); }
    // One block, whose first K fragments are on their way.  STEADY: there is a next block, and a whole one after it; its transfers
    // and the first fragments of the next one go between the MFMAs.
    auto step = [&](auto bufc, auto steadyc, int b) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value;
        constexpr bool STEADY = decltype(steadyc)::value;
        constexpr uint32_t kt = buf * 2 * C::TILE_BYTES, vt = kt + C::TILE_BYTES;
        const int b2 = b + 2 * NW;
        const bool next2 = STEADY || b2 < n_blocks;
        const uint16_t *k2 = k + (long long)(b2 * TB) * g.kv_stride_tok, *v2 = v + (long long)(b2 * TB) * g.kv_stride_tok;
        constexpr uint32_t kn = (buf ^ 1) * 2 * C::TILE_BYTES;
        f32x16 s[2], dp[2];
        bf16x8 kx[N];
        uint32_t pw[2][8];
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        // dS of two scores of row block r, left in s[r]
        auto ds2 = [&](int r, int i) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 2 * i; e < 2 * i + 2; ++e) s[r][e] = fast_exp2(fmaf(s[r][e], c_log2, neg_l[r])) * dp[r][e];
            pw[r][i] = pack2(s[r][2 * i], s[r][2 * i + 1]);
            asm volatile("" : "+v"(pw[r][i]), "+v"(s[r][2 * i]), "+v"(s[r][2 * i + 1]));      // stays where it stands
        };
        auto mask = [&](int r) __attribute__((always_inline)) {
            if (b < vis.n_full) return;
            keep_branch();
            const int n = vis.mine[r] - b * TB - 4 * hh;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (8 * (i >> 2) + (i & 3) >= n) s[r][i] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) pw[r][i] = pack2(s[r][2 * i], s[r][2 * i + 1]);
        };
        auto frag = [&](int r, int u) __attribute__((always_inline)) {
            return __builtin_bit_cast(bf16x8, make_uint4(pw[r][4 * u], pw[r][4 * u + 1], pw[r][4 * u + 2], pw[r][4 * u + 3]));
        };
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            const bf16x8 kfrag = x[ks];
            if (ks + AHEAD < C::NKS) x[ks + AHEAD] = lds_b128(la.row[ks + AHEAD] + kt);
            __builtin_amdgcn_sched_barrier(0);
            s[0] = mfma32(kfrag, qf[0][ks], ks == 0 ? zero : s[0]);
            __builtin_amdgcn_sched_barrier(0);
            s[1] = mfma32(kfrag, qf[1][ks], ks == 0 ? zero : s[1]);
            __builtin_amdgcn_sched_barrier(0);
            x[ks] = lds_b128(la.row[ks] + vt);             // the fragments of V, in the places that are free
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            dp[0] = mfma32(x[ks], gf[0][ks], ks == 0 ? nd[0] : dp[0]);
            __builtin_amdgcn_sched_barrier(0);
        }
        auto read = [&](int st) __attribute__((always_inline)) {
            const uint32_t o = kt + st / C::NDB * 16 * C::ROW_BYTES;
            kx[st] = lds_tr(la.tr[0][st % C::NDB] + o, la.tr[1][st % C::NDB] + o);
        };
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {              // beside it dS of the first row block, and the reads of the third product
            dp[1] = mfma32(x[ks], gf[1][ks], ks == 0 ? nd[1] : dp[1]);
            __builtin_amdgcn_sched_barrier(0);
            for (int i = ks * 8 / C::NKS; i < (ks + 1) * 8 / C::NKS; ++i) ds2(0, i);
            read(ks);
            __builtin_amdgcn_sched_barrier(0);
        }
        mask(0);
        if (!STEADY && next2) fetch_v(b2, buf);
#pragma unroll
        for (int st = 0; st < N; ++st) {                   // beside it dS of the second row block
            mfma_acc(dq[0][st % C::NDB], kx[st], frag(0, st / C::NDB));
            __builtin_amdgcn_sched_barrier(0);
            for (int i = st * 8 / N; i < (st + 1) * 8 / N; ++i) ds2(1, i);
            if (STEADY) fetch.one(v2, g.kv_stride_tok, lds + vt, st);
            __builtin_amdgcn_sched_barrier(0);
        }
        mask(1);
        reads_done();                                      // K is free
        if (!STEADY && next2) fetch_k(b2, buf);
        // Blocks with some |bf16(dS)| >= 2 (bit 14 of the pattern) also add the residuals dS - bf16(dS), as two more bf16
        // operands: three bf16 hold 24 bits, so dS reaches the product unrounded.
        uint32_t big = 0;
#pragma unroll
        for (int st = 0; st < N; ++st) {
            if (st == C::XFERS / 2 && (STEADY || b + NW < n_blocks)) {      // the next block has landed
                if (next2) wait_transfers<2 * C::XFERS>();
                else wait_transfers<0>();
#pragma unroll
                for (int ks = 0; ks < AHEAD; ++ks) x[ks] = lds_b128(la.row[ks] + kn);
            }
            mfma_acc(dq[1][st % C::NDB], kx[st], frag(1, st / C::NDB));
            __builtin_amdgcn_sched_barrier(0);
            if (STEADY && st < C::XFERS / 2) {
                fetch.one(k2, g.kv_stride_tok, lds + kt, 2 * st);
                fetch.one(k2, g.kv_stride_tok, lds + kt, 2 * st + 1);
            }
#pragma unroll
            for (int i = st * 8 / N; i < (st + 1) * 8 / N; ++i) big |= pw[0][i] | pw[1][i];
            __builtin_amdgcn_sched_barrier(0);
        }
        if (__any((big & 0x40004000u) != 0u)) {
#pragma unroll
            for (int n = 0; n < 2; ++n)
#pragma unroll
                for (int r = 0; r < 2; ++r) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const bf16x2 t = __builtin_bit_cast(bf16x2, pw[r][i]);
                        s[r][2 * i] -= (float)t[0];
                        s[r][2 * i + 1] -= (float)t[1];
                        pw[r][i] = pack2(s[r][2 * i], s[r][2 * i + 1]);
                    }
#pragma unroll
                    for (int st = 0; st < N; ++st) mfma_acc(dq[r][st % C::NDB], kx[st], frag(r, st / C::NDB));
                }
        }
    };
    if (sp < n_blocks) {
        if (sp + NW < n_blocks) wait_transfers<2 * C::XFERS>();
        else wait_transfers<0>();
#pragma unroll
        for (int ks = 0; ks < AHEAD; ++ks) x[ks] = lds_b128(la.row[ks]);
        using Steady = std::true_type; using Last = std::false_type;
        const int n_whole = n_blocks < g.lc / TB ? n_blocks : g.lc / TB;
        int b = sp;
        for (; b + 3 * NW < n_whole; b += 2 * NW) {        // two blocks at a time: the buffer is a compile-time offset of the reads
            step(IC<0>{}, Steady{}, b);
            step(IC<1>{}, Steady{}, b + NW);
        }
        for (; b < n_blocks; b += 2 * NW) {
            step(IC<0>{}, Last{}, b);
            if (b + NW < n_blocks) step(IC<1>{}, Last{}, b + NW);
        }
    }
    acc_settled<C::NDB>(dq);
    f32x4 old[C::OUT_VECS];
#pragma unroll
    for (int j = 0; j < C::OUT_VECS; ++j) {                // (rows past the end read the last one)
        const int i = tid + 64 * NW * j, r = row0 + i / (D / 4), c = 4 * (i % (D / 4));
        old[j] = *reinterpret_cast<const f32x4*>(a.dq + ((long long)(r < g.lq ? r : g.lq - 1) * g.nq + h) * D + c);
    }
    __syncthreads();
    stage64<C>(sm.stage, dq, sp, l32, hh, g.scale);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < C::OUT_VECS; ++j) {
        const int i = tid + 64 * NW * j;
        old[j] += staged_sum<C>(sm.stage, i / (D / 4), 4 * (i % (D / 4)));
    }
#pragma unroll
    for (int j = 0; j < C::OUT_VECS; ++j) {
        const int i = tid + 64 * NW * j, r = row0 + i / (D / 4), c = 4 * (i % (D / 4));
        if (r < g.lq) *reinterpret_cast<f32x4*>(a.dq + ((long long)r * g.nq + h) * D + c) = old[j];
    }
}

// dK / dV of 64 keys from the q rows of a run of heads: S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.  V stays in registers, K in
// LDS at D = 128 (dK and dV take 256 of a wavefront's 512 registers there) and in registers at D = 64.
template <class C> union QuadDkdvSmem {
    struct {
        unsigned char t[NW][C::NBUF][2 * C::TILE_BYTES];   // Q and dO block of each wavefront
        unsigned char k[2 * C::TILE_BYTES];                // the workgroup's K rows
        float lse[NW][C::NBUF][64], delta[NW][C::NBUF][64];      // row scalars of each wavefront's blocks (32 used; a transfer writes 64)
    } m;
    float stage[C::STAGE_FLOATS];
};

template <int D, bool ATOMIC_DKV>
__device__ __forceinline__ void dkdv_unit(const BwdArgs& a, const HeadRuns& runs, const int run, const int kv_tile, QuadDkdvSmem<QuadCfg<D>>& sm)
{
    using C = QuadCfg<D>;
    const AttnGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int sp = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    const int col0 = kv_tile * ROWS;
    const int n_heads = arg_byte(runs.len, run);
    const int h0 = arg_byte(runs.first, run);
    const int kvh = arg_byte(g.kv_of_q, h0);
    const uint32_t lds_all = (uint32_t)(uintptr_t)(&sm.m.t[0][0][0]);
    const uint32_t lds = lds_all + sp * C::NBUF * 2 * C::TILE_BYTES;
    // the unit's own keys: K in its place, V by way of the second buffer of wavefront 0
    const uint32_t lds_k = (uint32_t)(uintptr_t)(&sm.m.k[0]), lds_v = lds_all + 2 * C::TILE_BYTES;
    fetch_rows<C, ROWS, NW>(static_cast<const uint16_t*>(a.v) + (long long)kvh * g.kv_stride_head, g.kv_stride_tok, col0, g.lc, lds_v, sp, lane);
    fetch_rows<C, ROWS, NW>(static_cast<const uint16_t*>(a.k) + (long long)kvh * g.kv_stride_head, g.kv_stride_tok, col0, g.lc, lds_k, sp, lane);
    // the rows that see a key are a suffix of the shard: [my_first, lq); no row before row_first sees any of the keys,
    // all rows from row_full on see all of them
    const int first = rows_le(g.qs, pos_of_row(g.ks, col0 + lane < g.lc ? col0 + lane : g.lc - 1) - 1);
    const int first_here = col0 + lane < g.lc ? first : 0x7fffffff;
    const int my_first[2] = {__shfl(first_here, l32, 64), __shfl(first_here, 32 + l32, 64)};
    const int row_first = __builtin_amdgcn_readlane(first, 0);
    const int row_full = __builtin_amdgcn_readlane(first_here, 63);
    const int blk0 = row_first / TB;
    const int n_all = row_first < g.lq ? (g.lq + TB - 1) / TB - blk0 : 0;      // blocks of one head

    const BlockFetch<C> fetch(lane, g.q_stride_tok);
    const uint32_t lds_lse = (uint32_t)(uintptr_t)(&sm.m.lse[sp][0][0]), lds_delta = (uint32_t)(uintptr_t)(&sm.m.delta[sp][0][0]);
    // The workgroup's sequence of blocks: those of the first head of the run, then the next head's; a wavefront takes every fourth
    // one.  (h, t): the next block to ask for.  The last block of a head is moved back to the last 32 rows (the rows of the block
    // before are masked), so that all blocks are whole unless the shard has fewer rows.
    const int cnt = n_all * n_heads > sp ? (n_all * n_heads - sp + NW - 1) / NW : 0;
    int h = h0, t = sp;
    auto normalise = [&]() { while (t >= n_all) { t -= n_all; h = arg_byte(runs.next, h); } };
    auto start_of = [&](int row) { return row + TB <= g.lq || g.lq < TB ? row : g.lq - TB; };
    const uint32_t scalar_off = 4u * (uint32_t)(l32 < g.lq ? l32 : g.lq - 1);      // (a shard of fewer rows than a block has one block a head)
    auto scalars = [&](int buf, int hd, int row) __attribute__((always_inline)) {
        const long long first = (long long)hd * g.lq + row;
        lds_dma4_base(a.lse + first, scalar_off, __builtin_amdgcn_readfirstlane(lds_lse + buf * 256));
        lds_dma4_base(a.delta + first, scalar_off, __builtin_amdgcn_readfirstlane(lds_delta + buf * 256));
    };
    auto g_of = [&](int hd) { return static_cast<const uint16_t*>(a.d_o) + (long long)hd * g.q_stride_head; };
    auto q_of = [&](int hd) { return static_cast<const uint16_t*>(a.q) + (long long)hd * g.q_stride_head; };
    auto fetch_block = [&](int buf) __attribute__((always_inline)) {      // the block at the cursor
        const uint32_t dst = lds + buf * 2 * C::TILE_BYTES;
        const int row = start_of((blk0 + t) * TB);
        scalars(buf, h, row);
        fetch.issue(g_of(h), g.q_stride_tok, row, g.lq, dst + C::TILE_BYTES);
        fetch.issue(q_of(h), g.q_stride_tok, row, g.lq, dst);
    };
    int cur = 0, nxt = 0;                                  // first rows of this wavefront's next two blocks
    if (cnt > 0) {
        normalise();
        cur = (blk0 + t) * TB;
        fetch_block(0);
    }
    LaneXor<C> la(lane, lds);
    const LaneXor<C> la_v(lane, lds_v);
    uint32_t k_row = la.row0 - lds + lds_k;
    f32x16 dk[2][C::NDB], dv[2][C::NDB];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int db = 0; db < C::NDB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) { dk[r][db][i] = 0.f; dv[r][db][i] = 0.f; }
    acc_settled<C::NDB>(dk);
    acc_settled<C::NDB>(dv);
    const float scale_log2 = g.scale * LOG2E;
    if (cnt > 0) wait_transfers<2 * C::XFERS + 2>();
    else wait_transfers<0>();
    block_barrier();
    constexpr bool K_REGS = D == 64;
    bf16x8 vf[2][C::NKS], kf[K_REGS ? 2 : 1][K_REGS ? C::NKS : 1];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            vf[r][ks] = la_v.read_row(ks, r * C::TILE_BYTES);
            if constexpr (K_REGS) kf[r][ks] = lds_b128((k_row ^ (32u * ks)) + r * C::TILE_BYTES);
        }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            if constexpr (K_REGS) { asm volatile("" : "+a"(vf[r][ks])); asm volatile("" : "+a"(kf[r][ks])); }
            else pin(vf[r][ks]);
        }
    reads_done();
    block_barrier();                                          // the second buffers are free
    if (cnt > 1) {
        t += NW;
        normalise();
        nxt = (blk0 + t) * TB;
        fetch_block(1);
    }

    constexpr int N = 2 * C::NDB;
    static_assert(N == C::NKS, "one transposed read per MFMA");
    constexpr int AHEAD = D == 128 ? 2 : 3, EVERY = D == 128 ? 2 : 1;     // (registers; LDS gives four wavefronts about 4 KB in the time of two MFMAs)
    bf16x8 x[C::NKS], ka[4], kb[4];
    auto read_k = [&](int ks, uint32_t qt) __attribute__((always_inline)) {
        x[ks] = la.read_row(ks, qt);
        if constexpr (!K_REGS) { const uint32_t o = k_row ^ (32u * ks); ka[ks & 3] = lds_b128(o); kb[ks & 3] = lds_b128(o + C::TILE_BYTES); }
    };
    auto read_first = [&](uint32_t qt) __attribute__((always_inline)) {
        la.here();
        asm volatile("" : "+v"(k_row));
#pragma unroll
        for (int ks = 0; ks < AHEAD; ++ks) read_k(ks, qt);
    };
    // Block i of the wavefront, whose first fragments are on their way.  STEADY: two more follow (and blocks are whole); the transfers
    // of the second one, the scalar work for it and the first fragments of the next one go between the MFMAs.
    auto step = [&](auto bufc, auto steadyc, int i) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value;
        constexpr bool STEADY = decltype(steadyc)::value;
        constexpr uint32_t qt = buf * 2 * C::TILE_BYTES, gt = qt + C::TILE_BYTES, qn = (buf ^ 1) * 2 * C::TILE_BYTES;
        const bool have1 = STEADY || i + 1 < cnt, have2 = STEADY || i + 2 < cnt;
        const int row = start_of(cur);                     // (rows before `cur` belong to the block before)
        int row2 = 0, start2 = 0;
        const uint16_t *q2 = nullptr, *g2 = nullptr;
        float* const lse = &sm.m.lse[sp][buf][0];
        float* const delta = &sm.m.delta[sp][buf][0];
        f32x16 s[2], dp[2];
        bf16x8 y[N];
        uint32_t pw[2][8], dw[2][8];
        f32x4 l4[4];                                       // -log2e LSE of the lane's 16 rows
        float own_lse = 0.f, own_delta = 0.f;
        f32x16 nd;                                         // -Delta of the lane's 16 rows, which dP is accumulated on
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        // P and dS of two scores of key block c (rows 8 (i / 2) + 4 hh + 2 (i % 2), and the next)
        auto pd2 = [&](int c, int i) __attribute__((always_inline)) {
            const int rb = i >> 1, e = 2 * (i & 1);
            const float p0 = fast_exp2(fmaf(s[c][2 * i], scale_log2, l4[rb][e])), p1 = fast_exp2(fmaf(s[c][2 * i + 1], scale_log2, l4[rb][e + 1]));
            pw[c][i] = pack2(p0, p1);
            dw[c][i] = pack2(p0 * dp[c][2 * i], p1 * dp[c][2 * i + 1]);
            asm volatile("" : "+v"(pw[c][i]), "+v"(dw[c][i]));      // stays where it stands
        };
        auto mask = [&](int c) __attribute__((always_inline)) {     // (a row that sees nothing anywhere, LSE = -inf, is masked in every block)
            if (cur >= row_full && cur + TB <= g.lq) return;
            keep_branch();
            const int lo = my_first[c] > cur ? my_first[c] : cur;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r0 = row + 8 * (i >> 1) + 4 * hh + 2 * (i & 1);
                const uint32_t keep = (r0 >= lo && r0 < g.lq ? 0xffffu : 0u) | (r0 + 1 >= lo && r0 + 1 < g.lq ? 0xffff0000u : 0u);
                pw[c][i] &= keep;
                dw[c][i] &= keep;
            }
        };
        auto frag = [&](const uint32_t (&w)[8], int u) __attribute__((always_inline)) {
            return __builtin_bit_cast(bf16x8, make_uint4(w[4 * u], w[4 * u + 1], w[4 * u + 2], w[4 * u + 3]));
        };
        // S of both key blocks
        la.here();
        asm volatile("" : "+v"(k_row));
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            const bf16x8 qfrag = x[ks];
            if (ks + AHEAD < C::NKS) read_k(ks + AHEAD, qt);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (K_REGS) s[0] = mfma32(qfrag, kf[0][ks], ks == 0 ? zero : s[0]);
            else s[0] = mfma32(qfrag, ka[ks & 3], ks == 0 ? zero : s[0]);
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 1 && have2) {                        // where the block after the next lies
                t += NW;
                normalise();
                row2 = (blk0 + t) * TB;
                start2 = start_of(row2);
                q2 = q_of(h) + (long long)start2 * g.q_stride_tok;
                g2 = g_of(h) + (long long)start2 * g.q_stride_tok;
            }
            if (ks == 0) { own_lse = lse[lane]; own_delta = delta[lane]; }       // (private to the wavefront)
            if (ks == C::NKS / 2) { lse[lane] = own_lse * -LOG2E; delta[lane] = -own_delta; }
            if (ks == C::NKS - 1) {
#pragma unroll
                for (int rb = 0; rb < 4; ++rb) {
                    const f32x4 d4 = *reinterpret_cast<const f32x4*>(&delta[8 * rb + 4 * hh]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) nd[4 * rb + e] = d4[e];
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (K_REGS) s[1] = mfma32(qfrag, kf[K_REGS ? 1 : 0][ks], ks == 0 ? zero : s[1]);
            else s[1] = mfma32(qfrag, kb[ks & 3], ks == 0 ? zero : s[1]);
            __builtin_amdgcn_sched_barrier(0);
            if (ks % EVERY == EVERY - 1) x[ks / EVERY] = la.read_row(ks / EVERY, gt);      // the fragments of dO, in the places that are free
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {
            if (C::NKS / EVERY + ks < C::NKS) x[C::NKS / EVERY + ks] = la.read_row(C::NKS / EVERY + ks, gt);
            __builtin_amdgcn_sched_barrier(0);
            dp[0] = mfma32(x[ks], vf[0][ks], ks == 0 ? nd : dp[0]);
            for (int rb = ks * 4 / C::NKS; rb < (ks + 1) * 4 / C::NKS; ++rb) l4[rb] = *reinterpret_cast<const f32x4*>(&lse[8 * rb + 4 * hh]);
            __builtin_amdgcn_sched_barrier(0);
        }
        auto read_tr = [&](uint32_t tile, int st) __attribute__((always_inline)) { y[st] = la.read_tr(st / C::NDB, st % C::NDB, tile); };
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) {              // beside it P and dS of the first key block, and the reads of dO^T
            dp[1] = mfma32(x[ks], vf[1][ks], ks == 0 ? nd : dp[1]);
            __builtin_amdgcn_sched_barrier(0);
            for (int i = ks * 8 / C::NKS; i < (ks + 1) * 8 / C::NKS; ++i) pd2(0, i);
            read_tr(gt, ks);
            __builtin_amdgcn_sched_barrier(0);
        }
        mask(0);
#pragma unroll
        for (int st = 0; st < N; ++st) {                   // beside it those of the second one
            mfma_acc(dv[0][st % C::NDB], y[st], frag(pw[0], st / C::NDB));
            __builtin_amdgcn_sched_barrier(0);
            for (int i = st * 8 / N; i < (st + 1) * 8 / N; ++i) pd2(1, i);
            __builtin_amdgcn_sched_barrier(0);
        }
        mask(1);
        reads_done();                                      // dO and the row scalars are free
        if (have2) scalars(buf, h, start2);
        if (!STEADY && have2) fetch.issue(g_of(h), g.q_stride_tok, start2, g.lq, lds + gt);
#pragma unroll
        for (int st = 0; st < N; ++st) {                   // beside it the reads of Q^T
            mfma_acc(dv[1][st % C::NDB], y[st], frag(pw[1], st / C::NDB));
            __builtin_amdgcn_sched_barrier(0);
            read_tr(qt, st);
            if (STEADY) fetch.one(g2, g.q_stride_tok, lds + gt, st);
            __builtin_amdgcn_sched_barrier(0);
        }
        constexpr int FREE = N / 4, LANDED = FREE + C::XFERS / 2;
#pragma unroll
        for (int st = 0; st < N; ++st) {
            if (st == FREE) {                              // Q is free
                reads_done();
                if (!STEADY && have2) fetch.issue(q_of(h), g.q_stride_tok, start2, g.lq, lds + qt);
            }
            if (st == LANDED && have1) {                   // the next block has landed
                if (have2) wait_transfers<2 * C::XFERS + 2>();
                else wait_transfers<0>();
                read_first(qn);
            }
            mfma_acc(dk[0][st % C::NDB], y[st], frag(dw[0], st / C::NDB));
            __builtin_amdgcn_sched_barrier(0);
            if (STEADY && st >= FREE && st < LANDED) fetch.one(q2, g.q_stride_tok, lds + qt, 2 * (st - FREE));
            mfma_acc(dk[1][st % C::NDB], y[st], frag(dw[1], st / C::NDB));
            __builtin_amdgcn_sched_barrier(0);
            if (STEADY && st >= FREE && st < LANDED) fetch.one(q2, g.q_stride_tok, lds + qt, 2 * (st - FREE) + 1);
        }
        cur = nxt;
        nxt = row2;
    };
    if (cnt > 0) {
        using Steady = std::true_type; using Last = std::false_type;
        if (cnt > 1) wait_transfers<2 * C::XFERS + 2>();
        else wait_transfers<0>();
        read_first(0);
        int i = 0;
        if (g.lq >= TB)
            for (; i + 3 < cnt; i += 2) {                  // two blocks at a time: the buffer is a compile-time offset of the reads
                step(IC<0>{}, Steady{}, i);
                step(IC<1>{}, Steady{}, i + 1);
            }
        for (; i < cnt; i += 2) {
            step(IC<0>{}, Last{}, i);
            if (i + 1 < cnt) step(IC<1>{}, Last{}, i + 1);
        }
    }

    acc_settled<C::NDB>(dk);
    acc_settled<C::NDB>(dv);
    auto write_out = [&](float* out, const f32x16 (&acc)[2][C::NDB], float w) {
        __syncthreads();
        stage64<C>(sm.stage, acc, sp, l32, hh, w);
        __syncthreads();
        if (ATOMIC_DKV) {          // consecutive lanes on consecutive floats
#pragma unroll 8
            for (int i = tid; i < ROWS * D; i += 64 * NW) {
                const int r = i / D, c = i % D;
                float x = sm.stage[r * C::PITCH + c];
#pragma unroll
                for (int s = 1; s < NW; ++s) x += sm.stage[(s * ROWS + r) * C::PITCH + c];
                if (col0 + r < g.lc) global_atomic_add(out + ((long long)(col0 + r) * g.nkv + kvh) * D + c, x);
            }
        } else {
            f32x4 x[C::OUT_VECS];
#pragma unroll
            for (int j = 0; j < C::OUT_VECS; ++j) {
                const int i = tid + 64 * NW * j;
                x[j] = staged_sum<C>(sm.stage, i / (D / 4), 4 * (i % (D / 4)));
            }
#pragma unroll
            for (int j = 0; j < C::OUT_VECS; ++j) {
                const int i = tid + 64 * NW * j, r = col0 + i / (D / 4), c = 4 * (i % (D / 4));
                if (r >= g.lc) continue;
                f32x4* op = reinterpret_cast<f32x4*>(out + ((long long)r * g.nkv + kvh) * D + c);
                if (a.accumulate) x[j] += *op;
                *op = x[j];
            }
        }
    };
    write_out(a.dv, dv, 1.0f);
    write_out(a.dk, dk, g.scale);
}

// One launch for both halves of a backward step: workgroups [0, n_dkdv) are dK / dV units (the longer ones, first), the
// others dQ units.  Within each, heads (runs) side by side and the longest tiles first.
template <int D, bool ATOMIC_DKV>
__global__ void __launch_bounds__(256, 1) bwd_quad_bf16_kernel(const BwdArgs a, const HeadRuns runs, const unsigned n_dkdv, const int n_q_tiles)
{
    __shared__ __attribute__((aligned(1024))) union { QuadDkdvSmem<QuadCfg<D>> dkdv; QuadDqSmem<QuadCfg<D>> dq; } sm;
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

hipError_t hexi_launch_fwd_quad_bf16(const FwdArgs& a, QuadRest rest, hipStream_t s)
{
    if (rest.tiles == 0) rest.tiles = (a.g.lq + ROWS - 1) / ROWS;
    const dim3 grid((unsigned)a.g.nq, (unsigned)rest.tiles);
    if (a.g.d == 128) fwd_quad_bf16_kernel<128><<<grid, 256, 0, s>>>(a, rest);
    else if (a.g.d == 64) fwd_quad_bf16_kernel<64><<<grid, 256, 0, s>>>(a, rest);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// dq, dkdv: which halves; runs: the head runs of the dK / dV workgroups
hipError_t hexi_launch_bwd_quad_bf16(const BwdArgs& a, bool dq, const HeadRuns& runs, bool shared, hipStream_t s)
{
    const int n_q_tiles = dq ? (a.g.lq + ROWS - 1) / ROWS : 0;
    const int n_keys = shared ? hexi_keys_seen(a.g) : a.g.lc;
    const unsigned n_dkdv = (unsigned)((n_keys + ROWS - 1) / ROWS) * (unsigned)runs.n;
    const unsigned grid = n_dkdv + (unsigned)n_q_tiles * (unsigned)a.g.nq;
    if (grid == 0) return hipSuccess;
    if (a.g.d == 128) {
        if (shared) bwd_quad_bf16_kernel<128, true><<<grid, 256, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
        else bwd_quad_bf16_kernel<128, false><<<grid, 256, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
    } else if (a.g.d == 64) {
        if (shared) bwd_quad_bf16_kernel<64, true><<<grid, 256, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
        else bwd_quad_bf16_kernel<64, false><<<grid, 256, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
    } else return hipErrorInvalidValue;
    return hipGetLastError();
}

// bf16 ring step (forward, dQ, dK/dV) for launches too small to fill the chip with the 256-row / 128-key workgroups of
// the other bf16 kernels: a workgroup owns 32 (or, q rows only, 64) stationary rows (q rows of one head; keys of one kv head in
// the dK/dV kernel) and its 8 wavefronts split the streamed rows between them, 32 at a time (32 stationary rows: block b
// goes to wavefront b % 8).  A wavefront streams its own blocks through a private piece of LDS, without any barrier before
// the end, where the partial results are combined through LDS in a fixed order.
//
// What bounds it: on the shards it is chosen for, the serial chain of a workgroup, which is 8 (or 4) times shorter than
// that of the large workgroups, of which there are too few there: 1024 rows x 8 heads are 32 workgroups of 256 rows on
// 256 CUs, and 256 of 32.  Per 32-row block a wavefront takes 1.5 to 2 us, about twice its MFMAs and vector work: the
// transfers into LDS (16 KB per block and wavefront) hold it while it issues them and while it waits.  With 64 rows per
// workgroup (forward and dQ) two wavefronts share every streamed block, double-buffered: 1.4 us per block, but chains twice
// as long.  The large kernels stream an eighth as much per row and stay the better choice once they fill the chip: see the
// rules in hexi_shapes.h.  Measured, us per call (head_dim 128, fully visible chunk), large workgroups -> these:
//   512 rows x 1024 keys, 24 / 8 heads: forward 32.0 -> 16.3, dQ 47.6 -> 20.3, dK/dV 46.3 -> 21.2;
//   300 x 700, 4 / 2 heads: 27.5 -> 9.7, 35.3 -> 11.2, 23.9 -> 11.5.
//
// Operand layouts are those of the large kernels (hexi_mfma.h): scores transposed in the forward and dQ kernels (a lane
// owns a q row), keys across the lanes in the dK/dV kernel; accumulator registers go straight back in as operands, the
// other operand through transposed LDS reads.  A block's LDS image is [32][D] bf16 with the 16-byte pieces of a row
// permuted by piece ^ swz(row), which makes the 128-bit row reads (16 rows, one piece) and the transposed 64-bit reads
// (4 rows x 64 bytes) both touch all 64 banks once.
#include <cstddef>
#include "hexi_internal.h"
#include "hexi_mfma.h"

namespace {

constexpr int NW = 8;          // wavefronts per workgroup
constexpr int TB = 32;         // rows of a block, stationary or streamed
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float NEG_BIG = -1.0e30f;        // finite stand-in for "no key seen yet"
constexpr float RESCALE_SLACK = 8.0f;

// a value that is the same in all lanes, in a scalar register
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// R: 32-row blocks of stationary rows per workgroup; S = 8 / R wavefronts share a block and split the streamed rows
template <int D_, int R_> struct SplitCfg {
    static constexpr int D = D_, R = R_, S = NW / R, ROWS = TB * R;
    static constexpr int NBUF = R == 1 ? 1 : 2;            // buffers per split
    static_assert(D == 64 || D == 128, "head_dim 64 or 128");
    static constexpr int NKS = D / 16;                     // 16-wide contraction steps across the head dimension
    static constexpr int NDB = D / 32;                     // 32-column blocks of an output
    static constexpr int ROW_BYTES = 2 * D, PIECES = D / 8;
    static constexpr int TILE_BYTES = TB * ROW_BYTES;      // one block of one tensor: 8 or 4 KB
    static constexpr int XFERS = TILE_BYTES / 1024;        // wave-wide transfers per block: 8 or 4
    static constexpr int PITCH = D + 4;                    // floats per staged output row
    static constexpr int STAGE_FLOATS = NW * TB * PITCH;
    static constexpr int BUF_BYTES = S * 2 * TILE_BYTES;   // one buffer of all splits, both tensors
    // position of 16-byte piece `c` of row r: c ^ swz(r)
    __host__ __device__ static constexpr int swz(int r) { return D == 128 ? (((r & 3) << 2) | ((r >> 2) & 3)) : (((r & 2) << 1) | ((r >> 2) & 3)); }
};

typedef const bf16x8 HEXI_LDS* lds_b128_ptr;
__device__ __forceinline__ bf16x8 lds_b128(uint32_t addr) { return *(lds_b128_ptr)(uintptr_t)addr; }
__device__ __forceinline__ bf16x8 lds_tr(uint32_t a, uint32_t b)
{
    return join_halves(__builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 HEXI_LDS*)(uintptr_t)a), __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 HEXI_LDS*)(uintptr_t)b));
}

// At most N of this wavefront's transfers are still in flight (they complete in order).
template <int N> __device__ __forceinline__ void wait_transfers() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// This wavefront's LDS reads have returned: the block they came from may be overwritten.
__device__ __forceinline__ void reads_done()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Transfers of one block by one wavefront: lane parts of the source offsets.  Rows 16 apart share their lane part.
template <class C> struct BlockFetch {
    static constexpr int HALF = C::XFERS / 2;
    static constexpr int RPX = 1024 / C::ROW_BYTES;        // rows per transfer: 4 or 8
    uint32_t off[HALF];
    int rl;
    __device__ __forceinline__ BlockFetch(int lane, long long stride_tok)
    {
        rl = lane / C::PIECES;
        const int p = lane % C::PIECES;
#pragma unroll
        for (int i = 0; i < HALF; ++i) {
            const int r = i * RPX + rl;
            off[i] = 2u * (uint32_t)(r * (int)stride_tok) + 16u * (uint32_t)(p ^ C::swz(r));
        }
    }
    // rows [row0, row0 + 32) of `src`; rows past `total` re-read the last one (row0 < total)
    __device__ __forceinline__ void issue(const uint16_t* src, long long stride_tok, int row0, int total, uint32_t lds) const
    {
        const uint16_t* base = src + (long long)row0 * stride_tok;
        if (row0 + TB <= total) {
#pragma unroll
            for (int i = 0; i < C::XFERS; ++i)
                lds_dma16_base(base + (long long)(i / HALF * 16) * stride_tok, off[i % HALF], __builtin_amdgcn_readfirstlane(lds + i * 1024));
        } else {
#pragma unroll
            for (int i = 0; i < C::XFERS; ++i) {
                uint32_t o = off[i % HALF] + 2u * (uint32_t)(i / HALF * 16 * (int)stride_tok);
                const int over = row0 + i * RPX + rl - (total - 1);
                if (over > 0) o -= 2u * (uint32_t)(over * (int)stride_tok);
                lds_dma16_base(base, o, __builtin_amdgcn_readfirstlane(lds + i * 1024));
            }
        }
    }
};

// Lane parts of the LDS reads of a block.
template <class C> struct LaneAddr {
    uint32_t row[C::NKS];          // row l32, columns 16 ks + 8 hh .. + 7
    uint32_t tr[2][C::NDB];        // transposed: rows 8 second + 4 hh + jj (+ 16 u), columns 32 db + 16 grp2 + 4 (j16 % 4) .. + 3
    __device__ __forceinline__ LaneAddr(int lane, uint32_t base)
    {
        const int l32 = lane & 31, hh = lane >> 5, grp2 = (lane >> 4) & 1, j16 = lane & 15, jj = j16 >> 2;
#pragma unroll
        for (int ks = 0; ks < C::NKS; ++ks) row[ks] = base + (uint32_t)(l32 * C::ROW_BYTES + 16 * ((2 * ks + hh) ^ C::swz(l32)));
#pragma unroll
        for (int sec = 0; sec < 2; ++sec)
#pragma unroll
            for (int db = 0; db < C::NDB; ++db) {
                const int r = 8 * sec + 4 * hh + jj, piece = 4 * db + 2 * grp2 + ((j16 & 3) >> 1);
                tr[sec][db] = base + (uint32_t)(r * C::ROW_BYTES + 16 * (piece ^ C::swz(r)) + 8 * (j16 & 1));
            }
    }
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

// acc[db] += (columns of the block at `tile`) x p over its 32 rows; p[u] holds rows 16 u .. + 15 in accumulator order.
// STREAM_FIRST: the block's columns are the first operand (the accumulator's rows), else p is.
template <class C, bool STREAM_FIRST> __device__ __forceinline__ void col_product(f32x16 (&acc)[C::NDB], const LaneAddr<C>& la, const uint32_t tile, const bf16x8 (&p)[2])
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
        acc[db] = STREAM_FIRST ? mfma32(x[st & 3], p[u], acc[db]) : mfma32(p[u], x[st & 3], acc[db]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Keeps the compiler from turning the (wave-uniform) branch it stands in into selects that every block would execute.
__device__ __forceinline__ void keep_branch() { asm volatile(""); }

// Entry i of a byte table in the kernel arguments, through an aligned 32-bit read (a byte read would go through the vector
// memory path: it would hold up the first transfers by its latency, and wait for every transfer in flight in a loop).
__device__ __forceinline__ int arg_byte(const void* table, int i)
{
    return uniform((static_cast<const uint32_t*>(table)[i >> 2] >> (8 * (i & 3))) & 0xff);
}
static_assert(offsetof(AttnGeom, kv_of_q) % 4 == 0 && offsetof(HeadRuns, first) % 4 == 0 && offsetof(HeadRuns, next) % 4 == 0 &&
              offsetof(HeadRuns, len) % 4 == 0 && HEXI_MAX_HEADS % 4 == 0, "the tables are read in words");

// seg_pos_of_row and seg_rows_le with the first two segments in a straight line: their table entries are then read together
// at the start of the kernel, not one after the other (a table's unused row0 entries hold the total, so a second segment
// that does not exist changes nothing).
__device__ __forceinline__ int pos_of_row(const SegTable& t, int row)
{
    int p = row >= t.row0[1] ? t.start[1] + (row - t.row0[1]) : t.start[0] + row;
    for (int s = 2; s < t.n; ++s)
        if (row >= t.row0[s]) p = t.start[s] + (row - t.row0[s]);
    return p;
}
__device__ __forceinline__ int rows_le(const SegTable& t, int p)
{
    auto in_seg = [&](int s) {
        const int len = t.row0[s + 1] - t.row0[s], k = p - t.start[s] + 1;
        return k < 0 ? 0 : (k > len ? len : k);
    };
    int c = in_seg(0) + in_seg(1);
    for (int s = 2; s < t.n; ++s) c += in_seg(s);
    return c;
}

// What the rows of a q tile see of the chunk (prefixes of its keys).
struct Visible {
    int mine;       // keys the lane's row sees (0 for padding rows)
    int n_all;      // keys some row of the workgroup sees
    int n_full;     // 32-key blocks every row of the wavefront sees in full
    __device__ __forceinline__ Visible(const AttnGeom& g, int row0, int wg_last_row, int l32, int hh)
    {
        // lanes 0..31 look up the wavefront's rows, the others the workgroup's last row
        const int row = hh == 0 ? (row0 + l32 < g.lq ? row0 + l32 : g.lq - 1) : wg_last_row;
        const int n = rows_le(g.ks, pos_of_row(g.qs, row));
        n_all = __builtin_amdgcn_readlane(n, 32);
        n_full = row0 < g.lq ? __builtin_amdgcn_readlane(n, 0) / TB : 0;
        mine = __shfl(n, l32, 64);
        if (row0 + l32 >= g.lq) mine = 0;
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

// (at head_dim 64 two workgroups fit a CU if the registers are held to 128)
template <int D, int R>
__global__ void __launch_bounds__(512, D == 64 ? 4 : 2) fwd_split_bf16_kernel(const FwdArgs a, const int n_q_tiles)
{
    using C = SplitCfg<D, R>;
    constexpr int S = C::S;
    const AttnGeom& g = a.g;
    __shared__ __attribute__((aligned(1024))) union {
        unsigned char t[S][C::NBUF][2 * C::TILE_BYTES];    // K and V block of each split
        struct { float stage[C::STAGE_FLOATS], m[NW * TB], l[NW * TB], lr[NW * TB], w[NW * TB], wa[C::ROWS]; } e;
    } sm;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave % R, sp = wave / R;                // row block, split
    const int l32 = lane & 31, hh = lane >> 5;

    // heads of a q tile side by side, the longest (last) q tiles first
    const int h = blockIdx.x;
    const int wg_row0 = (n_q_tiles - 1 - (int)blockIdx.y) * C::ROWS, row0 = wg_row0 + TB * rb;
    const int kvh = arg_byte(g.kv_of_q, h);
    const int my_row = row0 + l32;
    const int my_row_c = my_row < g.lq ? my_row : g.lq - 1;
    const uint16_t* k = static_cast<const uint16_t*>(a.k) + (long long)kvh * g.kv_stride_head;
    const uint16_t* v = static_cast<const uint16_t*>(a.v) + (long long)kvh * g.kv_stride_head;
    const uint16_t* qp = static_cast<const uint16_t*>(a.q) + (long long)my_row_c * g.q_stride_tok + (long long)h * g.q_stride_head + 8 * hh;
    bf16x8 qf[C::NKS];
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);

    const uint32_t lds = (uint32_t)(uintptr_t)(&sm.t[0][0][0]) + sp * C::NBUF * 2 * C::TILE_BYTES;
    const LaneAddr<C> la(lane, lds);
    const BlockFetch<C> fetch(lane, g.kv_stride_tok);
    // R = 1: the wavefront fetches K and V of its blocks; R = 2: one wavefront of a split K, the other V
    auto fetch_k = [&](int b, int buf) { if (R == 1 || rb == 0) fetch.issue(k, g.kv_stride_tok, b * TB, g.lc, lds + buf * 2 * C::TILE_BYTES); };
    auto fetch_v = [&](int b, int buf) { if (R == 1 || rb == 1) fetch.issue(v, g.kv_stride_tok, b * TB, g.lc, lds + buf * 2 * C::TILE_BYTES + C::TILE_BYTES); };

    // the first block is asked for before it is known that some row sees it
    if (sp * TB < g.lc) { fetch_k(sp, 0); fetch_v(sp, 0); }
    const Visible vis(g, row0, (wg_row0 + C::ROWS < g.lq ? wg_row0 + C::ROWS : g.lq) - 1, l32, hh);
    const int n_blocks = (vis.n_all + TB - 1) / TB;
    if (n_blocks == 0 && a.accumulate) {                   // merging an empty partial is the identity
        wait_transfers<0>();
        return;
    }

    f32x16 oacc[C::NDB];
#pragma unroll
    for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
    const float c_log2 = g.scale * LOG2E, inv_c_log2 = 1.0f / c_log2;
    float m_run = NEG_BIG, thr_raw = NEG_BIG;          // any finite score exceeds the threshold: the first one sets the maximum
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
        if (__any(mx > thr_raw)) {                     // running maximum, raised only when a block exceeds it by more than 2^8
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

#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) pin(qf[ks]);       // no wait for these inside the loop
    if constexpr (R == 1) {
        for (int b = sp; b < n_blocks; b += S) {
            const bool more = b + S < n_blocks;
            wait_transfers<C::XFERS>();                    // K has landed, V may still be in flight
            f32x16 s = row_product<C>(la, 0, [&](int ks) { return qf[ks]; });
            reads_done();
            if (more) fetch_k(b + S, 0);
            bf16x8 pf[2];
            softmax(s, b, pf);
            if (more) wait_transfers<C::XFERS>();
            else wait_transfers<0>();
            col_product<C, true>(oacc, la, C::TILE_BYTES, pf);
            reads_done();
            if (more) fetch_v(b + S, 0);
        }
    } else {
        const int n_steps = (n_blocks + S - 1) / S;        // the same for all wavefronts of the workgroup
        auto step = [&](auto bufc, int st) __attribute__((always_inline)) {
            constexpr int buf = decltype(bufc)::value;
            constexpr uint32_t tile = buf * 2 * C::TILE_BYTES;
            const int b = st * S + sp;
            wait_transfers<0>();
            wg_barrier();                                  // the step's blocks have landed, and everyone is done with the other buffer
            if (b + S < n_blocks) { fetch_k(b + S, buf ^ 1); fetch_v(b + S, buf ^ 1); }
            if (b < n_blocks) {
                f32x16 s = row_product<C>(la, tile, [&](int ks) { return qf[ks]; });
                bf16x8 pf[2];
                softmax(s, b, pf);
                col_product<C, true>(oacc, la, tile + C::TILE_BYTES, pf);
            }
            reads_done();
        };
        for (int st = 0; st < n_steps; st += 2) {          // two steps at a time: the buffer is a compile-time offset of the reads
            step(IC<0>{}, st);
            if (st + 1 < n_steps) step(IC<1>{}, st + 1);
        }
    }

    // combine the splits: weights per (row, split), merged with the running (o, lse), then a row-contiguous pass.
    // Wavefront s R + rb staged split s of row block rb: statistics of a row of the workgroup in split s at s ROWS + row.
    const float l_run = sum_across_halves((ps[0] + ps[1]) + (ps[2] + ps[3]));
    const float lr_run = sum_across_halves((psr[0] + psr[1]) + (psr[2] + psr[3]));
    wait_transfers<0>();                               // (a first block that no row sees)
    __syncthreads();                                   // every wavefront is done with its blocks
    stage_transposed<C>(&sm.e.stage[wave * TB * C::PITCH], oacc, l32, hh, 1.0f);
    if (hh == 0) { sm.e.m[wave * TB + l32] = m_run; sm.e.l[wave * TB + l32] = l_run; sm.e.lr[wave * TB + l32] = lr_run; }
    __syncthreads();
    if (tid < C::ROWS) {
        float m = NEG_BIG, l = 0.f, lr = 0.f, e[S];
#pragma unroll
        for (int s = 0; s < S; ++s) m = fmaxf(m, sm.e.m[s * C::ROWS + tid]);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            e[s] = fast_exp2(sm.e.m[s * C::ROWS + tid] - m);
            l += e[s] * sm.e.l[s * C::ROWS + tid];
            lr += e[s] * sm.e.lr[s * C::ROWS + tid];
        }
        float inv = 0.f, lse_new = -INFINITY, wa = 0.f;
        if (l > 0.f) {
            inv = lr > 0.f ? 1.0f / lr : 0.f;
            lse_new = (m + __log2f(l)) * LN2;
        }
        float wb = inv;
        if (wg_row0 + tid < g.lq) {
            float* lp = a.lse + (long long)h * g.lq + wg_row0 + tid;
            if (a.accumulate) {
                const float la_old = *lp;
                const float mm = fmaxf(la_old, lse_new);
                if (mm != -INFINITY) {
                    const float ea = __expf(la_old - mm), eb = __expf(lse_new - mm);
                    const float r = 1.0f / (ea + eb);
                    wa = ea * r;
                    wb = eb * r * inv;
                    lse_new = mm + __logf(ea + eb);
                }
            }
            *lp = lse_new;
        }
#pragma unroll
        for (int s = 0; s < S; ++s) sm.e.w[s * C::ROWS + tid] = e[s] * wb;
        sm.e.wa[tid] = wa;
    }
    __syncthreads();
    for (int i = tid; i < C::ROWS * D / 4; i += 64 * NW) {
        const int r = i / (D / 4), c = 4 * (i % (D / 4));
        if (wg_row0 + r >= g.lq) continue;
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s) x += sm.e.w[s * C::ROWS + r] * *reinterpret_cast<const f32x4*>(&sm.e.stage[(s * C::ROWS + r) * C::PITCH + c]);
        f32x4* op = reinterpret_cast<f32x4*>(a.o + ((long long)(wg_row0 + r) * g.nq + h) * D + c);
        if (a.accumulate) x += sm.e.wa[r] * *op;
        *op = x;
    }
}

// dQ: dP^T = V dO^T, S^T = K Q^T, dS^T = P^T (dP^T - Delta), dQ^T += K^T dS^T.
template <class C> union DqSmem {
    unsigned char t[C::S][C::NBUF][2 * C::TILE_BYTES];     // K and V block of each split
    float stage[C::STAGE_FLOATS];
};

template <int D, int R>
__device__ __forceinline__ void dq_unit(const BwdArgs& a, const int h, const int q_tile, DqSmem<SplitCfg<D, R>>& sm)
{
    using C = SplitCfg<D, R>;
    constexpr int S = C::S;
    const AttnGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave % R, sp = wave / R;
    const int l32 = lane & 31, hh = lane >> 5;
    const int wg_row0 = q_tile * C::ROWS, row0 = wg_row0 + TB * rb;
    const int kvh = arg_byte(g.kv_of_q, h);
    const int my_row = row0 + l32;
    const int my_row_c = my_row < g.lq ? my_row : g.lq - 1;
    const uint16_t* k = static_cast<const uint16_t*>(a.k) + (long long)kvh * g.kv_stride_head;
    const uint16_t* v = static_cast<const uint16_t*>(a.v) + (long long)kvh * g.kv_stride_head;
    bf16x8 qf[C::NKS], gf[C::NKS];
    const long long q_off = (long long)my_row_c * g.q_stride_tok + (long long)h * g.q_stride_head + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) {
        gf[ks] = *reinterpret_cast<const bf16x8*>(static_cast<const uint16_t*>(a.d_o) + q_off + 16 * ks);
        qf[ks] = *reinterpret_cast<const bf16x8*>(static_cast<const uint16_t*>(a.q) + q_off + 16 * ks);
    }
    const float lse = a.lse[(long long)h * g.lq + my_row_c];
    const float delta = a.delta[(long long)h * g.lq + my_row_c];

    const uint32_t lds = (uint32_t)(uintptr_t)(&sm.t[0][0][0]) + sp * C::NBUF * 2 * C::TILE_BYTES;
    const LaneAddr<C> la(lane, lds);
    const BlockFetch<C> fetch(lane, g.kv_stride_tok);
    auto fetch_k = [&](int b, int buf) { if (R == 1 || rb == 0) fetch.issue(k, g.kv_stride_tok, b * TB, g.lc, lds + buf * 2 * C::TILE_BYTES); };
    auto fetch_v = [&](int b, int buf) { if (R == 1 || rb == 1) fetch.issue(v, g.kv_stride_tok, b * TB, g.lc, lds + buf * 2 * C::TILE_BYTES + C::TILE_BYTES); };
    if (sp * TB < g.lc) { fetch_v(sp, 0); fetch_k(sp, 0); }
    const Visible vis(g, row0, (wg_row0 + C::ROWS < g.lq ? wg_row0 + C::ROWS : g.lq) - 1, l32, hh);
    const int n_blocks = (vis.n_all + TB - 1) / TB;
    if (n_blocks == 0) {                                   // dq_acc unchanged
        wait_transfers<0>();
        return;
    }

    const float c_log2 = g.scale * LOG2E;

    f32x16 dq[C::NDB];
#pragma unroll
    for (int db = 0; db < C::NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) dq[db][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < C::NKS; ++ks) { pin(gf[ks]); pin(qf[ks]); }
    const float neg_l = lse == -INFINITY ? -INFINITY : -lse * LOG2E;       // a row whose LSE is infinite has P = 0
    asm volatile("" ::"v"(neg_l), "v"(delta));

    // dQ^T += K^T dS^T of block b, whose K image is at byte `tile`
    auto accumulate = [&](const f32x16& s, const f32x16& dp, int b, uint32_t tile) __attribute__((always_inline)) {
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
        col_product<C, true>(dq, la, tile, hi);
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
                col_product<C, true>(dq, la, tile, part);
            }
        }
    };
    if constexpr (R == 1) {
        for (int b = sp; b < n_blocks; b += S) {
            const bool more = b + S < n_blocks;
            wait_transfers<C::XFERS>();                    // V has landed, K may still be in flight
            const f32x16 dp = row_product<C>(la, C::TILE_BYTES, [&](int ks) { return gf[ks]; });
            reads_done();
            wait_transfers<0>();
            if (more) fetch_v(b + S, 0);
            const f32x16 s = row_product<C>(la, 0, [&](int ks) { return qf[ks]; });
            accumulate(s, dp, b, 0);
            reads_done();
            if (more) fetch_k(b + S, 0);
        }
    } else {
        const int n_steps = (n_blocks + S - 1) / S;
        auto step = [&](auto bufc, int st) __attribute__((always_inline)) {
            constexpr int buf = decltype(bufc)::value;
            constexpr uint32_t tile = buf * 2 * C::TILE_BYTES;
            const int b = st * S + sp;
            wait_transfers<0>();
            wg_barrier();
            if (b + S < n_blocks) { fetch_v(b + S, buf ^ 1); fetch_k(b + S, buf ^ 1); }
            if (b < n_blocks) {
                const f32x16 dp = row_product<C>(la, tile + C::TILE_BYTES, [&](int ks) { return gf[ks]; });
                const f32x16 s = row_product<C>(la, tile, [&](int ks) { return qf[ks]; });
                accumulate(s, dp, b, tile);
            }
            reads_done();
        };
        for (int st = 0; st < n_steps; st += 2) {
            step(IC<0>{}, st);
            if (st + 1 < n_steps) step(IC<1>{}, st + 1);
        }
    }
    wait_transfers<0>();                                   // (a first block that no row sees)
    __syncthreads();
    stage_transposed<C>(&sm.stage[wave * TB * C::PITCH], dq, l32, hh, g.scale);
    __syncthreads();
    for (int i = tid; i < C::ROWS * D / 4; i += 64 * NW) {
        const int r = i / (D / 4), c = 4 * (i % (D / 4));
        if (wg_row0 + r >= g.lq) continue;
        f32x4 x = *reinterpret_cast<const f32x4*>(&sm.stage[r * C::PITCH + c]);
#pragma unroll
        for (int s = 1; s < S; ++s) x += *reinterpret_cast<const f32x4*>(&sm.stage[(s * C::ROWS + r) * C::PITCH + c]);
        f32x4* op = reinterpret_cast<f32x4*>(a.dq + ((long long)(wg_row0 + r) * g.nq + h) * D + c);
        *op += x;
    }
}

// dK / dV of 32 keys from the q rows of a run of heads: S = Q K^T, dP = dO V^T, dV += P^T dO, dK += dS^T Q.  The keys'
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
__device__ __forceinline__ void dkdv_unit(const BwdArgs& a, const HeadRuns& runs, const int run, const int kv_tile, DkdvSmem<SplitCfg<D, 1>>& sm)
{
    using C = SplitCfg<D, 1>;
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
    // K by wavefront 0, V by wavefront 1
    if (wave < 2) {
        const BlockFetch<C> kv_fetch(lane, g.kv_stride_tok);
        const uint16_t* src = static_cast<const uint16_t*>(wave ? a.v : a.k) + (long long)kvh * g.kv_stride_head;
        kv_fetch.issue(src, g.kv_stride_tok, col0, g.lc, __builtin_amdgcn_readfirstlane(lds_kv + wave * C::TILE_BYTES));
    }
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
    if (wave < 2) {
        // K / V were requested first: whatever is in flight behind them is this wavefront's first block
        if (left > 0) wait_transfers<2 * C::XFERS + 2>();
        else wait_transfers<0>();
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
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
        col_product<C, false>(dv, la, C::TILE_BYTES, pf);
        reads_done();
        if (more) fetch_g(h, next_row);
        col_product<C, false>(dk, la, 0, df);
        reads_done();
        if (more) fetch_q(h, next_row);
    }

    // lane holds column 32 db + l32; register r holds key 8 (r / 4) + 4 hh + r % 4
    auto write_out = [&](float* out, const f32x16 (&acc)[C::NDB], float w) {
        __syncthreads();
        float* st = &sm.stage[wave * TB * C::PITCH];
#pragma unroll
        for (int db = 0; db < C::NDB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st[(8 * (r >> 2) + 4 * hh + (r & 3)) * C::PITCH + 32 * db + l32] = acc[db][r] * w;
        __syncthreads();
        if (ATOMIC_DKV) {          // consecutive lanes on consecutive floats
            for (int i = tid; i < TB * D; i += 64 * NW) {
                const int r = i / D, c = i % D;
                if (col0 + r >= g.lc) continue;
                float x = sm.stage[r * C::PITCH + c];
#pragma unroll
                for (int s = 1; s < NW; ++s) x += sm.stage[(s * TB + r) * C::PITCH + c];
                global_atomic_add(out + ((long long)(col0 + r) * g.nkv + kvh) * D + c, x);
            }
        } else {
            for (int i = tid; i < TB * D / 4; i += 64 * NW) {
                const int r = i / (D / 4), c = 4 * (i % (D / 4));
                if (col0 + r >= g.lc) continue;
                f32x4 x = *reinterpret_cast<const f32x4*>(&sm.stage[r * C::PITCH + c]);
#pragma unroll
                for (int s = 1; s < NW; ++s) x += *reinterpret_cast<const f32x4*>(&sm.stage[(s * TB + r) * C::PITCH + c]);
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
// others dQ units of 32 R rows.  Within each, heads (runs) side by side and the longest tiles first.
template <int D, int R, bool ATOMIC_DKV>
__global__ void __launch_bounds__(512) bwd_split_bf16_kernel(const BwdArgs a, const HeadRuns runs, const unsigned n_dkdv, const int n_q_tiles)
{
    __shared__ __attribute__((aligned(1024))) union { DkdvSmem<SplitCfg<D, 1>> dkdv; DqSmem<SplitCfg<D, R>> dq; } sm;
    if (blockIdx.x < n_dkdv) {
        const int tile = uniform((int)(blockIdx.x / (unsigned)runs.n));
        dkdv_unit<D, ATOMIC_DKV>(a, runs, (int)blockIdx.x - tile * runs.n, tile, sm.dkdv);
    } else {
        const unsigned unit = blockIdx.x - n_dkdv;
        const int tile = uniform((int)(unit / (unsigned)a.g.nq));
        dq_unit<D, R>(a, (int)unit - tile * a.g.nq, n_q_tiles - 1 - tile, sm.dq);
    }
}

}  // namespace

hipError_t hexi_launch_fwd_split_bf16(const FwdArgs& a, int rows, hipStream_t s)
{
    const int n_q_tiles = (a.g.lq + rows - 1) / rows;
    const dim3 grid((unsigned)a.g.nq, (unsigned)n_q_tiles);
    if (a.g.d == 128 && rows == 32) fwd_split_bf16_kernel<128, 1><<<grid, 512, 0, s>>>(a, n_q_tiles);
    else if (a.g.d == 128 && rows == 64) fwd_split_bf16_kernel<128, 2><<<grid, 512, 0, s>>>(a, n_q_tiles);
    else if (a.g.d == 64 && rows == 32) fwd_split_bf16_kernel<64, 1><<<grid, 512, 0, s>>>(a, n_q_tiles);
    else if (a.g.d == 64 && rows == 64) fwd_split_bf16_kernel<64, 2><<<grid, 512, 0, s>>>(a, n_q_tiles);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// dq_rows: rows per dQ workgroup (32 or 64; 0: no dQ); runs: the head runs of the dK / dV workgroups (none: no dK / dV)
hipError_t hexi_launch_bwd_split_bf16(const BwdArgs& a, int dq_rows, const HeadRuns& runs, bool shared, hipStream_t s)
{
    const int n_q_tiles = dq_rows > 0 ? (a.g.lq + dq_rows - 1) / dq_rows : 0;
    const unsigned n_dkdv = (unsigned)((a.g.lc + TB - 1) / TB) * (unsigned)runs.n;
    const unsigned grid = n_dkdv + (unsigned)n_q_tiles * (unsigned)a.g.nq;
    if (grid == 0) return hipSuccess;
    auto launch = [&](auto d, auto r) {
        constexpr int D = decltype(d)::value, R = decltype(r)::value;
        if (shared) bwd_split_bf16_kernel<D, R, true><<<grid, 512, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
        else bwd_split_bf16_kernel<D, R, false><<<grid, 512, 0, s>>>(a, runs, n_dkdv, n_q_tiles);
        return hipGetLastError();
    };
    if (a.g.d == 128) return dq_rows == 64 ? launch(IC<128>{}, IC<2>{}) : launch(IC<128>{}, IC<1>{});
    if (a.g.d == 64) return dq_rows == 64 ? launch(IC<64>{}, IC<2>{}) : launch(IC<64>{}, IC<1>{});
    return hipErrorInvalidValue;
}

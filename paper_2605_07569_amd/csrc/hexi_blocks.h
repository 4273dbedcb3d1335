// Pieces shared by the bf16 kernels whose wavefronts stream 32-row blocks through a private part of LDS (hexi_bf16_split.hip,
// hexi_bf16_quad.hip).  A block's LDS image is [32][D] bf16 with the 16-byte pieces of a row permuted by piece ^ swz(row), which makes
// the 128-bit row reads (16 rows, one piece) and the transposed 64-bit reads (4 rows x 64 bytes) both touch all 64 banks once.
#pragma once
#include <cstddef>
#include "hexi_internal.h"
#include "hexi_mfma.h"

namespace {

constexpr int TB = 32;         // rows of a block, stationary or streamed
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float NEG_BIG = -1.0e30f;        // finite stand-in for "no key seen yet"
constexpr float RESCALE_SLACK = 8.0f;

// a value that is the same in all lanes, in a scalar register
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// A block of one tensor.
template <int D_> struct BlockCfg {
    static constexpr int D = D_;
    static_assert(D == 64 || D == 128, "head_dim 64 or 128");
    static constexpr int NKS = D / 16;                     // 16-wide contraction steps across the head dimension
    static constexpr int NDB = D / 32;                     // 32-column blocks of an output
    static constexpr int ROW_BYTES = 2 * D, PIECES = D / 8;
    static constexpr int TILE_BYTES = TB * ROW_BYTES;      // 8 or 4 KB
    static constexpr int XFERS = TILE_BYTES / 1024;        // wave-wide transfers per block: 8 or 4
    static constexpr int PITCH = D + 4;                    // floats per staged output row
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

// Workgroup barrier behind which LDS holds what the other wavefronts put there before it (after their own waits).
__device__ __forceinline__ void block_barrier()
{
    wg_barrier();
    asm volatile("" ::: "memory");
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
    // transfer i of a block all of whose rows exist; `base`: the block's first row
    __device__ __forceinline__ void one(const uint16_t* base, long long stride_tok, uint32_t lds, int i) const
    {
        lds_dma16_base(base + (long long)(i / HALF * 16) * stride_tok, off[i % HALF], __builtin_amdgcn_readfirstlane(lds + i * 1024));
    }
    // rows [row0, row0 + 32) of `src`; rows past `total` re-read the last one (row0 < total)
    __device__ __forceinline__ void issue(const uint16_t* src, long long stride_tok, int row0, int total, uint32_t lds) const
    {
        const uint16_t* base = src + (long long)row0 * stride_tok;
        if (row0 + TB <= total) {
#pragma unroll
            for (int i = 0; i < C::XFERS; ++i) one(base, stride_tok, lds, i);
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

// The stationary rows of a workgroup, ROWS x D from row0 on, into LDS as blocks, shared out over its wavefronts; rows past `total`
// repeat the last one.  (Read by every wavefront for itself, their fragments are the slowest part of a short unit's start: a load
// of 16 bytes of each of 32 rows takes the memory path as long as four whole-row ones.)
template <class C, int ROWS, int NWAVES> __device__ __forceinline__ void fetch_rows(const uint16_t* src, long long stride_tok, int row0, int total, uint32_t lds, int wave, int lane)
{
    constexpr int N = ROWS / TB * C::XFERS, RPX = 1024 / C::ROW_BYTES;       // transfers, rows per transfer
    const int first = row0 < total ? row0 : total - 1;
    const uint16_t* base = src + (long long)first * stride_tok;
#pragma unroll
    for (int j = 0; j < (N + NWAVES - 1) / NWAVES; ++j) {
        const int x = NWAVES * j + wave;
        if (N % NWAVES != 0 && x >= N) break;
        const int r = x * RPX + lane / C::PIECES, row = row0 + r;
        lds_dma16_base(base, 2u * (uint32_t)(((row < total ? row : total - 1) - first) * (int)stride_tok) + 16u * (uint32_t)((lane % C::PIECES) ^ C::swz(r)),
                       __builtin_amdgcn_readfirstlane(lds + x * 1024));
    }
}

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

// The same addresses from two registers: they differ from each other in bits that no carry crosses (a block starts at a multiple of
// 1 KB), so one exclusive or in front of a read replaces a register kept through the loop.
template <class C> struct LaneXor {
    uint32_t row0, tr0;
    __device__ __forceinline__ LaneXor(int lane, uint32_t base)
    {
        const int l32 = lane & 31, hh = lane >> 5, grp2 = (lane >> 4) & 1, j16 = lane & 15, r = 4 * hh + (j16 >> 2);
        row0 = base + (uint32_t)(l32 * C::ROW_BYTES + 16 * (hh ^ C::swz(l32)));
        tr0 = base + (uint32_t)(r * C::ROW_BYTES + 16 * ((2 * grp2 + ((j16 & 3) >> 1)) ^ C::swz(r)) + 8 * (j16 & 1));
    }
    __device__ __forceinline__ void here() { asm volatile("" : "+v"(row0), "+v"(tr0)); }     // what follows is computed where it stands
    __device__ __forceinline__ bf16x8 read_row(int ks, uint32_t tile) const { return lds_b128((row0 ^ (32u * ks)) + tile); }
    // rows 16 u .. + 15, columns 32 db .. + 31 of the block at `tile`, transposed
    __device__ __forceinline__ bf16x8 read_tr(int u, int db, uint32_t tile) const
    {
        const uint32_t o = tile + (uint32_t)(u * 16 * C::ROW_BYTES);
        return lds_tr((tr0 ^ (64u * db)) + o, (tr0 ^ (64u * db + 32u)) + (o + 8 * C::ROW_BYTES));
    }
};

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

}  // namespace

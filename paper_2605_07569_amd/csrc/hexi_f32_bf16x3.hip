// fp32 attention with its products on the bf16 matrix instructions: every fp32 operand is cut into three bf16 values whose sum it is exactly (24 bits
// in 8 + 8 + 8), and the six largest of the nine products of two cut operands are added up in fp32.  A bf16 product is exact in fp32; the three left out are up
// to 2^-22 of the whole one (2^-25.4 rms), of either sign.  v_mfma_f32_32x32x16_bf16 keeps denormals and rounds its sums without bias (0.41 ulp rms
// over random operands, v_mfma_f32_16x16x4_f32 0.54) and once in 16 products instead of 4, so the results are no further from fp64 than those of
// the fp32 instruction (hexi_f32.hip): relative errors of o, dq, dk, dv at 4096 rows x 4096 keys x 16/4 heads x 128 1.2e-6, 1.4e-6, 2.4e-6, 2.4e-6 with
// it alone, 5e-7, 7e-7, 5e-7, 5e-7 here; over 250 random steps of 64 to 16000 keys, K scaled by 1 and by 3, no output is further off.
// Six bf16 products cost 6 / 16 of the fp32 one.  What bounds these kernels then: where 64-row units fill the chip, the forward and dQ execute 1.1 PFLOP/s
// in bf16, at the power limit (1.95 GHz, matrix pipes 53 % busy; a library product of 8192 x 8192 x 8192 on random bf16 operands reaches 1.16 on
// the same card); dK / dV the cutting of four streamed operands for two, 11.2 vector instructions to a matrix one, 0.9; shorter launches the length
// of their units (28 to 34 % busy).  us, 4096 x 4096 x 16/4 heads x 128, all keys visible, hexi_f32.hip / here: forward 1139 / 759, dQ 1559 / 1095, dK / dV
// 2367 / 1960; 4096 diagonal x 8 heads x 64, forward and backward: 168 / 121, 496 / 404.
//
// Shape.  Cutting costs 5.5 vector operations per element, and a vector operation beside a saturated matrix pipe takes 6 cycles (10 for the packing
// ones) next to 32x32x16 and 8.5 (13) next to 16x16x32; v_dot2_f32_bf16, which would subtract a packed value in one operation, waits for the
// matrix pipe (37 cycles).  So the 32x32x16 form throughout, operands cut once where they can be: a workgroup's 32 or 64 stationary rows (q rows, or
// keys for dK / dV) are cut at its start and their operands kept in LDS; 4 wavefronts, one per SIMD with its 512 registers, split the
// streamed rows in blocks of 32, each through a slot of its own without any barrier, and combine their results through LDS at the end.  Per
// block the rows arrive twice: by transfers into the slot for the scores, and as columns straight into registers for the accumulation
// (a column of 32 rows is what neighbouring lanes read together; rows of 64 lanes read directly cost a cycle per lane, 64 instead of 16).  The
// cutting of a step stands between the matrix instructions of the step before, and a slot is asked for again before the products of the last step (dQ 1 to 3 %).  8 wavefronts, two per SIMD, with 16x16x32 products: 926 us forward;
// 64 rows against 32: 757 / 930.
//
// Values.  A cut loses bits of a value below 2^-110 (2^-133 is the smallest bf16: up to 2^-134 of it), an infinite one has no rest (inf - inf), and the
// probabilities of the forward, up to 2^8 here, may overflow in a sum that would not.  A unit therefore looks its operands and results over
// (largest(), stationary_range(), Extremes) and, where the cut may show in a result, hands its rows to the units on the fp32 instruction
// (hexi_f32_units.h) before anything is written: values, infinities and NaN come out as there.  For the results that are kept it costs the
// forward one v_maximum3_f32 for two values of V and the backward one for two of dS, less than the sums that need no care for NaN any more give back: 3056
// rows x 12011 keys x 6/2 heads x 128, forward and backward, 2334 / 2335 us without / with it, 90 random backward steps 0.999.  A step that is all NaN
// takes three times as long.
#include "hexi_internal.h"
#include "hexi_mfma.h"
#include "hexi_shapes.h"
#include "hexi_f32_common.h"
#include "hexi_f32_units.h"

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// scale * log2(e) as two floats, the lower one positive: s * lo then has the sign of s, and a score of -inf gives 2^-inf without further care.
struct Log2Scale {
    float hi, lo;
    __device__ __forceinline__ explicit Log2Scale(float scale)
    {
        hi = scale * LOG2E_HI;
        lo = fmaf(scale, LOG2E_HI, -hi) + scale * LOG2E_LO;
        if (lo <= 0.f) {
            hi = __uint_as_float(__float_as_uint(hi) - 1u);
            lo = fmaf(scale, LOG2E_HI, -hi) + scale * LOG2E_LO;
        }
        lo = fmaxf(lo, 1.17549435e-38f);
    }
};

template <int D_, int NB_> struct X3Cfg {
    static constexpr int D = D_;
    static_assert(D == 64 || D == 128, "head_dim 64 or 128");
    static constexpr int NW = 4;                       // wavefronts, one per SIMD, which split the streamed rows
    static constexpr int NB = NB_, ROWS = 32 * NB;     // stationary rows of a workgroup: 32 or 64
    static constexpr int BLK = 32;                     // streamed rows of a block
    static constexpr int NK = D / 16;                  // contraction steps of a score
    static constexpr int NJ = D / 32;                  // columns of a lane in an accumulation, and accumulators of 32 columns
    static constexpr int ROW_BYTES = 4 * D, BLOCK_BYTES = BLK * ROW_BYTES;
    static constexpr int XFERS = BLOCK_BYTES / 1024;   // transfers of a block into LDS
    static constexpr int PIECES = NK * NB * 3 * 1024;  // bytes of a stationary tensor's operands in LDS
    static constexpr int PITCH = D + 4;                // floats per staged output row
    static constexpr int STAGE_FLOATS = NW * ROWS * PITCH;
};

// The three bf16 operands of eight values: x = h + m + l exactly.  h holds the upper 16 bits of x (cut, so that no finite x becomes infinite), m
// the rounded rest, l what is left of it.
struct Split3 { bf16x8 h, m, l; };
__device__ __forceinline__ unsigned pack_rounded(float a, float b)
{
    const bf16x2 t = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(unsigned, t);
}
__device__ __forceinline__ Split3 split8(float x0, float x1, float x2, float x3, float x4, float x5, float x6, float x7)
{
    const float x[8] = {x0, x1, x2, x3, x4, x5, x6, x7};
    u32x4 h, m, l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
        h[i] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
        a -= __uint_as_float(__float_as_uint(a) & 0xffff0000u);
        b -= __uint_as_float(__float_as_uint(b) & 0xffff0000u);
        m[i] = pack_rounded(a, b);
        a -= __uint_as_float(m[i] << 16);
        b -= __uint_as_float(m[i] & 0xffff0000u);
        l[i] = pack_rounded(a, b);
    }
    return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}
__device__ __forceinline__ Split3 split8(const f32x4& a, const f32x4& b) { return split8(a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]); }

// max(m, |a|, |b|), NaN if one of them is
__device__ __forceinline__ float largest(float m, float a, float b) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_fabsf(a), __builtin_fabsf(b)), m); }
// over the lanes of the wavefront
__device__ __forceinline__ float largest_of_wave(float x)
{
    auto rotated = [&](auto by) { return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + decltype(by)::value, 0xf, 0xf, false)); };
    x = largest(x, x, rotated(IC<8>{}));
    x = largest(x, x, rotated(IC<4>{}));
    x = largest(x, x, rotated(IC<2>{}));
    x = largest(x, x, rotated(IC<1>{}));
    const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = largest(0.f, __uint_as_float(rows[0]), __uint_as_float(rows[1]));
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return largest(0.f, __uint_as_float(halves[0]), __uint_as_float(halves[1]));
}

// The largest of the wavefronts' values, which they have put into a row of `top`.
template <int NW> __device__ __forceinline__ float largest_of_workgroup(const float (&top)[NW])
{
    float m = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) m = __builtin_elementwise_maximum(m, top[w]);
    return m;
}

// What a unit's results depend on besides the products themselves.  Stationary values are to be zero or within [2^-100, 2^60): their cuts lose
// nothing, and what the cuts of streamed values lose moves a score (in units of log2, scale below 2^20) by 2^-127 2^60 2^21 at most.  Then a sum of n products p v is off by
// n 2^-134 (max p + max v) besides its roundings, and p itself, a dS, by 2^-127 max s with s the stationary values of dP: nothing that 24 bits of
// the result show if it is zero or not below 2^24 times that.  The backward takes P and dS times 2^40, which lose nothing then, so that max v need not be
// known (in the second term it is taken for 2^10); dS that are all below what dP loses, or below 2^-100, are too small.
constexpr float SMALLEST = 7.88860905e-31f;                            // 2^-100
constexpr float CUT_LOSS = 7.70371978e-34f, SCORE_LOSS = 9.86076132e-32f;      // 2^24 2^-134, 2^24 2^-127
constexpr float UP = 1099511627776.f, DOWN = 1.f / UP;                 // 2^40
__device__ __forceinline__ unsigned scale_out_of_range(float x) { return (unsigned)!(x < 1048576.f) | (unsigned)!(x > 1e-18f); }      // (its product with DOWN is no denormal)
__device__ __forceinline__ unsigned too_small(float largest_value) { return (unsigned)(largest_value > 0.f) & (unsigned)(largest_value < SMALLEST); }
__device__ __forceinline__ unsigned ds_too_small(float ds_up, float s)
{
    return (unsigned)(ds_up > 0.f) & ((unsigned)(ds_up < SMALLEST * UP) | (unsigned)(ds_up < SCORE_LOSS * UP * s));
}

// Results: their largest magnitude and the smallest that is not zero, as its bits without the sign, less one.
struct Extremes {
    float top = 0.f;
    unsigned low = 0xffffffffu;
    __device__ __forceinline__ static unsigned bits(float x) { return (__float_as_uint(x) << 1) - 1u; }
    __device__ __forceinline__ void add(float a, float b)
    {
        top = largest(top, a, b);
        low = min(low, min(bits(a), bits(b)));
    }
    __device__ __forceinline__ unsigned not_finite_or_below(float least) const
    {
        return (unsigned)!(top < INFINITY) | (unsigned)(low < bits(largest(1.4e-45f, least, least)));      // (a limit that underflows is the smallest value)
    }
};
// Whether any thread of the workgroup finds its values so; votes: a word of LDS for each wavefront.
template <int NW> __device__ __forceinline__ bool any_of_workgroup(unsigned x, unsigned* votes, int tid)
{
    const unsigned any = __any(x != 0u);
    if ((tid & 63) == 0) votes[tid >> 6] = any;
    __syncthreads();
    unsigned sum = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) sum |= votes[w];
    return sum != 0u;
}

// Operands of a stationary tensor in LDS: step ks, row block n, piece p at ((NB ks + n) 3 + p) KB, a lane's 16 bytes at 16 lane.
template <class C> __device__ __forceinline__ void put_stationary(unsigned char* lds, const float* src, long long stride_tok, int row0, int total, int wave, int lane)
{
#pragma unroll
    for (int i = 0; i < C::NK * C::NB / C::NW; ++i) {
        const int c = wave + C::NW * i, ks = c / C::NB, row = row0 + 32 * (c % C::NB) + (lane & 31);
        const float* p = src + (long long)(row < total ? row : total - 1) * stride_tok + 16 * ks + 8 * (lane >> 5);
        const Split3 s = split8(*reinterpret_cast<const f32x4*>(p), *reinterpret_cast<const f32x4*>(p + 4));
        unsigned char* d = lds + c * 3072 + 16 * lane;
        *reinterpret_cast<bf16x8*>(d) = s.h;
        *reinterpret_cast<bf16x8*>(d + 1024) = s.m;
        *reinterpret_cast<bf16x8*>(d + 2048) = s.l;
    }
}

// The upper pieces that put_stationary() left there: sets `odd` where a value is out of range, and returns a bound of the thread's share of them.
template <class C> __device__ __forceinline__ float stationary_range(const unsigned char* lds, int wave, int lane, unsigned& odd)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    u16x2 low = 0xffff, high = 0;                         // smallest nonzero one (less one), largest: upper 16 bits, without sign
#pragma unroll
    for (int i = 0; i < C::NK * C::NB / C::NW; ++i) {
        const u32x4 h = *reinterpret_cast<const u32x4*>(lds + (wave + C::NW * i) * 3072 + 16 * lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const u16x2 u = __builtin_bit_cast(u16x2, h[e] & 0x7fff7fffu), one = 1;
            low = __builtin_elementwise_min(low, (u16x2)(u - one));
            high = __builtin_elementwise_max(high, u);
        }
    }
    const unsigned l = min(low[0], low[1]), m = max(high[0], high[1]);
    odd |= (unsigned)(l < 0x0d80u - 1u) | (unsigned)(m >= 0x5d80u);         // 2^-100, 2^60
    return __uint_as_float((m + 1u) << 16);
}

// A block of 32 streamed rows on its way to the scores: transfers into the wavefront's own piece of LDS, the 16-byte pieces of a row permuted by
// piece ^ (row & 15), so that the reads of 16 rows' pieces meet all banks once.
template <class C> struct RowBlock {
    uint32_t slot, src[C::XFERS], rd[4];
    __device__ __forceinline__ static int row_of(int i, int lane) { return (1024 * i + 16 * lane) / C::ROW_BYTES; }
    __device__ __forceinline__ RowBlock(const unsigned char* lds, int lane, long long stride_tok)
    {
        slot = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);
#pragma unroll
        for (int i = 0; i < C::XFERS; ++i) {
            const int r = row_of(i, lane), p = (1024 * i + 16 * lane) % C::ROW_BYTES / 16;
            src[i] = 4u * (uint32_t)(r * (int)stride_tok) + 16u * (uint32_t)(p ^ (r & 15));
        }
        // piece 4 ks + 2 hh + i of row l: steps ks and ks + 4 are 256 bytes apart
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) rd[ks] = (uint32_t)((lane & 31) * C::ROW_BYTES + 16 * ((4 * ks + 2 * (lane >> 5)) ^ (lane & 15)));
    }
    // rows past `total` re-read the last one
    __device__ __forceinline__ void request(const float* base, long long stride_tok, int row0, int total, int lane) const
    {
        const float* b = base + (long long)row0 * stride_tok;
        if (row0 + C::BLK <= total) {
#pragma unroll
            for (int i = 0; i < C::XFERS; ++i) lds_dma16_base(b, src[i], slot + 1024 * i);
        } else {
#pragma unroll
            for (int i = 0; i < C::XFERS; ++i) {
                uint32_t o = src[i];
                const int r = row_of(i, lane);
                if (row0 + r >= total) o -= 4u * (uint32_t)((row0 + r - (total - 1)) * (int)stride_tok);
                lds_dma16_base(b, o, slot + 1024 * i);
            }
        }
    }
    // columns 16 ks + 8 hh .. + 7 of row l
    __device__ __forceinline__ void read(f32x4 (&x)[2], const unsigned char* lds, int ks) const
    {
        x[0] = *reinterpret_cast<const f32x4*>(lds + rd[ks & 3] + 256 * (ks >> 2));
        x[1] = *reinterpret_cast<const f32x4*>(lds + (rd[ks & 3] ^ 16u) + 256 * (ks >> 2));
    }
};
template <int YOUNGER> __device__ __forceinline__ void landed()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(YOUNGER) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// 32 streamed rows as the other operand of an accumulation over them: lane (hh, c) holds columns NJ c .. of rows 16 u + 8 (e / 4) + 4 hh + e % 4.
template <class C> struct ColBlock {
    typedef float vec __attribute__((ext_vector_type(C::NJ)));
    vec x[2][8];
    __device__ __forceinline__ void load(const float* src, long long stride_tok, int row0, int total, int hh, int c)
    {
        const char* base = reinterpret_cast<const char*>(src + (long long)row0 * stride_tok);
        const uint32_t step = 4u * (uint32_t)stride_tok;
        const uint32_t lane_off = 4u * (uint32_t)(C::NJ * c);
        if (row0 + C::BLK <= total) {
            const uint32_t off = 4u * step * (uint32_t)hh + lane_off;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) x[u][e] = *reinterpret_cast<const vec*>(base + (size_t)((16 * u + 8 * (e / 4) + e % 4) * step) + off);
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int r = 16 * u + 8 * (e / 4) + 4 * hh + e % 4, rc = row0 + r < total ? r : total - 1 - row0;
                    x[u][e] = *reinterpret_cast<const vec*>(base + ((uint32_t)rc * step + lane_off));
                }
        }
    }
    template <bool TOP> __device__ __forceinline__ Split3 split(int u, int j, float& top) const      // TOP: top is their largest magnitude so far
    {
#pragma unroll
        for (int e = 0; e < 8 && TOP; e += 2) top = largest(top, x[u][e][j], x[u][e + 1][j]);
        return split8(x[u][0][j], x[u][1][j], x[u][2][j], x[u][3][j], x[u][4][j], x[u][5][j], x[u][6][j], x[u][7][j]);
    }
};

__device__ __forceinline__ float probability(float s, const Log2Scale& c, float nl_hi, float nl_lo) { return fast_exp2(fmaf(s, c.hi, nl_hi) + fmaf(s, c.lo, nl_lo)); }

// one MFMA, then vector work of the next step in its shadow
template <int N, int V, int DS> __device__ __forceinline__ void interleave()
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        HEXI_SCHED_MFMA(1);
        HEXI_SCHED_VALU(V);
        if (DS) HEXI_SCHED_DSREAD(DS);
    }
}

// s[n], register 4 b + t: streamed row 8 b + 4 hh + t times stationary row 32 n + l; slot_free() once the block has been read, before the products of the
// last step.
template <class C, class F> __device__ __forceinline__ void scores(f32x16 (&s)[C::NB], const RowBlock<C>& rows, const unsigned char* slot, const unsigned char* stat, F&& slot_free)
{
    constexpr int NB = C::NB;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    f32x16 lo[NB];
    f32x4 raw[2];
    bf16x8 b[2][NB][3];
    auto read_stat = [&](int ks) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int p = 0; p < 3; ++p) b[ks & 1][n][p] = *reinterpret_cast<const bf16x8*>(stat + (NB * ks + n) * 3072 + 1024 * p);
    };
    rows.read(raw, slot, 0);
    read_stat(0);
    Split3 t = split8(raw[0], raw[1]);
    rows.read(raw, slot, 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < C::NK; ++ks) {
        Split3 next = t;
        if (ks + 1 < C::NK) {
            read_stat(ks + 1);
            next = split8(raw[0], raw[1]);
            if (ks + 2 < C::NK) rows.read(raw, slot, ks + 2);
        } else {
            reads_done();
            slot_free();
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const bf16x8 (&q)[3] = b[ks & 1][n];
            s[n] = mfma32(t.h, q[0], ks == 0 ? zero : s[n]);
            lo[n] = mfma32(t.h, q[1], ks == 0 ? zero : lo[n]);
        }
#pragma unroll
        for (int n = 0; n < NB; ++n) lo[n] = mfma32(t.h, b[ks & 1][n][2], lo[n]);
#pragma unroll
        for (int n = 0; n < NB; ++n) lo[n] = mfma32(t.m, b[ks & 1][n][0], lo[n]);
#pragma unroll
        for (int n = 0; n < NB; ++n) lo[n] = mfma32(t.m, b[ks & 1][n][1], lo[n]);
#pragma unroll
        for (int n = 0; n < NB; ++n) lo[n] = mfma32(t.l, b[ks & 1][n][0], lo[n]);
        interleave<6 * NB, 8 / NB, 1>();
        __builtin_amdgcn_sched_barrier(0);
        t = next;
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) s[n] += lo[n];
}

// acc[n][j], register 4 b + t: column NJ (8 b + 4 hh + t) + j of stationary row 32 n + l; p[n]: probabilities or dS as scores() leaves its results.
// APART: the block's sum by itself, then added, for dK / dV and for long chains of the others: one rounding of the running value in 32 rows instead of 12.
// Against the fp32 instruction, error without / with it: dv of 3643 rows of 4 heads 1.1 / 0.43, o of 12000 keys x 128 columns 1.13 / 0.37, of 5000 keys
// x 64 1.06 / 0.4.  A backward is 4 % slower with it in dK / dV, a forward 5 %.
template <class C, bool APART, bool TOP> __device__ __forceinline__ void accumulate(f32x16 (&acc)[C::NB][C::NJ], const ColBlock<C>& v, const f32x16 (&p)[C::NB], float& top)
{
    constexpr int NB = C::NB;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    Split3 po[2][NB];
    auto split_p = [&](int u) {
#pragma unroll
        for (int n = 0; n < NB; ++n)
            po[u][n] = split8(p[n][8 * u], p[n][8 * u + 1], p[n][8 * u + 2], p[n][8 * u + 3], p[n][8 * u + 4], p[n][8 * u + 5], p[n][8 * u + 6], p[n][8 * u + 7]);
    };
    split_p(0);
    if (APART) split_p(1);
    Split3 t = v.template split<TOP>(0, 0, top);
    f32x16 sum[NB];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int st = 0; st < 2 * C::NJ; ++st) {
        const int u = APART ? st % 2 : st / C::NJ, j = APART ? st / 2 : st % C::NJ, st1 = st + 1;
        Split3 next = t;
        if (st1 < 2 * C::NJ) next = v.template split<TOP>(APART ? st1 % 2 : st1 / C::NJ, APART ? st1 / 2 : st1 % C::NJ, top);
        f32x16* to[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) to[n] = APART ? &sum[n] : &acc[n][j];
#pragma unroll
        for (int n = 0; n < NB; ++n) *to[n] = mfma32(t.l, po[u][n].h, APART && u == 0 ? zero : *to[n]);
#pragma unroll
        for (int n = 0; n < NB; ++n) *to[n] = mfma32(t.h, po[u][n].l, *to[n]);
#pragma unroll
        for (int n = 0; n < NB; ++n) *to[n] = mfma32(t.m, po[u][n].m, *to[n]);
#pragma unroll
        for (int n = 0; n < NB; ++n) *to[n] = mfma32(t.m, po[u][n].h, *to[n]);
#pragma unroll
        for (int n = 0; n < NB; ++n) *to[n] = mfma32(t.h, po[u][n].m, *to[n]);
#pragma unroll
        for (int n = 0; n < NB; ++n) *to[n] = mfma32(t.h, po[u][n].h, *to[n]);
        interleave<6 * NB, 8 / NB, 0>();
        __builtin_amdgcn_sched_barrier(0);
        t = next;
        if (APART && u == 1) {
#pragma unroll
            for (int n = 0; n < NB; ++n) acc[n][j] += sum[n];
        }
        if (!APART && j == C::NJ - 1 && u == 0) { split_p(1); __builtin_amdgcn_sched_barrier(0); }
    }
}

template <class C> __device__ __forceinline__ void zero_acc(f32x16 (&acc)[C::NB][C::NJ])
{
#pragma unroll
    for (int n = 0; n < C::NB; ++n)
#pragma unroll
        for (int i = 0; i < C::NJ; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[n][i][r] = 0.f;
}

// The wavefront's ROWS x D block, times w, as rows of a staging area.
template <class C> __device__ __forceinline__ void stage_rows(float* stage, const f32x16 (&acc)[C::NB][C::NJ], int lane, float w)
{
    const int hh = lane >> 5;
#pragma unroll
    for (int n = 0; n < C::NB; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            typename ColBlock<C>::vec x;
#pragma unroll
            for (int j = 0; j < C::NJ; ++j) x[j] = acc[n][j][r] * w;
            *reinterpret_cast<typename ColBlock<C>::vec*>(&stage[(32 * n + (lane & 31)) * C::PITCH + C::NJ * (8 * (r / 4) + 4 * hh + r % 4)]) = x;
        }
}

template <class C> union X3FwdSmem {
    struct { unsigned char q[C::PIECES], rows[C::NW][C::BLOCK_BYTES]; } t;
    struct { float stage[C::STAGE_FLOATS], m[C::NW * C::ROWS], l[C::NW * C::ROWS], w[C::NW * C::ROWS], wa[C::ROWS], top[C::NW]; unsigned votes[C::NW]; } e;
};

// One thread per row of a workgroup whose streamed rows were split S ways: the weights of the splits (references, in units of log2, at
// ref_of[split * ROWS + row], sums at l_of) and of the running o; returns the row's new LSE.
template <int ROWS, int S> __device__ __forceinline__ float combine_rows(const FwdArgs& a, int h, int row0, int tid, const float* ref_of, const float* l_of, float* w_of, float* wa_of)
{
    float m = -INFINITY, l = 0.f, e[S];
#pragma unroll
    for (int s = 0; s < S; ++s) m = l_of[s * ROWS + tid] == 0.f ? m : fmaxf(m, ref_of[s * ROWS + tid]);      // (a split that saw nothing of the row has no reference)
#pragma unroll
    for (int s = 0; s < S; ++s) {
        e[s] = l_of[s * ROWS + tid] == 0.f ? 0.f : fast_exp2(ref_of[s * ROWS + tid] - m);
        l += e[s] * l_of[s * ROWS + tid];
    }
    // the sum is up to 2^8 times that of an exact maximum, and its logarithm would lose those bits: in fp64, over the mantissa alone
    float lse_part = -INFINITY;
    if (l > 0.f) {
        int ex;
        const float f = __builtin_frexpf(l, &ex);
        lse_part = (float)(((double)m + (double)ex) * 0.6931471805599453 + (double)logf(f));
    }
    float wb = l > 0.f ? 1.0f / l : 0.f, wa = 0.f, lse_new = lse_part;
    const int row = row0 + tid;
    if (row < a.g.lq) {
        if (a.accumulate) {
            const float la_old = a.lse[(long long)h * a.g.lq + row];
            const float mm = fmaxf(la_old, lse_part);
            if (mm == -INFINITY) { wb = 0.f; lse_new = -INFINITY; }
            else {
                const float ea = expf(la_old - mm), eb = expf(lse_part - mm), inv = 1.0f / (ea + eb);
                wa = ea * inv;
                wb *= eb * inv;
                lse_new = mm + logf(ea + eb);
            }
        }
    }
#pragma unroll
    for (int s = 0; s < S; ++s) w_of[s * ROWS + tid] = e[s] * wb;
    wa_of[tid] = wa;
    return lse_new;
}

// False, with nothing written, where the results are left to the units on the fp32 instruction.
template <int D, int NB> __device__ __forceinline__ bool fwd_unit(const FwdArgs& a, const int h, const int row0, X3FwdSmem<X3Cfg<D, NB>>& sm)
{
    using C = X3Cfg<D, NB>;
    constexpr int NW = C::NW, ROWS = C::ROWS;
    const AttnGeom& g = a.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hh = lane >> 5, l32 = lane & 31;
    const int kvh = g.kv_of_q[h];
    const int last_row = (row0 + ROWS < g.lq ? row0 + ROWS : g.lq) - 1;
    const int n_vis = seg_rows_le(g.ks, seg_pos_of_row(g.qs, last_row));      // visible columns form the prefix [0, n_vis)
    const int n_full = seg_rows_le(g.ks, seg_pos_of_row(g.qs, row0));         // columns that every row sees
    if (n_vis == 0 && a.accumulate) return true;                              // merging an empty partial is the identity
    const int n_blocks = (n_vis + C::BLK - 1) / C::BLK;
    int vis[NB];                                                              // columns that rows 32 n + l see
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int row = row0 + 32 * n + l32;
        vis[n] = row < g.lq ? seg_rows_le(g.ks, seg_pos_of_row(g.qs, row)) : 0;
    }
    const float* k = static_cast<const float*>(a.k) + (long long)kvh * g.kv_stride_head;
    const float* v = static_cast<const float*>(a.v) + (long long)kvh * g.kv_stride_head;
    unsigned char* const slot = sm.t.rows[wave];
    const RowBlock<C> rows(slot, lane, g.kv_stride_tok);
    int b = wave;
    if (b < n_blocks) rows.request(k, g.kv_stride_tok, C::BLK * b, g.lc, lane);
    const Log2Scale c(g.scale);
    float v_top = 0.f;
    put_stationary<C>(sm.t.q, static_cast<const float*>(a.q) + (long long)h * g.q_stride_head, g.q_stride_tok, row0, g.lq, wave, lane);
    __syncthreads();
    const unsigned char* stat = sm.t.q + 16 * lane;

    f32x16 acc[NB][C::NJ];
    zero_acc<C>(acc);
    const float slack = 8.0f / c.hi;
    // a row's reference, in units of log2, is raised when a score exceeds it by more than 8 of them
    float ref[NB], limit[NB], l_run[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) { ref[n] = 0.f; limit[n] = -INFINITY; l_run[n] = 0.f; }

    auto walk = [&](auto apart) {
        for (; b < n_blocks; b += NW) {
            f32x16 s[NB];
            ColBlock<C> vc;
            landed<0>();
            vc.load(v, g.kv_stride_tok, C::BLK * b, g.lc, hh, l32);
            __builtin_amdgcn_sched_barrier(0);
            scores<C>(s, rows, slot, stat, [&]() { if (b + NW < n_blocks) rows.request(k, g.kv_stride_tok, C::BLK * (b + NW), g.lc, lane); });
            __builtin_amdgcn_sched_barrier(0);
            if (C::BLK * b + C::BLK > n_full) {
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (C::BLK * b + 8 * (r / 4) + 4 * hh + r % 4 >= vis[n]) s[n][r] = -INFINITY;
            }
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                float mx = max3(s[n][0], s[n][1], s[n][2]);
#pragma unroll
                for (int r = 3; r < 15; r += 2) mx = max3(mx, s[n][r], s[n][r + 1]);
                mx = max2(mx, s[n][15]);
                if (__any(mx > limit[n])) {
                    const float top = max_across_halves(mx);
                    if (top > limit[n]) {
                        const float to = top * c.hi, alpha = limit[n] == -INFINITY ? 0.f : fast_exp2(ref[n] - to);
                        ref[n] = to;
                        limit[n] = top + slack;
                        l_run[n] *= alpha;
#pragma unroll
                        for (int i = 0; i < C::NJ; ++i) acc[n][i] *= alpha;
                    }
                }
                float part[4];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    s[n][r] = fast_exp2(fmaf(s[n][r], c.lo, fmaf(s[n][r], c.hi, -ref[n])));
                    part[r & 3] = r < 4 ? s[n][r] : part[r & 3] + s[n][r];
                }
                l_run[n] += (part[0] + part[1]) + (part[2] + part[3]);
            }
            accumulate<C, decltype(apart)::value, true>(acc, vc, s, v_top);
        }
    };
    // the sums of o: 16 columns of 32 keys round 12 times, and a chain of more than about 2600 (7000) keys would end further from fp64 than in the 16-row units
    if (n_vis > (D == 64 ? 2048 : 5120)) walk(std::true_type{});
    else walk(std::false_type{});

    // Combine the splits and merge with the running (o, lse): weights per (row, split), then a row-contiguous pass.
    unsigned odd = scale_out_of_range(g.scale);
    stationary_range<C>(sm.t.q, wave, lane, odd);
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        l_run[n] = sum_across_halves(l_run[n]);
        odd |= (unsigned)!(l_run[n] < INFINITY);
    }
    v_top = largest_of_wave(v_top);
    __syncthreads();              // the operands are free
    stage_rows<C>(&sm.e.stage[wave * ROWS * C::PITCH], acc, lane, 1.0f);
    if (hh == 0) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            sm.e.m[wave * ROWS + 32 * n + l32] = ref[n];
            sm.e.l[wave * ROWS + 32 * n + l32] = l_run[n];
        }
    }
    const int tid = threadIdx.x;
    if (lane == 0) sm.e.top[wave] = v_top;
    __syncthreads();
    float lse_new = 0.f;
    if (tid < ROWS) lse_new = combine_rows<ROWS, NW>(a, h, row0, tid, sm.e.m, sm.e.l, sm.e.w, sm.e.wa);
    __syncthreads();
    v_top = largest_of_workgroup(sm.e.top);
    odd |= too_small(v_top);
    const float least = CUT_LOSS * (float)n_vis * (256.f + v_top);      // (the probabilities' largest is 2^8)
    constexpr int PARTS = ROWS * D / 4 / (64 * NW);
    f32x4 out[PARTS];
    Extremes ends;
#pragma unroll
    for (int u = 0; u < PARTS; ++u) {
        const int i = tid + 64 * NW * u, r = i / (D / 4), c = 4 * (i % (D / 4));
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NW; ++s) x += sm.e.w[s * ROWS + r] * *reinterpret_cast<const f32x4*>(&sm.e.stage[(s * ROWS + r) * C::PITCH + c]);
        ends.add(x[0], x[1]);
        ends.add(x[2], x[3]);
        out[u] = x;
        __builtin_amdgcn_sched_barrier(0);
    }
    odd |= ends.not_finite_or_below(least);
    if (any_of_workgroup<NW>(odd, sm.e.votes, tid)) return false;
    if (tid < ROWS && row0 + tid < g.lq) a.lse[(long long)h * g.lq + row0 + tid] = lse_new;
#pragma unroll
    for (int u = 0; u < PARTS; ++u) {
        const int i = tid + 64 * NW * u, r = i / (D / 4), c = 4 * (i % (D / 4));
        if (row0 + r >= g.lq) continue;
        f32x4* op = reinterpret_cast<f32x4*>(a.o + ((long long)(row0 + r) * g.nq + h) * D + c);
        if (a.accumulate) out[u] += sm.e.wa[r] * *op;
        *op = out[u];
    }
    return true;
}

// The units on the fp32 instruction as 256 threads run them, 16 rows one after another; four chains for a score, as the other pass may have been cut
template <int D> using Rows16 = rows16::F32Cfg<D, true, false, 4, 4, true>;

// Which rows a launch takes in units of 64 and of 32 rows: the last `n64` 64-row tiles (heads side by side, the longest first), the tiles before
// them as two 32-row units each.
template <int D>
__global__ void __launch_bounds__(256, 1) fwd_f32x3_kernel(const FwdArgs a, const unsigned n64, const int n_tiles)
{
    __shared__ __attribute__((aligned(1024))) union { X3FwdSmem<X3Cfg<D, 2>> two; X3FwdSmem<X3Cfg<D, 1>> one; rows16::FwdSmem<Rows16<D>> rows; } sm;
    const unsigned nq = a.g.nq, u = blockIdx.x - n64, t = blockIdx.x < n64 ? blockIdx.x : n64 + u / 2;
    const int h = (int)(t % nq), tile0 = 64 * (n_tiles - 1 - (int)(t / nq)), row0 = blockIdx.x < n64 ? tile0 : tile0 + 32 * (1 - (int)(u & 1));
    if (row0 >= a.g.lq || (blockIdx.x < n64 ? fwd_unit<D, 2>(a, h, row0, sm.two) : fwd_unit<D, 1>(a, h, row0, sm.one))) return;
    const int end = row0 + (blockIdx.x < n64 ? 64 : 32);
    for (int row = row0; row < end && row < a.g.lq; row += 16) {
        __syncthreads();
        rows16::fwd_unit<Rows16<D>>(a, h, row / 16, sm.rows);
    }
}

template <class C> union X3BwdSmem {
    struct { unsigned char t[2][C::PIECES], rows[C::NW][C::BLOCK_BYTES]; };
    struct { float stage[C::STAGE_FLOATS], top[2][C::NW]; unsigned votes[C::NW]; };
};
template <class C> union X3KvSmem {
    struct {
        unsigned char t[2][C::PIECES], rows[C::NW][C::BLOCK_BYTES];
        float scalars[C::NW][3][32];                       // the row scalars of each wavefront's block: -LSE log2(e) in two floats, Delta
    };
    struct { float stage[2][C::STAGE_FLOATS], top[2][C::NW]; unsigned votes[C::NW]; };
};

// dQ: S^T = K Q^T and dP^T = V dO^T per block, dS^T = P^T (dP^T - Delta), dQ^T += K^T dS^T.
template <int D, int NB> __device__ __forceinline__ bool dq_unit(const BwdArgs& a, const int h, const int row0, X3BwdSmem<X3Cfg<D, NB>>& sm)
{
    using C = X3Cfg<D, NB>;
    constexpr int NW = C::NW, ROWS = C::ROWS;
    const AttnGeom& g = a.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hh = lane >> 5, l32 = lane & 31;
    const int kvh = g.kv_of_q[h];
    const int last_row = (row0 + ROWS < g.lq ? row0 + ROWS : g.lq) - 1;
    const int n_vis = seg_rows_le(g.ks, seg_pos_of_row(g.qs, last_row));
    const int n_full = seg_rows_le(g.ks, seg_pos_of_row(g.qs, row0));
    if (n_vis == 0) return true;                          // dq_acc unchanged
    const int n_blocks = (n_vis + C::BLK - 1) / C::BLK;
    const Log2Scale c(g.scale);
    int vis[NB];
    float nl_hi[NB], nl_lo[NB], delta[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int row = row0 + 32 * n + l32, row_c = row < g.lq ? row : g.lq - 1;
        vis[n] = row < g.lq ? seg_rows_le(g.ks, seg_pos_of_row(g.qs, row)) : 0;
        neg_lse_log2(a.lse[(long long)h * g.lq + row_c], nl_hi[n], nl_lo[n]);
        delta[n] = UP * a.delta[(long long)h * g.lq + row_c];
    }
    const float* k = static_cast<const float*>(a.k) + (long long)kvh * g.kv_stride_head;
    const float* v = static_cast<const float*>(a.v) + (long long)kvh * g.kv_stride_head;
    unsigned char* const slot = sm.rows[wave];
    const RowBlock<C> rows(slot, lane, g.kv_stride_tok);
    int b = wave;
    if (b < n_blocks) rows.request(k, g.kv_stride_tok, C::BLK * b, g.lc, lane);
    const long long q_off = (long long)h * g.q_stride_head;
    float ds_top = 0.f;
    put_stationary<C>(sm.t[0], static_cast<const float*>(a.q) + q_off, g.q_stride_tok, row0, g.lq, wave, lane);
    put_stationary<C>(sm.t[1], static_cast<const float*>(a.d_o) + q_off, g.q_stride_tok, row0, g.lq, wave, lane);
    __syncthreads();
    const unsigned char *q_stat = sm.t[0] + 16 * lane, *g_stat = sm.t[1] + 16 * lane;

    f32x16 acc[NB][C::NJ];
    zero_acc<C>(acc);
    auto walk = [&](auto apart) {
        for (; b < n_blocks; b += NW) {
            f32x16 s[NB], dp[NB];
            ColBlock<C> kc;
            landed<0>();
            scores<C>(s, rows, slot, q_stat, [&]() { rows.request(v, g.kv_stride_tok, C::BLK * b, g.lc, lane); });
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[n][r] = probability(s[n][r], c, nl_hi[n], nl_lo[n]);
            landed<0>();
            kc.load(k, g.kv_stride_tok, C::BLK * b, g.lc, hh, l32);
            __builtin_amdgcn_sched_barrier(0);
            scores<C>(dp, rows, slot, g_stat, [&]() { if (b + NW < n_blocks) rows.request(k, g.kv_stride_tok, C::BLK * (b + NW), g.lc, lane); });
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[n][r] *= fmaf(dp[n][r], UP, -delta[n]);
            if (C::BLK * b + C::BLK > n_full) {
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (C::BLK * b + 8 * (r / 4) + 4 * hh + r % 4 >= vis[n]) s[n][r] = 0.f;
            }
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int r = 0; r < 16; r += 2) ds_top = largest(ds_top, s[n][r], s[n][r + 1]);
            accumulate<C, decltype(apart)::value, false>(acc, kc, s, ds_top);
        }
    };
    if (n_vis > 64 * D) walk(std::true_type{});            // (dq of the 16-row units rounds more often in its scores: 8000 and 13000 keys)
    else walk(std::false_type{});
    unsigned odd = scale_out_of_range(g.scale);
    stationary_range<C>(sm.t[0], wave, lane, odd);
    float g_top = largest_of_wave(stationary_range<C>(sm.t[1], wave, lane, odd));
    ds_top = largest_of_wave(ds_top);
    __syncthreads();
    stage_rows<C>(&sm.stage[wave * ROWS * C::PITCH], acc, lane, g.scale * DOWN);
    const int tid = threadIdx.x;
    if (lane == 0) { sm.top[0][wave] = g_top; sm.top[1][wave] = ds_top; }
    __syncthreads();
    g_top = largest_of_workgroup(sm.top[0]);
    ds_top = largest_of_workgroup(sm.top[1]);
    odd |= ds_too_small(ds_top, g_top);
    const float least = g.scale * (float)n_vis * (CUT_LOSS * (ds_top * DOWN) + 1024.f * SCORE_LOSS * g_top);
    constexpr int PARTS = ROWS * D / (64 * NW);
    float out[PARTS];             // consecutive lanes on consecutive floats
    Extremes ends;
#pragma unroll
    for (int u = 0; u < PARTS; ++u) {
        const int i = tid + 64 * NW * u, r = i / D, c = i % D;
        out[u] = sm.stage[r * C::PITCH + c];
#pragma unroll
        for (int s = 1; s < NW; ++s) out[u] += sm.stage[(s * ROWS + r) * C::PITCH + c];
        if (u % 2 == 1) ends.add(out[u - 1], out[u]);
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    odd |= ends.not_finite_or_below(least);
    if (any_of_workgroup<NW>(odd, sm.votes, tid)) return false;
    // Added with atomics: chunks of one shard may be in flight on several streams.
    // One addition per element and call, so calls in stream order still have a fixed order.
#pragma unroll
    for (int u = 0; u < PARTS; ++u) {
        const int i = tid + 64 * NW * u, r = i / D, c = i % D;
        if (row0 + r < g.lq) global_atomic_add(a.dq + ((long long)(row0 + r) * g.nq + h) * D + c, out[u]);
    }
    return true;
}

// dK / dV: the stationary rows are keys, the streamed rows q rows of every q head that reads the kv head, one head after the other:
// S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS.  With two runs a unit takes the first or the second half of those heads and adds its result
// to zeros: 0 + a + b = 0 + b + a, so the order of the two does not show.
template <int D, int NB> __device__ __forceinline__ bool dkdv_unit(const BwdArgs& a, const int kvh, const int kv_tile, const int h_first, const int h_end, const bool atomic,
                                                                        X3KvSmem<X3Cfg<D, NB>>& sm)
{
    using C = X3Cfg<D, NB>;
    constexpr int NW = C::NW, ROWS = C::ROWS, BLK = C::BLK;
    const AttnGeom& g = a.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hh = lane >> 5, l32 = lane & 31;
    const int col0 = kv_tile * ROWS;
    const int last_col = (col0 + ROWS < g.lc ? col0 + ROWS : g.lc) - 1;
    const int row_first = seg_rows_le(g.qs, seg_pos_of_row(g.ks, col0) - 1);         // rows before it see nothing of the tile
    const int row_full = seg_rows_le(g.qs, seg_pos_of_row(g.ks, last_col) - 1);      // rows from it on see all of it
    const bool key_ragged = col0 + ROWS > g.lc;
    int first[NB];                                        // the first row that sees keys 32 n + l
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int col = col0 + 32 * n + l32;
        first[n] = col < g.lc ? seg_rows_le(g.qs, seg_pos_of_row(g.ks, col) - 1) : 0x7fffffff;
    }
    const int block0 = row_first / BLK, n_blocks = (g.lq + BLK - 1) / BLK, per_head = row_first < g.lq ? n_blocks - block0 : 0;      // 0: keys that no row sees
    const Log2Scale c(g.scale);
    auto next_head = [&](int h) { for (++h; h < h_end && g.kv_of_q[h] != kvh; ++h) {} return h; };

    int h = next_head(h_first - 1), left = 0;             // `left` heads from h on
    for (int i = h; i < h_end; i = next_head(i)) ++left;
    if (left == 0 || per_head == 0) {
        for (int i = threadIdx.x; i < ROWS * D / 4 && !atomic && !a.accumulate; i += 64 * NW) {      // (else the zeros, or sums, are there)
            const int r = i / (D / 4), c = 4 * (i % (D / 4));
            if (col0 + r >= g.lc) continue;
            const long long at = ((long long)(col0 + r) * g.nkv + kvh) * D + c;
            *reinterpret_cast<f32x4*>(a.dv + at) = f32x4{0.f, 0.f, 0.f, 0.f};
            *reinterpret_cast<f32x4*>(a.dk + at) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        return true;
    }
    const float n_rows = (float)left * (float)(g.lq - row_first);

    f32x16 dk[NB][C::NJ], dv[NB][C::NJ];
    zero_acc<C>(dk);
    zero_acc<C>(dv);
    float ds_top = 0.f;
    {
        // this wavefront's next block: number b of head h; the blocks of all heads in one sequence are dealt to the wavefronts in turn
        int b = block0 + wave;
        auto settle = [&]() { while (b >= n_blocks && left > 0) { b -= per_head; h = next_head(h); --left; } };
        settle();
        unsigned char* const slot = sm.rows[wave];
        const RowBlock<C> rows(slot, lane, g.q_stride_tok);
        auto request_q = [&]() { rows.request(static_cast<const float*>(a.q) + (long long)h * g.q_stride_head, g.q_stride_tok, BLK * b, g.lq, lane); };
        if (left > 0) request_q();                        // (with few rows there may be no block for this one)
        const long long k_off = (long long)kvh * g.kv_stride_head;
        put_stationary<C>(sm.t[0], static_cast<const float*>(a.k) + k_off, g.kv_stride_tok, col0, g.lc, wave, lane);
        put_stationary<C>(sm.t[1], static_cast<const float*>(a.v) + k_off, g.kv_stride_tok, col0, g.lc, wave, lane);
        __syncthreads();
        const unsigned char *k_stat = sm.t[0] + 16 * lane, *v_stat = sm.t[1] + 16 * lane;
        while (left > 0) {
            const long long off = (long long)h * g.q_stride_head;
            const int r0 = BLK * b;
            f32x16 p[NB], ds[NB];
            const long long ri = (long long)h * g.lq + (r0 + l32 < g.lq ? r0 + l32 : g.lq - 1);
            const float lse = a.lse[ri], delta = a.delta[ri];
            landed<0>();
            scores<C>(p, rows, slot, k_stat, [&]() { rows.request(static_cast<const float*>(a.d_o) + off, g.q_stride_tok, r0, g.lq, lane); });
            __builtin_amdgcn_sched_barrier(0);
            {
                float nl_hi, nl_lo;
                neg_lse_log2(lse, nl_hi, nl_lo);
                float (&sc)[3][32] = sm.scalars[wave];      // (both half-waves write the same)
                sc[0][l32] = nl_hi;
                sc[1][l32] = nl_lo;
                sc[2][l32] = delta;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
            const float (&sc)[3][32] = sm.scalars[wave];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 nl_hi = *reinterpret_cast<const f32x4*>(&sc[0][8 * q + 4 * hh]), nl_lo = *reinterpret_cast<const f32x4*>(&sc[1][8 * q + 4 * hh]);
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int t = 0; t < 4; ++t) p[n][4 * q + t] = UP * probability(p[n][4 * q + t], c, nl_hi[t], nl_lo[t]);
            }
            if (r0 < row_full || key_ragged || r0 + BLK > g.lq) {
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int row = r0 + 8 * (r / 4) + 4 * hh + r % 4;
                        if (row < first[n] || row >= g.lq) p[n][r] = 0.f;
                    }
            }
            landed<0>();
            ColBlock<C> gc;
            gc.load(static_cast<const float*>(a.d_o) + off, g.q_stride_tok, r0, g.lq, hh, l32);
            __builtin_amdgcn_sched_barrier(0);
            b += NW;
            settle();
            scores<C>(ds, rows, slot, v_stat, [&]() { if (left > 0) request_q(); });
            ColBlock<C> qc;
            qc.load(static_cast<const float*>(a.q) + off, g.q_stride_tok, r0, g.lq, hh, l32);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 dl = *reinterpret_cast<const f32x4*>(&sc[2][8 * q + 4 * hh]);
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int t = 0; t < 4; ++t) ds[n][4 * q + t] = p[n][4 * q + t] * (ds[n][4 * q + t] - dl[t]);
            }
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int r = 0; r < 16; r += 2) ds_top = largest(ds_top, ds[n][r], ds[n][r + 1]);
            accumulate<C, true, false>(dv, gc, p, ds_top);
            accumulate<C, true, false>(dk, qc, ds, ds_top);
        }
    }
    unsigned odd = scale_out_of_range(g.scale);
    stationary_range<C>(sm.t[0], wave, lane, odd);
    const float v_top = largest_of_wave(stationary_range<C>(sm.t[1], wave, lane, odd));
    ds_top = largest_of_wave(ds_top);
    // consecutive lanes on consecutive floats where they are added with atomics, on consecutive 16 bytes where they are stored
    constexpr int PARTS = ROWS * D / (64 * NW);
    const int tid = threadIdx.x;
    auto float_of = [&](int u) { return atomic ? tid + 64 * NW * u : 4 * tid + 256 * NW * (u / 4) + u % 4; };
    auto gather = [&](float (&out)[PARTS], const float* stage) {
        Extremes ends;
#pragma unroll
        for (int u = 0; u < PARTS; ++u) {
            const int i = float_of(u), at = i / D * C::PITCH + i % D;
            out[u] = stage[at];
#pragma unroll
            for (int s = 1; s < NW; ++s) out[u] += stage[s * ROWS * C::PITCH + at];
            if (u % 2 == 1) ends.add(out[u - 1], out[u]);
            if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        return ends;
    };
    __syncthreads();
    stage_rows<C>(&sm.stage[0][wave * ROWS * C::PITCH], dv, lane, DOWN);
    stage_rows<C>(&sm.stage[1][wave * ROWS * C::PITCH], dk, lane, g.scale * DOWN);
    if (lane == 0) { sm.top[0][wave] = v_top; sm.top[1][wave] = ds_top; }
    __syncthreads();
    float out_v[PARTS], out_k[PARTS];
    const Extremes ends_v = gather(out_v, sm.stage[0]), ends_k = gather(out_k, sm.stage[1]);
    const float v_all = largest_of_workgroup(sm.top[0]), ds_all = largest_of_workgroup(sm.top[1]);
    odd |= ds_too_small(ds_all, v_all) | ends_v.not_finite_or_below(n_rows * 2.f * CUT_LOSS) |
           ends_k.not_finite_or_below(g.scale * n_rows * (CUT_LOSS * (ds_all * DOWN) + 1024.f * SCORE_LOSS * v_all));
    if (any_of_workgroup<NW>(odd, sm.votes, tid)) return false;
    auto write_out = [&](float* to, const float (&out)[PARTS]) {
#pragma unroll
        for (int u = 0; u < PARTS; u += 4) {
            if (atomic) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = float_of(u + e), r = i / D;
                    if (col0 + r < g.lc) global_atomic_add(to + ((long long)(col0 + r) * g.nkv + kvh) * D + i % D, out[u + e]);
                }
            } else {
                const int i = float_of(u), r = i / D;
                if (col0 + r >= g.lc) continue;
                f32x4 x = {out[u], out[u + 1], out[u + 2], out[u + 3]};
                f32x4* op = reinterpret_cast<f32x4*>(to + ((long long)(col0 + r) * g.nkv + kvh) * D + i % D);
                if (a.accumulate) x += *op;
                *op = x;
            }
        }
    };
    write_out(a.dv, out_v);
    write_out(a.dk, out_k);
    return true;
}

// The backward step in one launch: workgroups [0, n_dkdv) are dK / dV units (the longer ones, first, and of two runs the
// one with more heads before the other: 703 us where two runs a tile side by side take 840, 3056 x 3000 x 6/2 heads), the others dQ units of 64 and of 32 rows.
template <int D, int KB>
__global__ void __launch_bounds__(256, 1) bwd_f32x3_kernel(const BwdArgs a, const unsigned n_dkdv, const unsigned runs, const unsigned n64, const int n_tiles)
{
    __shared__ __attribute__((aligned(1024))) union { X3KvSmem<X3Cfg<D, KB>> kv; X3BwdSmem<X3Cfg<D, 2>> two; X3BwdSmem<X3Cfg<D, 1>> one;
                                                      rows16::DkdvSmem<Rows16<D>> kv_rows; rows16::DqSmem<Rows16<D>> q_rows; } sm;
    const unsigned nq = a.g.nq;
    if (blockIdx.x < n_dkdv) {
        const unsigned per_run = n_dkdv / runs, run = blockIdx.x / per_run, u = blockIdx.x - run * per_run, tile = u / (unsigned)a.g.nkv;
        const int kvh = (int)(u - tile * a.g.nkv), key0 = 32 * KB * (int)tile;
        const bool atomic = runs == 2;
        int first = 0, end = a.g.nq;
        if (atomic) {             // the first half of the heads that read kvh, or the rest
            int n = 0, half = 0;
            for (int h = 0; h < end; ++h) n += a.g.kv_of_q[h] == kvh;
            for (n = (n + 1) / 2; n > 0; ++half) n -= a.g.kv_of_q[half] == kvh;
            (run ? first : end) = half;
        }
        if (dkdv_unit<D, KB>(a, kvh, (int)tile, first, end, atomic, sm.kv)) return;
        for (int key = key0; key < key0 + 32 * KB && key < a.g.lc; key += 16) {
            __syncthreads();
            rows16::dkdv_unit<Rows16<D>>(a, kvh, key / 16, sm.kv_rows, first, end, atomic);
        }
    } else {
        const unsigned w = blockIdx.x - n_dkdv, u = w - n64, t = w < n64 ? w : n64 + u / 2;
        const int h = (int)(t % nq), tile0 = 64 * (n_tiles - 1 - (int)(t / nq)), row0 = w < n64 ? tile0 : tile0 + 32 * (1 - (int)(u & 1));
        if (row0 >= a.g.lq || (w < n64 ? dq_unit<D, 2>(a, h, row0, sm.two) : dq_unit<D, 1>(a, h, row0, sm.one))) return;
        const int end = row0 + (w < n64 ? 64 : 32);
        for (int row = row0; row < end && row < a.g.lq; row += 16) {
            __syncthreads();
            rows16::dq_unit<Rows16<D>>(a, h, row / 16, sm.q_rows);
        }
    }
}

}  // namespace

hipError_t hexi_launch_fwd_f32x3(const FwdArgs& a, const F32x3Fwd& plan, hipStream_t s)
{
    const int n_tiles = (a.g.lq + 63) / 64;
    const unsigned n64 = (unsigned)plan.n64, grid = n64 + 2u * ((unsigned)(n_tiles * a.g.nq) - n64);
    if (a.g.d == 128) fwd_f32x3_kernel<128><<<grid, 256, 0, s>>>(a, n64, n_tiles);
    else if (a.g.d == 64) fwd_f32x3_kernel<64><<<grid, 256, 0, s>>>(a, n64, n_tiles);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t hexi_launch_bwd_f32x3(const BwdArgs& a, const F32x3Bwd& plan, hipStream_t s)
{
    const int n_tiles = (a.g.lq + 63) / 64, keys = 32 * plan.key_blocks;
    const unsigned tiles = a.want_dq ? (unsigned)(n_tiles * a.g.nq) : 0u, n64 = plan.rows64 ? tiles : 0u;
    const unsigned runs = (unsigned)plan.runs, n_dkdv = a.want_dkdv ? (unsigned)((a.g.lc + keys - 1) / keys * a.g.nkv) * runs : 0u;
    const unsigned grid = n_dkdv + n64 + 2u * (tiles - n64);
    if (runs == 2 && a.want_dkdv) {
        const hipError_t e = hexi_launch_zero2_f32(a.dk, a.dv, (long long)a.g.lc * a.g.nkv * a.g.d, s);
        if (e != hipSuccess) return e;
    }
    if (a.g.d == 128 && plan.key_blocks == 1) bwd_f32x3_kernel<128, 1><<<grid, 256, 0, s>>>(a, n_dkdv, runs, n64, n_tiles);
    else if (a.g.d == 64 && plan.key_blocks == 1) bwd_f32x3_kernel<64, 1><<<grid, 256, 0, s>>>(a, n_dkdv, runs, n64, n_tiles);
    else if (a.g.d == 64) bwd_f32x3_kernel<64, 2><<<grid, 256, 0, s>>>(a, n_dkdv, runs, n64, n_tiles);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

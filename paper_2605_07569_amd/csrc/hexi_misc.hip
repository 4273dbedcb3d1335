// HBM-bound elementwise kernels: two-term log-sum-exp merge, Delta = rowsum(dO * O), fills.
#include "hexi_internal.h"
#include <hip/hip_bf16.h>
#include <type_traits>

namespace {

// One thread per 4 consecutive head_dim elements of one (row, head).  WITH_LSE: the head_dim / 4 threads of a (row, head) are
// lanes of one wavefront (a power of two up to 64), all of which have read lse_acc before the first of them rewrites it.
// Otherwise this pass only reads the lse arrays and merge_lse_kernel rewrites lse_acc afterwards.
// o_*: [n_rows][nq][d] fp32, lse_*: [nq][n_rows].  Weights are formed as e_a/(e_a+e_b) with
// e_x = exp(lse_x - max), which keeps them exact convex weights; -inf on one side is the identity.
template <int OUT_MODE, bool WITH_LSE>  // 0: no o_final, 1: fp32 o_final, 2: bf16 o_final
__global__ void __launch_bounds__(256) merge_kernel(long long n_vec, int nq, int d4, long long n_rows,
                                                    float* __restrict__ o_acc, float* __restrict__ lse_acc,
                                                    const float* __restrict__ o_part, const float* __restrict__ lse_part,
                                                    void* __restrict__ o_final)
{
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n_vec) return;
    const long long rh = idx / d4;
    const int c4 = (int)(idx - rh * d4);
    const long long row = rh / nq;
    const int h = (int)(rh - row * nq);
    const long long li = (long long)h * n_rows + row;
    const float a = lse_acc[li], b = lse_part[li];
    const float m = fmaxf(a, b);
    typedef float nt_f32x4 __attribute__((ext_vector_type(4)));
    // A partial that saw nothing of the row has weight 0: o_acc and lse_acc stay, and o_acc need not be read or written.  o_part is read all the same: its
    // LSE is -inf also where the row's sum is NaN (a NaN key, a score that overflowed to +inf), and then 0 x NaN has to reach o.  Half of the rows in
    // most steps of a zigzag ring see nothing, all of them where the chunk lies in the future: 4096 rows x 24 heads x 128, us per merge, every row merged /
    // as here: no such row 27.7 / 27.5, half of them 27.8 / 20.4, all 27.7 / 12.2 (17.8 and 6.2 if o_part were not read either).
    const bool weightless = b == -INFINITY && fabsf(m) != INFINITY;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    bool stays = false;
    if (m != -INFINITY) {
        const nt_f32x4 ob = __builtin_nontemporal_load(reinterpret_cast<const nt_f32x4*>(o_part) + idx);
        stays = weightless && fabsf(ob[0]) < INFINITY && fabsf(ob[1]) < INFINITY && fabsf(ob[2]) < INFINITY && fabsf(ob[3]) < INFINITY;
        if (OUT_MODE == 0 && stays) return;
        const nt_f32x4 oa = __builtin_nontemporal_load(reinterpret_cast<const nt_f32x4*>(o_acc) + idx);
        const float ea = expf(a - m), eb = expf(b - m);
        const float inv = 1.0f / (ea + eb);
        const float wa = ea * inv, wb = eb * inv;
        r = stays ? make_float4(oa[0], oa[1], oa[2], oa[3])
                  : make_float4(wa * oa[0] + wb * ob[0], wa * oa[1] + wb * ob[1], wa * oa[2] + wb * ob[2], wa * oa[3] + wb * ob[3]);
    }
    if (!stays) { const nt_f32x4 r_v = {r.x, r.y, r.z, r.w}; __builtin_nontemporal_store(r_v, reinterpret_cast<nt_f32x4*>(o_acc) + idx); }
    // m + log(e_a + e_b), as merge_lse_kernel forms it
    if (WITH_LSE && c4 == 0) lse_acc[li] = (m == -INFINITY) ? -INFINITY : m + logf(expf(a - m) + expf(b - m));
    if (OUT_MODE == 1) reinterpret_cast<float4*>(o_final)[idx] = r;
    if (OUT_MODE == 2) {
        __hip_bfloat16 t[4] = {__float2bfloat16(r.x), __float2bfloat16(r.y), __float2bfloat16(r.z), __float2bfloat16(r.w)};
        reinterpret_cast<uint2*>(o_final)[idx] = *reinterpret_cast<const uint2*>(t);
    }
}

// Second pass: one thread per (row, head) rewrites lse_acc.
__global__ void __launch_bounds__(256) merge_lse_kernel(long long n, float* __restrict__ lse_acc, const float* __restrict__ lse_part)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float a = lse_acc[i], b = lse_part[i];
    const float m = fmaxf(a, b);
    lse_acc[i] = (m == -INFINITY) ? -INFINITY : m + logf(expf(a - m) + expf(b - m));
}

}  // namespace

hipError_t hexi_launch_merge(long long n_rows, int nq, int d, float* o_acc, float* lse_acc, const float* o_part,
                             const float* lse_part, void* o_final, int o_final_dtype, hipStream_t s)
{
    const int d4 = d / 4;
    const long long n_vec = n_rows * nq * d4;
    const unsigned grid = (unsigned)((n_vec + 255) / 256);
    const bool with_lse = d4 <= 64 && (d4 & (d4 - 1)) == 0;
    auto launch = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
        if (with_lse) merge_kernel<MODE, true><<<grid, 256, 0, s>>>(n_vec, nq, d4, n_rows, o_acc, lse_acc, o_part, lse_part, o_final);
        else merge_kernel<MODE, false><<<grid, 256, 0, s>>>(n_vec, nq, d4, n_rows, o_acc, lse_acc, o_part, lse_part, o_final);
    };
    if (!o_final) launch(std::integral_constant<int, 0>{});
    else if (o_final_dtype == HEXI_F32) launch(std::integral_constant<int, 1>{});
    else launch(std::integral_constant<int, 2>{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || with_lse) return e;
    const long long n = n_rows * nq;
    merge_lse_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, lse_acc, lse_part);
    return hipGetLastError();
}

namespace {

// Delta[h][i] = sum_c dO[i][h][c] * O[i][h][c]; O fp32 dense, dO in the input dtype with strides.
// D/4 consecutive lanes share one (row, head).
template <typename T, int D>
__global__ void __launch_bounds__(256) delta_kernel(long long lq, int nq, const float* __restrict__ o, const T* __restrict__ d_o,
                                                    long long stride_tok, long long stride_head, float* __restrict__ delta)
{
    constexpr int LANES = D / 4;
    const long long rh = ((long long)blockIdx.x * 256 + threadIdx.x) / LANES;
    const int c4 = threadIdx.x % LANES;
    float acc = 0.f;
    const bool valid = rh < lq * nq;
    long long row = 0; int h = 0;
    if (valid) {
        row = rh / nq; h = (int)(rh - row * nq);
        typedef float nt_f32x4 __attribute__((ext_vector_type(4)));
        const nt_f32x4 ov_v = __builtin_nontemporal_load(reinterpret_cast<const nt_f32x4*>(o + rh * D) + c4);
        const float4 ov = make_float4(ov_v[0], ov_v[1], ov_v[2], ov_v[3]);
        const T* p = d_o + row * stride_tok + h * stride_head + c4 * 4;
        float g0, g1, g2, g3;
        if constexpr (sizeof(T) == 4) {
            const float4 gv = *reinterpret_cast<const float4*>(p);
            g0 = gv.x; g1 = gv.y; g2 = gv.z; g3 = gv.w;
        } else {
            const uint2 raw = *reinterpret_cast<const uint2*>(p);
            g0 = __uint_as_float(raw.x << 16); g1 = __uint_as_float(raw.x & 0xffff0000u);
            g2 = __uint_as_float(raw.y << 16); g3 = __uint_as_float(raw.y & 0xffff0000u);
        }
        acc = ov.x * g0 + ov.y * g1 + ov.z * g2 + ov.w * g3;
    }
#pragma unroll
    for (int off = LANES / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (valid && c4 == 0) delta[(long long)h * lq + row] = acc;
}

}  // namespace

hipError_t hexi_launch_delta(long long lq, int nq, int d, const float* o, const void* d_o, int dtype,
                             long long stride_tok, long long stride_head, float* delta, hipStream_t s)
{
    const long long n_threads = lq * nq * (d / 4);
    const unsigned grid = (unsigned)((n_threads + 255) / 256);
    if (dtype == HEXI_F32) {
        if (d == 64) delta_kernel<float, 64><<<grid, 256, 0, s>>>(lq, nq, o, (const float*)d_o, stride_tok, stride_head, delta);
        else delta_kernel<float, 128><<<grid, 256, 0, s>>>(lq, nq, o, (const float*)d_o, stride_tok, stride_head, delta);
    } else {
        if (d == 64) delta_kernel<uint16_t, 64><<<grid, 256, 0, s>>>(lq, nq, o, (const uint16_t*)d_o, stride_tok, stride_head, delta);
        else delta_kernel<uint16_t, 128><<<grid, 256, 0, s>>>(lq, nq, o, (const uint16_t*)d_o, stride_tok, stride_head, delta);
    }
    return hipGetLastError();
}

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Two buffers of n4 16-byte pieces set to zero in one launch (dk and dv of a chunk): 4 pieces per thread.
__global__ void __launch_bounds__(256) zero2_kernel(f32x4_t* __restrict__ p, f32x4_t* __restrict__ q, long long n4)
{
    f32x4_t* out = blockIdx.y ? q : p;
    const long long i = (long long)blockIdx.x * 1024 + threadIdx.x;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (i + 256 * u < n4) out[i + 256 * u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
}

// The forward partial of a chunk that no row sees, in one launch: o (n4 16-byte pieces) zero by the first `o_blocks` workgroups, the n_lse values of lse
// -inf by the others.  4096 rows x 24 heads x 128: 16.3 us as two launches of 4-byte stores, 8.3 us.
__global__ void __launch_bounds__(256) empty_partial_kernel(f32x4_t* __restrict__ o, long long n4, unsigned o_blocks, float* __restrict__ lse, long long n_lse)
{
    if (blockIdx.x < o_blocks) {
        const long long i = (long long)blockIdx.x * 1024 + threadIdx.x;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + 256 * u < n4) o[i + 256 * u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    } else {
        const long long i = (long long)(blockIdx.x - o_blocks) * 256 + threadIdx.x;
        if (i < n_lse) lse[i] = -INFINITY;
    }
}

}  // namespace

hipError_t hexi_launch_empty_partial(float* o, float* lse, long long n_rows_heads, int d, hipStream_t s)
{
    const long long n4 = n_rows_heads * (d / 4);
    const unsigned o_blocks = (unsigned)((n4 + 1023) / 1024), lse_blocks = (unsigned)((n_rows_heads + 255) / 256);
    empty_partial_kernel<<<o_blocks + lse_blocks, 256, 0, s>>>(reinterpret_cast<f32x4_t*>(o), n4, o_blocks, lse, n_rows_heads);
    return hipGetLastError();
}

hipError_t hexi_launch_zero2_f32(float* p, float* q, long long n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const long long n4 = n / 4;
    zero2_kernel<<<dim3((unsigned)((n4 + 1023) / 1024), 2), 256, 0, s>>>(reinterpret_cast<f32x4_t*>(p), reinterpret_cast<f32x4_t*>(q), n4);
    return hipGetLastError();
}

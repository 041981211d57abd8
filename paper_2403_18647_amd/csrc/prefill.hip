// Row-wise kernels: the residual stream and the RMSNorm around the GEMMs.
//
// Decode blocks (at most 64 rows) use rms_rows, and norm_rows behind a split
// residual GEMM.  A block of more rows (prompt prefill) is weight-reuse bound
// rather than weight-stream bound, so its linear layers run as tiled matrix-core
// GEMMs (prefill_gemm.hip: bf16 on the packed weights, float on the caller's
// row-major ones, float accumulation and output).  RoPE with the Q / K / V
// writes and SwiGLU run in the epilogues of those GEMMs, everything else of it
// in norm_rows.  All round exactly where the decode kernels round (the values a bf16 model
// stores): the RMSNorm output bf16(x o g / rms), K and V, the SwiGLU product;
// Q and the residual stream stay float.  Rotary cos / sin come from the same
// table as the decode path.
#include <hip/hip_ext.h>

#include "device.h"
#include "kernels.h"

namespace sdsat {

// h[m][k] = elem(xg[m][k] / rms_m), rms_m = sqrt(sum_t ssq[m][t] / K + eps),
// xg and h in fragment order.  One wave per row and 64 of its 8-element chunks,
// which sums the row's partials for itself, in the order the decode GEMM does
// (lane-strided, then a wave butterfly).  Latency-bound: no barrier, and one
// round trip for the values and the first partials.  With 8 waves per 512 chunks
// of a 16-row tile (contiguous stores, but two rows' sums per wave and a barrier)
// blocks of 9 rows took, us, 256 wide, 2 heads, 4 layers: 156, now 151; 1024 wide:
// 188, now 182; the 7B 4-layer block of 6 rows 411.4, now 410.9; the 13B 3-layer
// block of 11 rows 498.2, now 497.4.
template <typename T>
__global__ void __launch_bounds__(64) rms_rows_kernel(const float* xg, int ld, const float* ssq, int n_ssq, int K, float eps,
                                                      int M, T* h) {
    const int m = blockIdx.y, lane = threadIdx.x, k = 8 * ((int)blockIdx.x * 64 + lane);
    const size_t off = frag_off(m, min(k, K - 8), ld, M);   // clamped into the row
    const Frag<float> v = Frag<float>::load(xg + off);
    const float* sr = ssq + (size_t)m * n_ssq;
    float sum = 0.f;
    for (int col = lane; col < n_ssq; col += 64) sum += sr[col];
    const float inv = 1.0f / sqrtf(wave_sum(sum) / (float)K + eps);
    const float x[8] = {v.lo.x * inv, v.lo.y * inv, v.lo.z * inv, v.lo.w * inv,
                        v.hi.x * inv, v.hi.y * inv, v.hi.z * inv, v.hi.w * inv};
    if (k < K) Frag<T>::from_f32(x).store(h + off);
}

// One row of a large block (more than 64 rows), or of a decode block behind a
// split residual GEMM: its new residual value and the next GEMM's normalised input h[m] = elem((x[m] o g) / rms_m), in one pass.
// EMBED: x[m] = E[token[m]] (layer 0; ids out of range set *err and read row 0);
// otherwise x[m] += y[m], the sum of a split contraction's parts in part order.
// One workgroup per row, four columns per thread and pass, every load issued
// first.  The sums of squares are formed per 16-column group in the order of the
// decode kernel that would form them -- the residual epilogue's butterfly
// (columns c, c + 8, then + 4, + 2, + 1), for EMBED embed_kernel's columns in
// turn -- and reduced in rms_rows' order (lane-strided, then a wave butterfly),
// so h is bitwise what a separate pass and rms_rows give: a token's layer 0 is
// the same in a prompt and in a decode block.  h is in fragment
// order, where 16 rows share each cache line: runs of 16 rows go to one XCD
// (workgroups go to the 8 XCDs round-robin), whose L2 then merges their writes;
// a decode block's few rows are spread over all of them instead.  Behind the
// split down GEMM it replaces a kernel that folded the partials and rms_rows.
static constexpr int kNormRowMaxThreads = 1024;
static constexpr int kNormRowPasses = 2;   // rows of up to 2 x 4 x 1024 columns
struct NormRowArgs {
    const float* y; int parts; size_t part_stride; int ldy;   // residual update
    const void* emb; int n_emb; const int* tokens; int* err;   // EMBED
    int M, N; float* x; const float* g; float eps; void* h; int ldh;
    int h_rows;   // rows of h's fragment order
    int spread;   // row = workgroup index
};
template <typename T, bool EMBED, int MAXP>
__global__ void __launch_bounds__(kNormRowMaxThreads) norm_rows_kernel(NormRowArgs a) {
    constexpr int P = kNormRowPasses;
    __shared__ float s_ssq[P * 4 * kNormRowMaxThreads / 16];
    __shared__ float s_inv;
    const int per = (int)gridDim.x / 8, t = threadIdx.x;
    const int m = a.spread ? (int)blockIdx.x : ((int)blockIdx.x % 8) * per + (int)blockIdx.x / 8;
    if (m >= a.M) return;
    float* x = a.x + (size_t)m * a.N;
    f32x4_t v[P], gv[P];
    size_t erow = 0;
    if constexpr (EMBED) {
        int tok = a.tokens[m];
        if (tok < 0 || tok >= a.n_emb) {
            if (t == 0) atomicOr(a.err, 1);
            tok = 0;
        }
        erow = (size_t)tok * a.N;
    }
#pragma unroll
    for (int c = 0; c < P; ++c) {
        const int n = min((c * (int)blockDim.x + t) * 4, a.N - 4);   // clamped into the row
#pragma unroll
        for (int i = 0; i < 4; ++i) gv[c][i] = a.g[n + i];
        if constexpr (EMBED) {
            const T* src = reinterpret_cast<const T*>(a.emb) + erow + n;
            if constexpr (sizeof(T) == 2) {
                const uint2 w = *reinterpret_cast<const uint2*>(src);
                v[c] = f32x4_t{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xFFFF0000u),
                               __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xFFFF0000u)};
            } else {
                v[c] = *reinterpret_cast<const f32x4_t*>(src);
            }
        } else {
            const float* y = a.y + (size_t)m * a.ldy + n;
            f32x4_t pv[MAXP];
#pragma unroll
            for (int q = 0; q < MAXP; ++q)
                if (q < a.parts) pv[q] = *reinterpret_cast<const f32x4_t*>(y + q * a.part_stride);
            const f32x4_t xv = *reinterpret_cast<const f32x4_t*>(x + n);
            v[c] = pv[0];
#pragma unroll
            for (int q = 1; q < MAXP; ++q)
                if (q < a.parts) v[c] += pv[q];
            v[c] = xv + v[c];
        }
    }
#pragma unroll
    for (int c = 0; c < P; ++c) {
        const int n = (c * (int)blockDim.x + t) * 4;
        if (n < a.N) *reinterpret_cast<f32x4_t*>(x + n) = v[c];
        if constexpr (EMBED) {   // column by column: each thread's four onto its left neighbour's sum
            float ss = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float in = __shfl_up(ss, 1, 64);
                if ((t & 3) != k) continue;
                ss = k ? fmaf(v[c][1], v[c][1], fmaf(v[c][0], v[c][0], in)) : fmaf(v[c][0], v[c][0], v[c][1] * v[c][1]);
                ss = fmaf(v[c][3], v[c][3], fmaf(v[c][2], v[c][2], ss));
            }
            if ((t & 3) == 3 && n < a.N) s_ssq[n / 16] = ss;
        } else {
            f32x4_t ss = n < a.N ? v[c] * v[c] : f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                ss[i] += __shfl_xor(ss[i], 2, 64);
                ss[i] += __shfl_xor(ss[i], 1, 64);
            }
            if ((t & 3) == 0 && n < a.N) s_ssq[n / 16] = (ss[0] + ss[2]) + (ss[1] + ss[3]);
        }
    }
    __syncthreads();
    if (t < 64) {
        const int n_ssq = a.N / 16;
        float sum = 0.f;
        for (int col = t; col < n_ssq; col += 64) sum += s_ssq[col];
        sum = wave_sum(sum);
        if (t == 0) s_inv = 1.0f / sqrtf(sum / (float)a.N + a.eps);
    }
    __syncthreads();
    const float inv = s_inv;
#pragma unroll
    for (int c = 0; c < P; ++c) {
        const int n = (c * (int)blockDim.x + t) * 4;
        if (n >= a.N) continue;
        const f32x4_t w = v[c] * gv[c] * inv;
        T* h = reinterpret_cast<T*>(a.h) + frag_off(m, n, a.ldh, a.h_rows);
        if constexpr (sizeof(T) == 2)
            *reinterpret_cast<uint2*>(h) = uint2{f32x2_to_bf16x2(w[0], w[1]), f32x2_to_bf16x2(w[2], w[3])};
        else
            *reinterpret_cast<f32x4_t*>(h) = w;
    }
}

hipError_t launch_rms_rows(int dtype, const float* xg, int ld, const float* ssq, int n_ssq, int K, float eps, int M,
                           void* h, hipStream_t s) {
    if (M < 1) return hipSuccess;
    if (K < 8 || K % 8 || ld < K) return hipErrorInvalidValue;   // whole chunks
    const dim3 grid((unsigned)((K / 8 + 63) / 64), (unsigned)M);
    if (dtype == 1)
        hipLaunchKernelGGL(rms_rows_kernel<uint16_t>, grid, dim3(64), 0, s, xg, ld, ssq, n_ssq, K, eps, M,
                           static_cast<uint16_t*>(h));
    else
        hipLaunchKernelGGL(rms_rows_kernel<float>, grid, dim3(64), 0, s, xg, ld, ssq, n_ssq, K, eps, M,
                           static_cast<float*>(h));
    return hipGetLastError();
}

template <bool EMBED, int MAXP>
static hipError_t norm_rows(int dtype, const NormRowArgs& a, hipStream_t s, hipEvent_t ev1 = nullptr) {
    if (a.N < 16 || a.N % 16 || a.N > kNormRowPasses * 4 * kNormRowMaxThreads || a.ldh < a.N) return hipErrorInvalidValue;
    const int per = ((a.M + 15) / 16 + 7) / 8 * 16;   // rows per XCD
    const dim3 grid(a.spread ? a.M : 8 * per), block(((a.N + 4 * kNormRowPasses - 1) / (4 * kNormRowPasses) + 63) / 64 * 64);
    auto kern = dtype == 1 ? norm_rows_kernel<uint16_t, EMBED, MAXP> : norm_rows_kernel<float, EMBED, MAXP>;
    if (ev1) hipExtLaunchKernelGGL(kern, grid, block, 0, s, nullptr, ev1, 0, a);
    else hipLaunchKernelGGL(kern, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_resid_norm_rows(int dtype, const float* y, int parts, size_t part_stride, int ldy, int M, int N,
                                  float* x, int ldx, const float* g, float eps, void* h, int ldh, hipStream_t s) {
    if (M < 1) return hipSuccess;
    if (parts < 1 || parts > kPrefillMaxSplit || ldx != N || ldy % 4 || part_stride % 4) return hipErrorInvalidValue;
    NormRowArgs a{};
    a.y = y; a.parts = parts; a.part_stride = part_stride; a.ldy = ldy;
    a.M = M; a.N = N; a.x = x; a.g = g; a.eps = eps; a.h = h; a.ldh = ldh;
    a.h_rows = (M + 15) & ~15;
    return norm_rows<false, kPrefillMaxSplit>(dtype, a, s);
}

hipError_t launch_fold_norm_rows(int dtype, const float* part, int parts, int M, int N, float* x, const float* g, float eps,
                                 void* h, int ldh, hipStream_t s, hipEvent_t ev1) {
    if (M < 1 || !part || parts < 1 || parts > kFoldMaxParts || ((size_t)M * N) % 4) return hipErrorInvalidValue;
    NormRowArgs a{};
    a.y = part; a.parts = parts; a.part_stride = (size_t)M * N; a.ldy = N;
    a.M = M; a.N = N; a.x = x; a.g = g; a.eps = eps; a.h = h; a.ldh = ldh; a.h_rows = M; a.spread = 1;
    return norm_rows<false, kFoldMaxParts>(dtype, a, s, ev1);
}

hipError_t launch_embed_norm_rows(int dtype, const void* embed, int n_rows_emb, const int* tokens, int M, int N, float* x,
                                  const float* g, float eps, void* h, int ldh, int* err, hipStream_t s) {
    if (M < 1) return hipSuccess;
    NormRowArgs a{};
    a.emb = embed; a.n_emb = n_rows_emb; a.tokens = tokens; a.err = err;
    a.M = M; a.N = N; a.x = x; a.g = g; a.eps = eps; a.h = h; a.ldh = ldh;
    a.h_rows = (M + 15) & ~15;
    return norm_rows<true, 1>(dtype, a, s);
}

}  // namespace sdsat

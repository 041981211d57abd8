// Skinny weight-streaming GEMM for block decode: Y[M, N] = X[M, K] . W[N, K]^T with
// M = batch * block rows (<= 64) and N, K model dimensions.  At M <= 64 the
// contraction does about M flops per weight byte, far below the matrix-core
// ridge, so the kernel is bound by streaming W from HBM once.  The design:
//
//  * W is pre-packed (launch_pack) into 16-column x 32-k tiles laid out in lane
//    order, so every wave-wide load is one contiguous 1 KiB (bf16) run and each
//    lane's 16 bytes is directly its matrix-core B fragment.
//  * One workgroup per column tile (3 or 4 above 16 rows).  Its waves split the
//    contraction into contiguous slices, stream their slice with two batches of
//    loads in flight, read the X fragments for the same steps straight from
//    global memory (the few X rows stay in L2, in fragment order), and reduce
//    their partial tiles through LDS in wave order: deterministic, with no device-scope fences or
//    atomics.
//  * An RMSNorm input arrives either already normalised and rounded to the
//    element type (rms_rows; blocks of several rows, whose float rows re-read by
//    every workgroup would cost as much traffic as the weights), or, for one-row
//    blocks, as the float rows x o g (gain applied by the producer): the kernel
//    then reduces the producer's per-tile sums of squares to each row's 1/rms
//    before its first matrix-core step and rounds x o g / rms to the element
//    type at the matrix-core input.  Both give the normalised activation a bf16
//    model stores, rounded once, bit for bit the same.
//  * Residual GEMMs whose tile count would leave some compute units a second
//    workgroup (13B: 320 tiles on 256 units), and long narrow ones of blocks of
//    several row tiles (four tiles per workgroup, so each row byte read feeds
//    four), spread each tile's waves over several workgroups and leave the
//    waves' partial rows to the row kernel that adds them, in the same wave
//    order, updates the residual and normalises (plan_gemm_resid,
//    launch_fold_norm_rows).
//  * Fused epilogues, the reduced tiles shared out over the waves:
//      EP_STORE   float output (LM-head logits)
//      EP_QKV     RoPE on Q and K columns, Q (float) to its buffer, K and V into
//                 the cache slots of the block rows (positions cache_len[b] + r)
//      EP_RESID   residual add into the float residual stream, the updated rows
//                 times the next RMSNorm's gain, and per-tile sums of squares
//                 that the next RMSNorm reduces
//      EP_SWIGLU  silu(gate) * up, rounded to the activation type
#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "device.h"
#include "kernels.h"

namespace sdsat {

size_t packed_elems(int n_tiles, int k_steps) { return (size_t)n_tiles * k_steps * 64 * 8; }

template <typename T>
__global__ void pack_kernel(PackArgs a) {
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // (tile, kstep, lane)
    const size_t total = (size_t)a.n_tiles * a.k_steps * 64;
    if (idx >= total) return;
    const int lane = (int)(idx & 63);
    const size_t tk = idx >> 6;
    const int ks = (int)(tk % a.k_steps);
    const int t = (int)(tk / a.k_steps);
    const int c = lane & 15, g = lane >> 4;
    long row = -1;   // stacked source row
    if (a.perm == PACK_PLAIN) {
        row = 16L * t + c;
    } else if (a.perm == PACK_ROPE) {
        const int tph = a.head_dim / 16, half = a.head_dim / 2;
        const int head = t / tph, j = t % tph;
        const int dim = c < 8 ? 8 * j + c : half + 8 * j + (c - 8);
        row = (long)head * a.head_dim + dim;
    } else {  // PACK_GATEUP
        const int f = 8 * t + (c & 7);
        row = f < a.F ? (c < 8 ? f : (long)a.F + f) : -1;
    }
    const T* src = nullptr;
    long r = row;
    if (row >= 0 && row < a.N) {
        if (r < a.N0) src = (const T*)a.src0;
        else if ((r -= a.N0) < a.N1) src = (const T*)a.src1;
        else { r -= a.N1; src = (const T*)a.src2; }
    }
    T* dst = (T*)a.dst + idx * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k = 32 * ks + 8 * g + e;
        float v = 0.f;
        if (src && k < a.K) v = to_f32<T>(src[r * a.K + k]);
        dst[e] = to_elem<T>(v);
    }
}

void launch_pack(const PackArgs& a, hipStream_t s) {
    const size_t total = (size_t)a.n_tiles * a.k_steps * 64;
    const int blocks = (int)((total + 255) / 256);
    if (a.dtype == 1) hipLaunchKernelGGL(pack_kernel<uint16_t>, dim3(blocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(pack_kernel<float>, dim3(blocks), dim3(256), 0, s, a);
}

// Plans (measured on MI355X with weights streamed from HBM):
//  * blocks of up to 16 rows: one column tile per workgroup, 8 waves for the
//    narrow [d, d] / [d, F] matrices (256 tiles, one workgroup per compute
//    unit), 4 for the wide ones; at least 4 contraction steps per wave
//    (several tiles per workgroup, or X staged in LDS, measured slower);
//  * blocks of more than 16 rows (batch 4 decode, prefill chunks) read more X
//    per weight fragment: for the wide matrices a workgroup of 4 waves takes 3
//    column tiles, so that one X load feeds 3 products and enough workgroups
//    are left (7B QKV: 256, one per compute unit).  us with 1 / 2 / 3 / 4 tiles,
//    7B, 24 rows: gate/up 41.0 / 39.6 / 33.5 / 45.6, QKV 25.0 / 27.4 / 25.1 /
//    29.2, LM head 55.3 / 54.7 / 48.5 / 55.6; 44 rows: 52.1 / 43.8 / 37.0 /
//    46.5, 31.4 / 31.5 / 26.0 / 31.6, 72.0 / 60.6 / 53.9 / 58.0; 64 rows: 60.6 /
//    51.4 / 41.4 / 54.5, 37.0 / 38.5 / 28.4 / 34.8, 83.4 / 71.1 / 59.5 / 63.6.
//    The narrow ones keep one tile per workgroup.  The waves per workgroup
//    depend on the matrix shape only where block-size invariance needs it: one
//    row tile and several column tiles both use 4 waves on the wide matrices.
GemmPlan plan_gemm(int M, int n_tiles, int k_steps) {
    GemmPlan p;
    p.mt = (M + 15) / 16;
    p.ntw = p.mt > 1 && n_tiles > 512 ? 3 : 1;
    int w = p.ntw > 1 ? 4 : (n_tiles <= 512 ? 8 : 4);
    while (w > 1 && k_steps < 4 * w) w /= 2;
    p.waves = w;
    p.grid = (n_tiles + p.ntw - 1) / p.ntw;
    p.lds_bytes = w * p.mt * p.ntw * 64 * 16;
    p.ksplit = 1;
    return p;
}

// Residual GEMMs (O, down) of narrow matrices whose tile count is not a
// multiple of the 256 compute units (13B: 320 tiles) leave some units two
// workgroups and the rest one.  Their tiles' waves are then spread over
// ksplit workgroups (320 x 4 = 1280 workgroups of 2 waves, 5 per unit); each
// wave keeps its slice of the contraction, and the row kernel that follows adds
// the waves' partials in wave order, as the single workgroup's LDS reduction
// does, so the results are the same bit for bit.  Measured at 13B, 11 rows: down
// (432 contraction steps) 39.4 -> 32.6 us; O (160 steps) 16.6 -> 17.1 us, its
// waves' work too short to pay for the partials, so it stays whole.
// Blocks of several row tiles re-read all of their rows in every workgroup (L2 hits, but at batch
// 4 x 6 rows the down GEMM's 528 KB of rows per workgroup outweigh its 352 KB of weights).  A narrow
// residual GEMM with a long contraction then takes four column tiles per workgroup, so each row byte
// feeds four tiles, and spreads each tile's wave slices over one-wave workgroups (same slices, same
// fold order: the same values).  Measured on the 7B down GEMM: batch 4 x 6 rows 29.2 -> 27.5 us,
// batch 8 x 6 rows 45.5 -> 34.0 us (a fold included); the O GEMM (128 steps) split the same way
// was slower at batch 8 and 10.
GemmPlan plan_gemm_resid(int M, int n_tiles, int k_steps) {
    GemmPlan p = plan_gemm(M, n_tiles, k_steps);
    if (p.mt > 1 && p.ntw == 1 && n_tiles <= 512 && k_steps >= 256) {
        p.ntw = 4;
        p.ksplit = p.waves;
        p.waves = 1;
        p.grid = (n_tiles + p.ntw - 1) / p.ntw * p.ksplit;
        p.lds_bytes = 0;   // partial tiles go to memory
        return p;
    }
    if (n_tiles > 512) {   // whole: the row kernel behind a split takes 8192 columns.  One tile per workgroup as for the
                           // narrow ones (9216 wide, FFN 24576, one layer, 24 / 48 / 64 rows: 458 / 569 / 643 us;
                           // 2 tiles at 24 rows and 4 beyond, row-major rows: 580 / 630 / 776 us)
        p.ntw = 1;
        p.grid = n_tiles;
        p.lds_bytes = p.waves * p.mt * 64 * 16;
        return p;
    }
    if (n_tiles <= 256 || k_steps < 256) return p;
    auto spread = [&](int k) {   // workgroup rounds over the average, per compute unit
        const long n = (long)n_tiles * k;
        return (double)((n + 255) / 256) * 256.0 / (double)n;
    };
    int best = 1;
    for (int k = 2; k <= p.waves; k *= 2)
        if (spread(k) < spread(best) - 1e-9) best = k;
    p.ksplit = best;
    p.waves /= best;
    p.grid = n_tiles * best;
    p.lds_bytes = p.waves * p.mt * 64 * 16;
    return p;
}

size_t gemm_resid_part_bytes(int n_tiles, int k_steps, int max_rows) {
    size_t most = 0;
    for (int m = 1; m <= std::min(std::max(max_rows, 1), 64); m += 16) {
        const GemmPlan p = plan_gemm_resid(std::min(m + 15, std::min(std::max(max_rows, 1), 64)), n_tiles, k_steps);
        if (p.ksplit > 1) most = std::max(most, (size_t)n_tiles * p.waves * p.ksplit * p.mt * 64 * 16);
    }
    return most;
}

// Steps per load batch (two batches in flight), sized so both batches of
// weight and X fragments fit the register budget (float X fragments of an
// RMSNorm input take twice the registers of bf16 ones).  The QKV GEMM on float
// rows takes 4 (142 VGPRs: its 3 workgroups of 4 waves per compute unit stay
// resident; 7B, 6 rows: 22.1 -> 21.2 us); the other float-row GEMMs keep 3
// (gate/up, 1376 workgroups, loses occupancy at 4: 32.4 -> 33.2 us at one row).
template <typename T, int EP, int MT, bool XF> struct Batch {
    static constexpr int U = MT == 1 ? (sizeof(T) == 2 ? (XF ? (EP == EP_QKV ? 4 : 3) : 4) : 2)
                                     : (sizeof(T) == 2 && !XF ? 2 : 1);
};

// X fragment as loaded: the element type, or raw floats of an RMSNorm input.
template <typename T, bool XF> struct XIn { using type = Frag<T>; };
template <typename T> struct XIn<T, true> { using type = Frag<float>; };

// Matrix-core A fragment from a loaded X fragment: RMSNorm inputs are scaled
// by the row's 1/rms and rounded to the element type here.
template <typename T, bool XF, typename XT>
__device__ __forceinline__ Frag<T> a_frag(const XT& x, float inv) {
    if constexpr (XF) {
        float v[8] = {x.lo.x * inv, x.lo.y * inv, x.lo.z * inv, x.lo.w * inv,
                      x.hi.x * inv, x.hi.y * inv, x.hi.z * inv, x.hi.w * inv};
        return Frag<T>::from_f32(v);
    } else {
        return x;
    }
}

// One batch of U contraction steps: the weight fragments of the NTW tiles
// (streamed, non-temporal) and the X fragments of every row tile.  Steps past
// the wave's slice reload the last step with X zeroed.
template <typename T, typename XT, int MT, int NTW, int U>
__device__ __forceinline__ void load_batch(Frag<T> (&w)[U][NTW], XT (&x)[U][MT], const T* const (&wp)[NTW],
                                           __amdgpu_buffer_rsrc_t xrs, const uint32_t (&xo)[MT],
                                           const uint32_t (&xst)[MT], int s, int nks) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int st = min(s + u, nks - 1);
#pragma unroll
        for (int j = 0; j < NTW; ++j) w[u][j] = Frag<T>::load_nt(wp[j] + (size_t)st * 512);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            x[u][mt] = buf_frag<typename XT::elem>(xrs, xo[mt], (uint32_t)st * xst[mt]);
            if (s + u >= nks) x[u][mt] = XT::zero();
        }
    }
}

template <typename T, bool XF, typename XT, int MT, int NTW, int U>
__device__ __forceinline__ void mma_batch(f32x4_t (&acc)[NTW][MT], const Frag<T> (&w)[U][NTW],
                                          const XT (&x)[U][MT], const float (&inv)[MT]) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const Frag<T> xa = a_frag<T, XF>(x[u][mt], inv[mt]);
#pragma unroll
            for (int j = 0; j < NTW; ++j) mma(acc[j][mt], xa, w[u][j]);
        }
}

// The steady state: a batch's products, each step's fragments reloaded with the
// step two batches ahead (s + u, inside the slice) as soon as they are used.
// The loads are unconditional so that the compiler's wait counts stay exact, and
// each step is kept together: with the row step a run-time value the scheduler
// puts a whole batch's loads behind its products, X before W, and the stream
// stalls (7B, 4 layers, 1 / 2 / 6 rows: 409.4 / 416.7 / 430 us, so 398.7 / 412 /
// 426; with the row step a constant, in an instance for one row: 400 / 415.6 / 429).
template <typename T, bool XF, typename XT, int MT, int NTW, int U>
__device__ __forceinline__ void step_batch(f32x4_t (&acc)[NTW][MT], Frag<T> (&w)[U][NTW], XT (&x)[U][MT],
                                           const float (&inv)[MT], const T* const (&wp)[NTW],
                                           __amdgpu_buffer_rsrc_t xrs, const uint32_t (&xo)[MT],
                                           const uint32_t (&xst)[MT], int s) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const Frag<T> xa = a_frag<T, XF>(x[u][mt], inv[mt]);
#pragma unroll
            for (int j = 0; j < NTW; ++j) mma(acc[j][mt], xa, w[u][j]);
        }
#pragma unroll
        for (int j = 0; j < NTW; ++j) w[u][j] = Frag<T>::load_nt(wp[j] + (size_t)(s + u) * 512);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            x[u][mt] = buf_frag<typename XT::elem>(xrs, xo[mt], (uint32_t)(s + u) * xst[mt]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Fused epilogue of one reduced 16 x 16 tile (column tile `tile`, row tile mt), run by one wave.
// acc[r] = Y[m = 16mt + 4g + r][column c of the tile]
// ep_in, gn: epilogue_inputs of this tile
template <typename T, int EP>
__device__ __forceinline__ void epilogue(const GemmArgs& a, int tile, int mt, const f32x4_t& acc, const float (&ep_in)[4],
                                         float gn, int c, int g) {
    const int M = a.M;
    if (EP == EP_STORE) {
        const int n = tile * 16 + c;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * mt + 4 * g + r;
            if (m < M && n < a.N) a.y[(size_t)m * a.ldy + n] = acc[r];
        }
    } else if (EP == EP_RESID) {
        const int n = tile * 16 + c;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * mt + 4 * g + r;
            float ss = 0.f;
            if (m < M && n < a.N) {
                const float v = ep_in[r] + acc[r];
                a.resid[(size_t)m * a.ldy + n] = v;
                a.xg_out[frag_off(m, n, a.ldxg, M)] = v * gn;
                ss = v * v;
            }
            ss += __shfl_xor(ss, 8, 64);
            ss += __shfl_xor(ss, 4, 64);
            ss += __shfl_xor(ss, 2, 64);
            ss += __shfl_xor(ss, 1, 64);
            if (c == 0 && m < M) a.ssq_out[(size_t)m * a.n_tiles + tile] = ss;
        }
    } else if (EP == EP_SWIGLU) {
        const int f = 8 * tile + (c & 7);
        T* u = reinterpret_cast<T*>(a.uout);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * mt + 4 * g + r;
            const float mine = acc[r];
            const float other = __shfl_xor(mine, 8, 64);
            if (c < 8 && m < M) {   // columns F.. are zero: packed weights hold zero rows there
                const float gate = mine, up = other;
                u[frag_off(m, f, a.ldu, M)] = to_elem<T>(gate / (1.0f + expf(-gate)) * up);
                if (tile == a.n_tiles - 1)   // and so are the chunks up to the padded length
                    for (int p = f + 8; p < a.ldu; p += 8) u[frag_off(m, p, a.ldu, M)] = to_elem<T>(0.f);
            }
        }
    } else if (EP == EP_QKV) {
        const int Dh = a.Dh, half = Dh / 2, H = a.H;
        const int tph = Dh / 16;
        const int head_all = tile / tph, j = tile % tph;
        const int sec = head_all / H, h = head_all % H;        // 0 = Q, 1 = K, 2 = V
        const int pi = 8 * j + (c & 7);
        const int dim = c < 8 ? pi : half + pi;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * mt + 4 * g + r;
            const float mine = acc[r];
            const float other = __shfl_xor(mine, 8, 64);
            if (m >= M || sec > 2) continue;
            const int b = m / a.q, row = m - b * a.q;
            const int L = __float_as_int(ep_in[r]);
            const int pos = L + row;                // cache slot of this block row
            if (pos >= a.S_max) {                   // the host checks capacity; never write past the cache
                atomicOr(a.err, 4);
                continue;
            }
            float out = mine;
            if (sec < 2) {
                // rotary position: the row's depth in the block (its ancestors
                // counted by the tree mask; row index for a chain), at most pos.
                // cos / sin come from the table (angle formed in double, rounded
                // to float).  Requesting them in the prologue, once the cache
                // lengths are in, measured slower.
                const int rpos = a.mask ? L + __popcll(a.mask[m]) - 1 : pos;
                const float2 csn = *reinterpret_cast<const float2*>(a.rope + ((size_t)rpos * half + pi) * 2);
                const float cs = csn.x, sn = csn.y;
                out = c < 8 ? mine * cs - other * sn : other * sn + mine * cs;
            }
            if (sec == 0) {
                reinterpret_cast<float*>(a.qbuf)[((size_t)m * H + h) * Dh + dim] = out;
            } else if (sec == 1) {
                reinterpret_cast<T*>(a.kc)[(((size_t)b * H + h) * a.S_max + pos) * Dh + dim] = to_elem<T>(out);
            } else {
                const size_t blk = ((size_t)b * H + h) * (a.S_max / 32) + pos / 32;
                reinterpret_cast<T*>(a.vc)[(blk * Dh + dim) * 32 + vperm(pos & 31)] = to_elem<T>(out);
            }
        }
    }
}

// What the epilogue of (tile, row tile mt) reads from memory: EP_RESID the residual values and the
// next RMSNorm's gain at this lane's column; EP_QKV the cache length of each row's sequence.
template <int EP>
__device__ __forceinline__ void epilogue_inputs(const GemmArgs& a, int tile, int mt, int c, int g, float (&ep_in)[4],
                                                float& gn) {
    const int n = tile * 16 + c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = 16 * mt + 4 * g + r;
        ep_in[r] = 0.f;
        if (EP == EP_RESID && m < a.M && n < a.N) ep_in[r] = a.resid[(size_t)m * a.ldy + n];
        if (EP == EP_QKV && m < a.M) ep_in[r] = __int_as_float(a.cache_len[m / a.q]);
    }
    gn = EP == EP_RESID && n < a.N ? a.gnext[n] : 0.f;
}

template <typename T, int EP, int MT, int NTW, bool XF>
// Workgroups of several tiles have 4 waves, the others at most 8.
__global__ void __launch_bounds__(NTW > 1 ? 256 : 512) gemm_kernel(GemmArgs a) {
    constexpr int U = Batch<T, EP, MT, XF>::U;
    using XT = typename XIn<T, XF>::type;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem_raw);   // [waves][MT][64]
    __shared__ float s_inv[64];

    const int nw = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = lane & 15, g = lane >> 4;
    const int M = a.M;
    // a split residual GEMM: workgroup (kpart, group of NTW tiles) holds waves kpart * nw .. of each
    // of its tiles' nwt
    const bool split = EP == EP_RESID && a.ksplit > 1;
    const int n_groups = (a.n_tiles + NTW - 1) / NTW;
    const int kpart = split ? (int)blockIdx.x / n_groups : 0;
    const int tile0 = ((int)blockIdx.x - kpart * n_groups) * NTW;
    const int nwt = split ? nw * a.ksplit : nw;
    const int gw = kpart * nw + wave;

    // this wave's contiguous slice of the contraction steps
    const int chunk = (a.k_steps + nwt - 1) / nwt;
    const int ks0 = gw * chunk;
    const int nks = max(0, min(a.k_steps, ks0 + chunk) - ks0);
    const T* wp[NTW];
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
        const int t = min(tile0 + j, a.n_tiles - 1);   // a tile past the end is read, not stored
        wp[j] = reinterpret_cast<const T*>(a.W) + (((size_t)t * a.k_steps + ks0) * 64 + lane) * 8;
    }

    // RMSNorm partial sums (wave w reduces rows w, w+nw, ...; the first two
    // are requested here, ahead of the weight stream) and the inputs of the
    // wave's first epilogue tiles.
    constexpr int NSQ = 4;   // ssq partials per lane and row (n_ssq <= 256)
    float sq[2][NSQ];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < NSQ; ++t) {
            const int m = wave + j * nw, col = lane + 64 * t;
            sq[j][t] = (XF && m < M && col < a.n_ssq) ? a.ssq[(size_t)m * a.n_ssq + col] : 0.f;
        }
    // The NTW x MT reduced tiles go to the waves round-robin: tile pr = wave + i * nw is
    // (column tile pr / MT, row tile pr % MT).
    constexpr int NPR = NTW * MT, NEP = (NPR + 3) / 4;   // 4 waves or more but for short contractions
    float ep_in[NEP][4], gnv[NEP];
#pragma unroll
    for (int i = 0; i < NEP; ++i) {
        const int pr = wave + i * nw;
        gnv[i] = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) ep_in[i][r] = 0.f;
        if (!split && pr < NPR && tile0 + pr / MT < a.n_tiles)
            epilogue_inputs<EP>(a, tile0 + pr / MT, pr % MT, c, g, ep_in[i], gnv[i]);
    }

    f32x4_t acc[NTW][MT];
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[j][mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Both weight batches are in flight before anything waits, then the loop
    // keeps two in flight.
    Frag<T> w0[U][NTW], w1[U][NTW];
    XT x0[U][MT], x1[U][MT];
    // X rows [0, M) as a buffer resource; lane offsets in bytes (rows past M
    // point past its end and read zeros without a memory access)
    constexpr uint32_t xes = sizeof(XT) / 8;   // bytes per X element as stored
    const uint32_t x_bytes = (uint32_t)M * (uint32_t)a.ldx * xes;
    const __amdgpu_buffer_rsrc_t xrs = buf_rsrc(XF ? (const void*)a.xf : a.xa, x_bytes);
    uint32_t xr[MT], xst[MT];   // lane offset of the slice's first step; bytes per step (the tile's rows x 32)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int rows = mt < MT - 1 ? 16 : M - 16 * (MT - 1);
        xst[mt] = 32u * rows * xes;
        xr[mt] = c < rows ? ((uint32_t)(16 * mt) * a.ldx + ((ks0 * 4 + g) * rows + c) * 8) * xes : x_bytes;
    }
    if (nks > 0) {
        load_batch<T, XT, MT, NTW, U>(w0, x0, wp, xrs, xr, xst, 0, nks);
        load_batch<T, XT, MT, NTW, U>(w1, x1, wp, xrs, xr, xst, U, nks);
    }

    // row scales 1/rms, needed before the first matrix-core step (rows past
    // the two prefetched ones, and partials past 64 * NSQ columns, are read now)
    float inv[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) inv[mt] = 1.f;
    if (XF) {
        for (int m = wave, j = 0; m < M; m += nw, ++j) {
            float v = 0.f;
            if (j < 2) {
#pragma unroll
                for (int t = 0; t < NSQ; ++t) v += sq[j < 1 ? 0 : 1][t];
                for (int col = lane + 64 * NSQ; col < a.n_ssq; col += 64) v += a.ssq[(size_t)m * a.n_ssq + col];
            } else {
                for (int col = lane; col < a.n_ssq; col += 64) v += a.ssq[(size_t)m * a.n_ssq + col];
            }
            v = wave_sum(v);
            if (lane == 0) s_inv[m] = 1.0f / sqrtf(v / (float)a.K + a.eps);
        }
        __syncthreads();
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int m = 16 * mt + c;
            inv[mt] = m < M ? s_inv[m] : 0.f;
        }
    }

    if (nks > 0) {
        // steady state: batches s (buffers 0) and s + U (buffers 1) are in
        // flight; each is refilled with the batch two ahead once consumed
        int s = 0;
        for (; s + 4 * U <= nks; s += 2 * U) {
            step_batch<T, XF, XT, MT, NTW, U>(acc, w0, x0, inv, wp, xrs, xr, xst, s + 2 * U);
            step_batch<T, XF, XT, MT, NTW, U>(acc, w1, x1, inv, wp, xrs, xr, xst, s + 3 * U);
        }
        // tail: steps s .. nks-1 (fewer than 4U), the first two batches loaded
        // (unconditional refills here, or one straight-line path per remaining
        // count, measured slower on MI355X)
        mma_batch<T, XF, XT, MT, NTW, U>(acc, w0, x0, inv);
        if (s + 2 * U < nks) load_batch<T, XT, MT, NTW, U>(w0, x0, wp, xrs, xr, xst, s + 2 * U, nks);
        if (s + U < nks) mma_batch<T, XF, XT, MT, NTW, U>(acc, w1, x1, inv);
        if (s + 3 * U < nks) load_batch<T, XT, MT, NTW, U>(w1, x1, wp, xrs, xr, xst, s + 3 * U, nks);
        if (s + 2 * U < nks) mma_batch<T, XF, XT, MT, NTW, U>(acc, w0, x0, inv);
        if (s + 3 * U < nks) mma_batch<T, XF, XT, MT, NTW, U>(acc, w1, x1, inv);
    }

    if (split) {   // raw partial rows of this wave's slice, added by the row kernel that follows
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
            if (tile0 + j >= a.n_tiles) break;
            const int n = (tile0 + j) * 16 + c;
            float* pp = a.part + (size_t)gw * M * a.N + n;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = 16 * mt + 4 * g + r;
                    if (m < M && n < a.N) pp[(size_t)m * a.N] = acc[j][mt][r];
                }
        }
        return;
    }

    // cross-wave reduction in wave order: every wave's partial tiles go to LDS, then each wave sums
    // its share of the tiles and runs their epilogues (one wave for all of them is a serial chain of
    // table loads and stores that the others wait for: 7B, 44 rows, 4 tiles per workgroup, QKV 45.8 ->
    // 31.0 us, gate/up 51.7 -> 44.3 us; 24 rows QKV 28.7 -> 25.5 us)
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) red[(wave * NPR + j * MT + mt) * 64 + lane] = acc[j][mt];
    __syncthreads();
    auto finish = [&](int pr, const float (&ein)[4], float gn) {
        const int tile = tile0 + pr / MT;
        if (tile >= a.n_tiles) return;
        f32x4_t v = red[pr * 64 + lane];
        for (int w = 1; w < nw; ++w) v += red[(w * NPR + pr) * 64 + lane];
        epilogue<T, EP>(a, tile, pr % MT, v, ein, gn, c, g);
    };
#pragma unroll
    for (int i = 0; i < NEP; ++i)
        if (wave + i * nw < NPR) finish(wave + i * nw, ep_in[i], gnv[i]);
    for (int pr = wave + NEP * nw; pr < NPR; pr += nw) {   // fewer than 4 waves
        float ein[4], gn = 0.f;
        if (tile0 + pr / MT < a.n_tiles) epilogue_inputs<EP>(a, tile0 + pr / MT, pr % MT, c, g, ein, gn);
        finish(pr, ein, gn);
    }
}

template <typename T, int EP, bool XF>
static hipError_t launch_mt(const GemmPlan& p, const GemmArgs& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const dim3 grid(p.grid), block(64 * p.waves);
    if (p.waves > (p.ntw > 1 ? 4 : 8) || !gemm_instance(EP, p.mt, p.ntw, XF)) return hipErrorInvalidValue;
    const bool split = p.ksplit > 1;   // ev1 is then the row kernel's
    if (split && (EP != EP_RESID || !a.part || a.ksplit != p.ksplit ||
                  p.grid != (a.n_tiles + p.ntw - 1) / p.ntw * p.ksplit))
        return hipErrorInvalidValue;
    if (!split && a.ksplit > 1) return hipErrorInvalidValue;
    auto go = [&](auto kernel) {
        if (ev0) hipExtLaunchKernelGGL(kernel, grid, block, p.lds_bytes, s, ev0, split ? nullptr : ev1, 0, a);
        else hipLaunchKernelGGL(kernel, grid, block, p.lds_bytes, s, a);
    };
    constexpr int NW = EP == EP_RESID ? 4 : 3;
    if (p.mt == 1 && p.ntw == 1) go(gemm_kernel<T, EP, 1, 1, XF>);
    else if constexpr (!XF) {
        switch (p.mt * 10 + p.ntw) {
            case 21: go(gemm_kernel<T, EP, 2, 1, false>); break;
            case 31: go(gemm_kernel<T, EP, 3, 1, false>); break;
            case 41: go(gemm_kernel<T, EP, 4, 1, false>); break;
            case 20 + NW: go(gemm_kernel<T, EP, 2, NW, false>); break;
            case 30 + NW: go(gemm_kernel<T, EP, 3, NW, false>); break;
            case 40 + NW: go(gemm_kernel<T, EP, 4, NW, false>); break;
            default: return hipErrorInvalidValue;
        }
    } else return hipErrorInvalidValue;
    return hipGetLastError();
}

// RMSNorm-input GEMMs (QKV, gate/up, LM head) read float x o g rows, or those
// rows already normalised and rounded (blocks of more than one row tile); O
// and down read element-type rows (attention output, SwiGLU product).
template <typename T>
static hipError_t launch_t(int ep, const GemmPlan& p, const GemmArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const bool xf = a.xf != nullptr;
    if (xf && !a.ssq) return hipErrorInvalidValue;
    switch (ep) {
        case EP_STORE:
            return xf ? launch_mt<T, EP_STORE, true>(p, a, s, e0, e1) : launch_mt<T, EP_STORE, false>(p, a, s, e0, e1);
        case EP_QKV: return xf ? launch_mt<T, EP_QKV, true>(p, a, s, e0, e1) : launch_mt<T, EP_QKV, false>(p, a, s, e0, e1);
        case EP_RESID: return xf ? hipErrorInvalidValue : launch_mt<T, EP_RESID, false>(p, a, s, e0, e1);
        case EP_SWIGLU:
            return xf ? launch_mt<T, EP_SWIGLU, true>(p, a, s, e0, e1) : launch_mt<T, EP_SWIGLU, false>(p, a, s, e0, e1);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm(int dtype, int ep, const GemmPlan& p, const GemmArgs& a, hipStream_t s, hipEvent_t ev0,
                       hipEvent_t ev1) {
    if (a.M < 1 || a.M > 64 || p.waves < 1 || p.waves > 16) return hipErrorInvalidValue;
    return dtype == 1 ? launch_t<uint16_t>(ep, p, a, s, ev0, ev1) : launch_t<float>(ep, p, a, s, ev0, ev1);
}

}  // namespace sdsat

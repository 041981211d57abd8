// Matrix-core GEMM for blocks of many rows (the prompt prefill before the
// draft/verify loop, Section 2.1): C[M, N] = A[M, K] . W[N, K]^T with A the
// normalised activations (element type, fragment order) and C float.  At
// hundreds of rows a weight byte feeds hundreds of flops, so unlike the decode
// GEMM this one is bound by the matrix cores and by how often operands are
// re-read, not by HBM.  Float models take prefill_gemm_kernel on the caller's
// row-major [out, in] weights -- up to three matrices stacked along N (Q | K |
// V, gate | up) -- and bf16 models prefill_mma_kernel on the packed ones.
//
// prefill_gemm_kernel: a workgroup of WM x WN waves computes a BM x BN tile of
// C, each wave a (16 TM) x (16 TN) sub-tile of matrix-core 16x16 tiles.  The
// contraction runs in stages of BK columns; both operands' stage tiles are
// staged in LDS (double-buffered), with the global loads of the next two stages
// in flight in registers while the current stage's fragments are read from LDS
// and multiplied; one barrier per stage.  LDS rows are padded by 32 bytes
// against bank conflicts.  Every element of C is accumulated by one wave in one
// fixed order of k, so results repeat bit for bit (in both kernels).
// Workgroups that share a weight tile (the same N tile, different M tiles) are
// placed on the same XCD (workgroups go to the 8 XCDs round-robin), so the
// weights come from HBM once and the other row tiles read them from that L2.
// Epilogues: C as float (O, down, LM head), or, from the C tile read back
// through LDS, RoPE with Q to its float buffer and K / V into the cache (QKV),
// or silu(gate) * up in the element type (gate | up) -- no float C round trip
// and no separate row kernel for these two.
#include "device.h"
#include "kernels.h"

namespace sdsat {

namespace {

// Stage geometry: BK contraction elements per LDS stage.
template <typename T, int BK_> struct PTile {
    static constexpr int BK = BK_;
    static constexpr int EPC = 16 / sizeof(T);          // elements per 16-byte chunk
    static constexpr int LDR = BK + 32 / sizeof(T);     // LDS row stride in elements (32 bytes of padding)
};

// Global -> registers: this thread's chunks of the A and W step tiles.  The loads are unconditional
// (indices clamped into the operands, the chunks past M, N or K zeroed when they are written to LDS), so
// the loop has no divergent branches and the waits for a register set count only the loads before it.
template <typename T, int BM, int BN, int NT, int BK, int EP>
struct StepLoad {
    static constexpr int EPC = PTile<T, BK>::EPC;
    static constexpr int CPR = PTile<T, BK>::BK / EPC;        // chunks per row of a stage tile
    static constexpr int NA = (BM * CPR + NT - 1) / NT, NW = (BN * CPR + NT - 1) / NT;
    static_assert(NA * NT == BM * CPR || NA == 1, "whole chunks per thread");
    static_assert(NW * NT == BN * CPR || NW == 1, "whole chunks per thread");
    u32x4_t a[NA], w[NW];
    bool ka[NA], kw[NW];

    __device__ __forceinline__ void load(const PrefillGemmArgs& p, int m0, int n0, int k0, int tid) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int c = tid + NT * i, kc = k0 + (c % CPR) * EPC, m = m0 + c / CPR;
            ka[i] = m < p.M && kc < p.K;
            a[i] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const T*>(p.A) +
                                                     frag_off(min(m, p.M - 1), min(kc, p.K - EPC), p.lda, (p.M + 15) & ~15));
        }
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int c = tid + NT * i, kc = k0 + (c % CPR) * EPC;
            int j, nn;
            if constexpr (EP == PG_SWIGLU) {
                // the tile's first BN / 2 rows are gate rows n0 / 2 .., the others the same up rows
                const int l = c / CPR, f = n0 / 2 + l % (BN / 2);
                j = l / (BN / 2);
                kw[i] = f < p.n_per && kc < p.K;
                nn = j * p.n_per + min(f, p.n_per - 1);
            } else {
                const int n = n0 + c / CPR;
                kw[i] = n < p.N && kc < p.K;
                nn = min(n, p.N - 1);
                j = nn / p.n_per;
            }
            // matrix j as an element offset from W0 (arithmetic, not a branch per lane; the pointer
            // stays a global one, so the load is a global load)
            const T* w0 = reinterpret_cast<const T*>(p.W0);
            const ptrdiff_t d1 = (reinterpret_cast<intptr_t>(p.W1) - reinterpret_cast<intptr_t>(p.W0)) / (ptrdiff_t)sizeof(T);
            const ptrdiff_t d2 = (reinterpret_cast<intptr_t>(p.W2) - reinterpret_cast<intptr_t>(p.W0)) / (ptrdiff_t)sizeof(T);
            const ptrdiff_t off = j == 0 ? 0 : (j == 1 ? d1 : d2);
            // cached: the other row tiles of this column tile read the same weights from L2
            w[i] = *reinterpret_cast<const u32x4_t*>(w0 + off + (ptrdiff_t)(nn - j * p.n_per) * p.K + min(kc, p.K - EPC));
        }
    }
    __device__ __forceinline__ void store(T* sa, T* sw, int tid) const {
        constexpr int LDR = PTile<T, BK>::LDR;
        const u32x4_t zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int c = tid + NT * i;
            if (NA * NT == BM * CPR || c < BM * CPR)
                *reinterpret_cast<u32x4_t*>(sa + (c / CPR) * LDR + (c % CPR) * EPC) = ka[i] ? a[i] : zero;
        }
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            const int c = tid + NT * i;
            if (NW * NT == BN * CPR || c < BN * CPR)
                *reinterpret_cast<u32x4_t*>(sw + (c / CPR) * LDR + (c % CPR) * EPC) = kw[i] ? w[i] : zero;
        }
    }
};

// Fused epilogues read the workgroup's C tile back from LDS (float rows of BN + 4: the 16 columns a
// wave's lanes write per row group land in distinct banks).
template <int BM, int BN> struct CTile { static constexpr int LD = BN + 4; static constexpr int BYTES = BM * LD * 4; };

template <typename T, int WM, int WN, int TM, int TN, int BK, int EP>
__global__ void __launch_bounds__(64 * WM * WN) prefill_gemm_kernel(PrefillGemmArgs p) {
    constexpr int BM = WM * TM * 16, BN = WN * TN * 16, NT = 64 * WM * WN;
    constexpr int LDR = PTile<T, BK>::LDR;
    constexpr int STAGE_BYTES = 2 * (BM + BN) * LDR * (int)sizeof(T);
    static_assert(EP == PG_STORE || CTile<BM, BN>::BYTES + BM * 4 <= STAGE_BYTES, "C tile fits the stage buffers");
    // the two stage buffers of A and W; after the last stage, the C tile of a fused epilogue
    __shared__ __align__(16) unsigned char smem[STAGE_BYTES];
    T (*s_a)[BM * LDR] = reinterpret_cast<T (*)[BM * LDR]>(smem);
    T (*s_w)[BN * LDR] = reinterpret_cast<T (*)[BN * LDR]>(smem + 2 * BM * LDR * sizeof(T));

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c = lane & 15, g = lane >> 4;
    // tile order: the row tiles of one column tile are consecutive on one XCD
    const int m_tiles = (p.M + BM - 1) / BM, n_tiles = (p.N + BN - 1) / BN;
    const int total = m_tiles * n_tiles;
    const int kpart = (int)blockIdx.x / total;
    int t = (int)blockIdx.x - kpart * total;
    if (total % 8 == 0) t = (t % 8) * (total / 8) + t / 8;
    const int m0 = (t % m_tiles) * BM, n0 = (t / m_tiles) * BN;
    const int wm = wave / WN, wn = wave % WN;

    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // this workgroup's share of the contraction (split-K: part kpart of p.ksplit, whole stages)
    const int stages_all = (p.K + BK - 1) / BK;
    const int per = (stages_all + p.ksplit - 1) / p.ksplit;
    const int st0 = kpart * per;
    const int steps = max(0, min(stages_all, st0 + per) - st0);
    const int kb = st0 * BK;
    // Two stages' global loads are in flight in registers while a third is read from LDS: at stage s
    // register set (s + 1) & 1 holds stage s + 1 (written to LDS after the stage-s products) and is
    // then reloaded with stage s + 3; set s & 1 holds stage s + 2, still arriving.  Loads past the
    // last stage read clamped, in-bounds addresses; their stage tiles are never read.
    StepLoad<T, BM, BN, NT, BK, EP> r0, r1;
    r0.load(p, m0, n0, kb, tid);
    r1.load(p, m0, n0, kb + BK, tid);
    r0.store(s_a[0], s_w[0], tid);
    __syncthreads();
    r0.load(p, m0, n0, kb + 2 * BK, tid);
    auto stage = [&](int s, StepLoad<T, BM, BN, NT, BK, EP>& next) {
        const int buf = s & 1;
#pragma unroll
        for (int kk = 0; kk < BK; kk += 32) {
            Frag<T> fa[TM], fw[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[i] = Frag<T>::load(&s_a[buf][((wm * TM + i) * 16 + c) * LDR + kk + 8 * g]);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fw[j] = Frag<T>::load(&s_w[buf][((wn * TN + j) * 16 + c) * LDR + kk + 8 * g]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) mma(acc[i][j], fa[i], fw[j]);
        }
        // keep the LDS write after the products and the next loads before the following stage's: left
        // to itself the scheduler moves loads next to the write that consumes them, which then waits
        // out their latency
        __builtin_amdgcn_sched_barrier(0);
        next.store(s_a[buf ^ 1], s_w[buf ^ 1], tid);
        __syncthreads();
        next.load(p, m0, n0, kb + (s + 3) * BK, tid);
        __builtin_amdgcn_sched_barrier(0);
    };
    // stages in pairs, an odd last stage after the loop: with no exit between the two halves the
    // waits before each LDS write count only the other register set's loads (a conditional second
    // half makes the compiler wait for every load at the top of the loop)
    int s = 0;
    for (; s + 1 < steps; s += 2) {
        stage(s, r1);
        stage(s + 1, r0);
    }
    if (s < steps) stage(s, r1);
    // acc[i][j][r] = C[row 16 i + 4 g + r of the wave tile][column 16 j + c]
    if constexpr (EP == PG_STORE) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int n = n0 + (wn * TN + j) * 16 + c;
                if (n >= p.N) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = m0 + (wm * TM + i) * 16 + 4 * g + r;
                    if (m < p.M) p.C[(size_t)kpart * p.c_part + (size_t)m * p.ldc + n] = acc[i][j][r];
                }
            }
    } else {
        // the C tile to LDS (every wave is past its last fragment reads), then each thread takes
        // pairs of columns of a row
        constexpr int LDC = CTile<BM, BN>::LD;
        float* tile = reinterpret_cast<float*>(smem);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    tile[((wm * TM + i) * 16 + 4 * g + r) * LDC + (wn * TN + j) * 16 + c] = acc[i][j][r];
        __syncthreads();
        if constexpr (EP == PG_QKV) {
            // the tile rows' cache positions, once per row (-1: past the cache, flagged, not written)
            int* s_pos = reinterpret_cast<int*>(smem + CTile<BM, BN>::BYTES);
            for (int r = tid; r < BM; r += NT) {
                const int m = m0 + r;
                int pos = -1;
                if (m < p.M) {
                    const int b = m / p.q;
                    pos = p.cache_len[b] + (m - b * p.q);
                    if (pos >= p.S_max) {   // the host checks capacity; never write past the cache
                        atomicOr(p.err, 4);
                        pos = -1;
                    }
                }
                s_pos[r] = pos;
            }
            __syncthreads();
            const int hd = p.Dh / 2;
            if (n0 / p.n_per == 2 && (n0 + BN - 1) / p.n_per == 2) {
                // a V tile: consecutive threads take consecutive rows of a column, so the 32 keys of a
                // cache block (one key-permuted 64-byte run per dimension) are written together
#pragma unroll 4
                for (int it = tid; it < BM * BN; it += NT) {
                    const int col = it / BM, r = it % BM, n = n0 + col, pos = s_pos[r];
                    if (pos < 0 || n >= p.N) continue;
                    const int m = m0 + r, b = m / p.q, h = (n % p.n_per) / p.Dh, i = (n % p.n_per) % p.Dh;
                    T* vo = static_cast<T*>(p.vc) + (((size_t)b * p.H + h) * (p.S_max / 32) + pos / 32) * p.Dh * 32 +
                            vperm(pos & 31);
                    vo[(size_t)i * 32] = to_elem<T>(tile[r * LDC + col]);
                }
            } else {
                // RoPE pairs columns i and i + Dh / 2 of a head (heads of Dh | BN columns start at tile
                // column multiples of Dh); the segment (Q, K, V) and head follow from the column
                constexpr int ITEMS = BM * (BN / 2) / NT;
                static_assert(ITEMS * NT == BM * (BN / 2), "whole items per thread");
#pragma unroll
                for (int u = 0; u < ITEMS; ++u) {
                    const int it = tid + u * NT;
                    const int r = it / (BN / 2), pr = it % (BN / 2), pos = s_pos[r];
                    const int a = (pr / hd) * p.Dh + pr % hd, n = n0 + a;
                    if (pos < 0 || n >= p.N) continue;
                    const int m = m0 + r, b = m / p.q;
                    const int seg = n / p.n_per, h = (n % p.n_per) / p.Dh, i = pr % hd;
                    const float x1 = tile[r * LDC + a], x2 = tile[r * LDC + a + hd];
                    if (seg == 2) {
                        T* vo = static_cast<T*>(p.vc) + (((size_t)b * p.H + h) * (p.S_max / 32) + pos / 32) * p.Dh * 32 +
                                vperm(pos & 31);
                        vo[(size_t)i * 32] = to_elem<T>(x1);
                        vo[(size_t)(i + hd) * 32] = to_elem<T>(x2);
                        continue;
                    }
                    const float2 csn = *reinterpret_cast<const float2*>(p.rope + ((size_t)pos * hd + i) * 2);
                    const float cs = csn.x, sn = csn.y;
                    const float y1 = x1 * cs - x2 * sn, y2 = x1 * sn + x2 * cs;
                    if (seg == 0) {
                        float* qo = p.qbuf + ((size_t)m * p.H + h) * p.Dh;
                        qo[i] = y1;
                        qo[i + hd] = y2;
                    } else {
                        T* ko = static_cast<T*>(p.kc) + (((size_t)b * p.H + h) * p.S_max + pos) * p.Dh;
                        ko[i] = to_elem<T>(y1);
                        ko[i + hd] = to_elem<T>(y2);
                    }
                }
            }
        } else {
            // columns 0 .. BN / 2 - 1 hold gate outputs n0 / 2 .., the others the same up outputs
            for (int it = tid; it < BM * (BN / 2); it += NT) {
                const int r = it / (BN / 2), i = it % (BN / 2);
                const int m = m0 + r, f = n0 / 2 + i;
                if (m >= p.M || f >= p.n_per) continue;
                const float gate = tile[r * LDC + i], v = tile[r * LDC + BN / 2 + i];
                static_cast<T*>(p.u)[frag_off(m, f, p.ldu, (p.M + 15) & ~15)] = to_elem<T>(gate / (1.0f + expf(-gate)) * v);
            }
        }
    }
}

template <typename T, int WM, int WN, int TM, int TN, int BK>
hipError_t go(const PrefillGemmArgs& p, hipStream_t s) {
    constexpr int BM = WM * TM * 16, BN = WN * TN * 16;
    static_assert(BN == 128, "fused epilogues: heads of 64 or 128 columns and 64 gate | 64 up outputs per tile");
    const long tiles = (long)((p.M + BM - 1) / BM) * ((p.N + BN - 1) / BN);
    auto kern = prefill_gemm_kernel<T, WM, WN, TM, TN, BK, PG_STORE>;
    if (p.ep == PG_QKV) kern = prefill_gemm_kernel<T, WM, WN, TM, TN, BK, PG_QKV>;
    else if (p.ep == PG_SWIGLU) kern = prefill_gemm_kernel<T, WM, WN, TM, TN, BK, PG_SWIGLU>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * p.ksplit)), dim3(64 * WM * WN), 0, s, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------- bf16
// C = A . W^T with both operands in fragment order: A as the row kernels and
// epilogues write it (frag_off, whole 16-row tiles), W as launch_pack lays it
// out for the decode GEMM.  A matrix-core fragment is then 1 KiB of consecutive
// memory in both, and a stage (one 32-wide step of the contraction) of a
// BM x BN tile is BM / 16 + BN / 16 such runs.  Each goes from memory straight
// into LDS (global_load_lds, 16 bytes per lane: no staging registers, no LDS
// write instructions), NST stages deep, and is read back as linear 16-byte lane
// accesses without bank conflicts.
//
// Per stage a wave waits until its own loads of the next stage have landed
// (vmcnt counts them: PER per stage, in order), meets the others at the one
// barrier -- after which that stage is complete in LDS, and the present stage,
// whose fragments every wave already holds in registers, may be overwritten --
// requests the stage NST ahead into the freed buffer, reads the next stage's
// fragments and runs the present stage's products meanwhile.
//
// The sums run over k in one order whatever the tile, so the tile shape is free:
// larger wave tiles read less LDS per product, smaller ones fill the chip when
// there are few rows (plan_prefill_mma).
template <int N> __device__ __forceinline__ void wait_loads() {   // at most N loads outstanding, LDS reads done
    // (the builtin rather than asm: the compiler then knows that no LDS read is pending)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void load_to_lds(const unsigned char* g, unsigned char* l) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}

template <int WM, int WN, int TM, int TN, int NST, int EP>
__global__ void __launch_bounds__(64 * WM * WN, WM * WN >= 8 || NST * (WM * TM + WN * TN) <= 80 ? 2 : 1)
    prefill_mma_kernel(PrefillGemmArgs p) {
    using T = uint16_t;
    constexpr int BMT = WM * TM, BNT = WN * TN, NW = WM * WN;   // 16-row / 16-column tiles, waves
    constexpr int FR = BMT + BNT;                               // fragments per stage
    constexpr int PA = (BMT + NW - 1) / NW, PW = (BNT + NW - 1) / NW, PER = PA + PW;   // loads per wave and stage
    constexpr int STAGE = FR * 1024;
    static_assert(NST >= 2 && (NST - 1) * PER < 64, "vmcnt range");
    __shared__ __align__(1024) unsigned char smem[NST * STAGE];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c = lane & 15, g = lane >> 4;
    const int wm = wave / WN, wn = wave % WN;
    // tile order: consecutive tiles (8 row tiles of a column tile, then the next column tile) on one XCD
    const int mt_all = (p.M + 15) / 16;
    const int m_tiles = (mt_all + BMT - 1) / BMT, n_tiles = (p.n_tiles + BNT - 1) / BNT;
    const int total = m_tiles * n_tiles, per_xcd = (total + 7) / 8;
    const int kpart = (int)blockIdx.x / (8 * per_xcd), bid = (int)blockIdx.x - kpart * 8 * per_xcd;
    const int t = (bid % 8) * per_xcd + bid / 8;
    if (t >= total) return;
    const int grp = t / (8 * n_tiles), in = t - grp * 8 * n_tiles, gm = min(8, m_tiles - 8 * grp);
    const int mt0 = (8 * grp + in % gm) * BMT, nt0 = in / gm * BNT;

    const int per = prefill_mma_part(p.k_steps, p.ksplit), k0 = kpart * per;
    const int steps = min(p.k_steps, k0 + per) - k0;   // at least 1: launch_prefill_mma

    // this wave's fragments of a stage (where they do not divide, the last is repeated: the same bytes to
    // the same place); tiles past the end read the last one and are not stored
    const unsigned char* src[PER];
    int dst[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int f = i < PA ? min(wave * PA + i, BMT - 1) : min(wave * PW + i - PA, BNT - 1);
        const size_t tile = i < PA ? min(mt0 + f, mt_all - 1) : min(nt0 + f, p.n_tiles - 1);
        src[i] = static_cast<const unsigned char*>(i < PA ? p.A : p.Wp) + (tile * p.k_steps + k0) * 1024 + lane * 16;
        dst[i] = (i < PA ? f : BMT + f) * 1024;
    }
    auto request = [&](int st, int buf) {   // steps past the last repeat it: in bounds, never used
        const size_t off = (size_t)min(st, steps - 1) * 1024;
#pragma unroll
        for (int i = 0; i < PER; ++i) load_to_lds(src[i] + off, smem + buf * STAGE + dst[i]);
    };
    struct Frags { Frag<T> a[TM], w[TN]; };
    auto fetch = [&](Frags& f, int buf) {
        const unsigned char* s = smem + buf * STAGE + lane * 16;
#pragma unroll
        for (int j = 0; j < TN; ++j) f.w[j] = Frag<T>::load(reinterpret_cast<const T*>(s + (BMT + wn * TN + j) * 1024));
#pragma unroll
        for (int i = 0; i < TM; ++i) f.a[i] = Frag<T>::load(reinterpret_cast<const T*>(s + (wm * TM + i) * 1024));
    };
    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int s = 0; s < NST; ++s) request(s, s);
    Frags f0, f1;
    wait_loads<(NST - 1) * PER>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    fetch(f0, 0);
    int buf = 0;   // the present stage's buffer
    auto stage = [&](int s, const Frags& now, Frags& next) {
        wait_loads<(NST - 2) * PER>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        request(s + NST, buf);
        buf = buf + 1 == NST ? 0 : buf + 1;
        fetch(next, buf);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) mma(acc[i][j], now.a[i], now.w[j]);
        // issue order: a read (and, first, a request) between every few products, from the start; left to
        // itself the scheduler sinks the reads to the end of the stage, where their latency is exposed
        constexpr int NRD = TM + TN, GAP = TM * TN / NRD;
#pragma unroll
        for (int i = 0; i < NRD; ++i) {
            if (i < PER) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // global -> LDS
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);               // LDS read
            __builtin_amdgcn_sched_group_barrier(0x008, GAP, 0);             // product
        }
        __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - NRD * GAP, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = 0;
    for (; s + 1 < steps; s += 2) {
        stage(s, f0, f1);
        stage(s + 1, f1, f0);
    }
    if (s < steps) stage(s, f0, f1);
    wait_loads<0>();   // no load may still be writing LDS when the workgroup ends

    // acc[i][j][r] = C[row 4g + r of row tile i][column c of column tile j]
    const int mt_w = mt0 + wm * TM, nt_w = nt0 + wn * TN;   // this wave's first tiles
    if constexpr (EP == PG_QKV) {
        // Written straight from the accumulators, RoPE's table loads and the cache's 2-byte stores take
        // 200 us of a 4092-row 7B launch's 524 us.  Each wave instead turns its tiles through a region of
        // the stage buffers (no other wave's: no barrier but the first) so that a lane holds 8
        // consecutive rotary pairs of one row (Q, K) or 4 consecutive keys of one dimension (V).
        constexpr int REGION = NST * STAGE / NW / 16 * 16, ROWS = 16 * TM;
        constexpr int LDQ = TN * 16 + 4, LDV = ROWS + 4;   // floats per staged row; 4 of padding spread the banks
        static_assert(TN <= 4, "a lane per row and column tile");
        static_assert(ROWS * 8 + (16 * LDQ > 16 * LDV ? 16 * LDQ : 16 * LDV) * 4 <= REGION, "the wave's LDS region");
        __syncthreads();   // every wave is past its last fragment read
        int2* s_pos = reinterpret_cast<int2*>(smem + wave * REGION);   // cache slot (-1: none) and sequence of each row
        float* st = reinterpret_cast<float*>(s_pos + ROWS);
        for (int r = lane; r < ROWS; r += 64) {
            const int m = 16 * mt_w + r, b = min(m, p.M - 1) / p.q;
            int pos = m < p.M ? p.cache_len[b] + (m - b * p.q) : -1;
            if (pos >= p.S_max) {   // the host checks capacity; never write past the cache
                atomicOr(p.err, 4);
                pos = -1;
            }
            s_pos[r] = make_int2(pos, b);
        }
        auto wave_sync = [] {   // LDS accesses of one wave are in order: only the compiler is held back
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        const int half = p.Dh / 2, tph = p.Dh / 16, nsec = p.H * tph;   // column tiles per head, per Q / K / V
        if (nt_w < 2 * nsec) {
            // lane -> (row of the tile, column tile j): rotary pairs 8jj .. 8jj + 7 of one head
            const int r = lane / TN, j = lane % TN, tile = nt_w + j, sec = tile / nsec;
            const bool mine = r < 16 && sec < 2;
            const int h = (tile % nsec) / tph, pi = 8 * (tile % tph);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                wave_sync();
#pragma unroll
                for (int jj = 0; jj < TN; ++jj)
#pragma unroll
                    for (int e = 0; e < 4; ++e) st[(4 * g + e) * LDQ + jj * 16 + c] = acc[i][jj][e];
                wave_sync();
                if (!mine) continue;
                const int2 ps = s_pos[16 * i + r];
                if (ps.x < 0) continue;
                const f32x4_t* x = reinterpret_cast<const f32x4_t*>(st + r * LDQ + j * 16);
                const f32x4_t* cs = reinterpret_cast<const f32x4_t*>(p.rope + ((size_t)ps.x * half + pi) * 2);
                float lo[8], hi[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float a = x[e / 4][e % 4], b = x[2 + e / 4][e % 4];
                    const float cc = cs[e / 2][2 * (e % 2)], sn = cs[e / 2][2 * (e % 2) + 1];
                    lo[e] = fmaf(a, cc, -(b * sn));   // rounded as in the float kernel above
                    hi[e] = fmaf(b, cc, a * sn);
                }
                if (sec == 0) {
                    float* q = p.qbuf + ((size_t)(16 * (mt_w + i) + r) * p.H + h) * p.Dh + pi;
                    Frag<float>::from_f32(lo).store(q);
                    Frag<float>::from_f32(hi).store(q + half);
                } else {
                    T* k = static_cast<T*>(p.kc) + (((size_t)ps.y * p.H + h) * p.S_max + ps.x) * p.Dh + pi;
                    Frag<T>::from_f32(lo).store(k);
                    Frag<T>::from_f32(hi).store(k + half);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int tile = nt_w + j;
            if (tile < 2 * nsec || tile >= p.n_tiles) continue;
            wave_sync();
#pragma unroll
            for (int i = 0; i < TM; ++i) *reinterpret_cast<f32x4_t*>(st + c * LDV + 16 * i + 4 * g) = acc[i][j];
            wave_sync();
            const int h = (tile % nsec) / tph, pi = 8 * (tile % tph);
            // lane -> (dimension, group of 4 keys): groups are aligned to the first row's slots, so 8 lanes
            // write a 32-key block's whole run of one dimension
            const int2 p0 = s_pos[0];
            const int off = p0.x < 0 ? 0 : p0.x & 3;
            for (int it = lane; it < 128 * ((ROWS / 4 + 8) / 8); it += 64) {
                const int col = (it >> 3) & 15, grp = (it & 7) + 8 * (it >> 7), rb = 4 * grp - off;
                if (rb >= ROWS) continue;
                const int dim = col < 8 ? pi + col : half + pi + col - 8;
                const int2 a = s_pos[max(rb, 0)], z = s_pos[min(rb + 3, ROWS - 1)];
                auto slot = [&](int2 ps) {
                    return static_cast<T*>(p.vc) +
                           ((((size_t)ps.y * p.H + h) * (p.S_max / 32) + ps.x / 32) * p.Dh + dim) * 32 + vperm(ps.x & 31);
                };
                const float* v = st + col * LDV + rb;
                if (rb >= 0 && rb + 3 < ROWS && a.x >= 0 && (a.x & 3) == 0 && z.x == a.x + 3 && z.y == a.y) {
                    *reinterpret_cast<uint2*>(slot(a)) = uint2{f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3])};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int row = rb + e;
                        if (row < 0 || row >= ROWS) continue;
                        const int2 ps = s_pos[row];
                        if (ps.x >= 0) *slot(ps) = to_elem<T>(v[e]);
                    }
                }
            }
        }
        return;
    }
    const int rows16 = (p.M + 15) & ~15;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int mt = mt_w + i;
        if (mt >= mt_all) break;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int tile = nt_w + j;
            if (tile >= p.n_tiles) break;
            if constexpr (EP == PG_STORE) {
                const int n = tile * 16 + c;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = 16 * mt + 4 * g + r;
                    if (m < p.M && n < p.N) p.C[(size_t)kpart * p.c_part + (size_t)m * p.ldc + n] = acc[i][j][r];
                }
            } else {
                const int f = 8 * tile + (c & 7);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = 16 * mt + 4 * g + r;
                    const float mine = acc[i][j][r], other = __shfl_xor(mine, 8, 64);
                    if (c >= 8 || m >= p.M) continue;
                    T* u = static_cast<T*>(p.u);
                    u[frag_off(m, f, p.ldu, rows16)] = to_elem<T>(mine / (1.0f + expf(-mine)) * other);
                    if (tile == p.n_tiles - 1)   // zero up to the padded length
                        for (int z = f + 8; z < p.ldu; z += 8) u[frag_off(m, z, p.ldu, rows16)] = 0;
                }
            }
        }
    }
}

template <int WM, int WN, int TM, int TN, int NST>
hipError_t go_mma(const PrefillGemmArgs& p, hipStream_t s) {
    const int total = (((p.M + 15) / 16 + WM * TM - 1) / (WM * TM)) * ((p.n_tiles + WN * TN - 1) / (WN * TN));
    const dim3 grid((unsigned)((total + 7) / 8 * 8 * p.ksplit)), block(64 * WM * WN);
    auto kern = prefill_mma_kernel<WM, WN, TM, TN, NST, PG_STORE>;
    if (p.ep == PG_QKV) kern = prefill_mma_kernel<WM, WN, TM, TN, NST, PG_QKV>;
    else if (p.ep == PG_SWIGLU) kern = prefill_mma_kernel<WM, WN, TM, TN, NST, PG_SWIGLU>;
    hipLaunchKernelGGL(kern, grid, block, 0, s, p);
    return hipGetLastError();
}

}  // namespace

int prefill_gemm_ksplit(int M, int N, int K) {
    const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
    if (K < 1024 || tiles >= 256) return 1;
    return tiles <= 128 && K >= 2048 ? 4 : 2;
}

// prefill_gemm_ksplit: a GEMM whose 128 x 128 tiles make less than one round of
// workgroups over the 256 compute units and whose contraction is long is split
// into parts whose partials the caller adds (O and down at 7B, 511 rows: 64
// tiles of 256 x 128, 4 parts, one round).  Float: 4 waves of 64 x 64, 32-wide
// stages.
hipError_t launch_prefill_gemm(int dtype, const PrefillGemmArgs& p, hipStream_t s) {
    if (p.M < 1 || p.N < 1 || p.K < 1 || p.K % 8 || p.n_per < 1 || p.N > 3 * p.n_per || !p.A || !p.W0 ||
        (p.N > p.n_per && !p.W1) || (p.N > 2 * p.n_per && !p.W2) || p.lda < p.K || p.ksplit < 1 || p.ksplit > kPrefillMaxSplit)
        return hipErrorInvalidValue;
    if (p.ep == PG_STORE) {
        if (!p.C || p.ldc < p.N || (p.ksplit > 1 && p.c_part < (size_t)p.M * p.ldc)) return hipErrorInvalidValue;
    } else if (p.ep == PG_QKV) {
        // heads tile the 128-column workgroup tiles; the segments are whole heads
        if (p.ksplit != 1 || p.N != 3 * p.n_per || (p.Dh != 64 && p.Dh != 128) || p.H < 1 || p.n_per != p.H * p.Dh ||
            p.q < 1 || p.M % p.q || p.S_max < 32 || p.S_max % 32 || !p.cache_len || !p.rope || !p.qbuf || !p.kc ||
            !p.vc || !p.err)
            return hipErrorInvalidValue;
    } else if (p.ep == PG_SWIGLU) {
        if (p.ksplit != 1 || p.N != 2 * p.n_per || !p.u || p.ldu < p.n_per) return hipErrorInvalidValue;
    } else {
        return hipErrorInvalidValue;
    }
    if (dtype != 1) return go<float, 2, 2, 4, 4, 32>(p, s);
    return launch_prefill_mma(plan_prefill_mma(p.M, p.n_tiles, p.k_steps, p.ksplit), p, s);
}

// The bf16 instances: workgroup tile (rows x columns), waves, stages in flight, and what one round of 256
// workgroups costs per 32-wide step (us, one workgroup per compute unit; `pair`: two fit one, both running).
// Measured on the 7B shapes at 70 .. 4092 rows; larger wave tiles cost less per product (256 x 256 0.80 us
// for four times the products of 128 x 128's 0.34), smaller ones leave fewer units idle in the last round.
struct MmaConfig { int bm, bn; float round, pair; };
static constexpr MmaConfig kMma[] = {
    {16, 16, 0.80f, 0.f}, {16, 12, 0.68f, 0.f}, {16, 8, 0.44f, 0.f}, {16, 6, 0.38f, 0.f},
    {8, 8, 0.34f, 0.47f}, {8, 6, 0.27f, 0.f}, {8, 4, 0.22f, 0.40f}, {8, 3, 0.19f, 0.30f},
};
int prefill_mma_configs() { return (int)(sizeof(kMma) / sizeof(kMma[0])); }

// The instance with the least estimated time: rounds of workgroups times their cost.  At 511 rows of the 7B
// model it takes 256 x 192 for gate | up (230 workgroups, 90 us; 256 x 256: 172 workgroups, 103 us;
// 128 x 128: 688, 116 us), 256 x 96 for QKV (256 workgroups, 58 us; 256 x 128: 192, 64 us); at 127 rows
// 128 x 96 (230, 47 us; 128 x 64: 344, 63 us) and 128 x 48 (256, 34 us); at 4092 rows 256 x 256 throughout
// (gate | up 640 us, 1.15 PFLOP/s; down 261 us, 1.4 PFLOP/s; with 128 x 128 tiles, register staging and
// row-major operands 891 and 469 us).
int plan_prefill_mma(int M, int n_tiles, int k_steps, int ksplit) {
    int best = 0;
    float least = 0.f;
    for (int i = 0; i < prefill_mma_configs(); ++i) {
        const MmaConfig& c = kMma[i];
        const long wg = (long)(((M + 15) / 16 + c.bm - 1) / c.bm) * ((n_tiles + c.bn - 1) / c.bn) * ksplit;
        float t;
        if (c.pair > 0.f) {
            const long rest = wg % 512;
            t = (float)(wg / 512) * c.pair + (rest > 256 ? c.pair : rest > 0 ? c.round : 0.f);
        } else {
            t = (float)((wg + 255) / 256) * c.round;
        }
        t *= (float)((k_steps + ksplit - 1) / ksplit);
        if (i == 0 || t < least) { least = t; best = i; }
    }
    return best;
}

hipError_t launch_prefill_mma(int cfg, const PrefillGemmArgs& p, hipStream_t s) {
    if (!p.A || !p.Wp || p.n_tiles < (p.N + 15) / 16 || p.k_steps < (p.K + 31) / 32 || p.lda != 32 * p.k_steps ||
        p.ksplit < 1 || (p.ksplit - 1) * prefill_mma_part(p.k_steps, p.ksplit) >= p.k_steps)   // no empty part
        return hipErrorInvalidValue;
    switch (cfg) {
        case 0: return go_mma<2, 4, 8, 4, 4>(p, s);
        case 1: return go_mma<2, 4, 8, 3, 5>(p, s);
        case 2: return go_mma<4, 2, 4, 4, 6>(p, s);
        case 3: return go_mma<4, 2, 4, 3, 6>(p, s);
        case 4: return go_mma<2, 2, 4, 4, 4>(p, s);
        case 5: return go_mma<4, 2, 2, 3, 5>(p, s);
        case 6: return go_mma<2, 2, 4, 2, 6>(p, s);
        case 7: return go_mma<4, 1, 2, 3, 6>(p, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace sdsat

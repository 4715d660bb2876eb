// Binary64 GEMM for the masked projection whose noise is too large for binary32
// cancellation (the Down projection at the sensitivity of Theorem 3): Out = A W^T (- C)
// with A (the binary64 masked input, or the mask itself for the correction) M x K,
// W N x K bfloat16 or float32 converted exactly to binary64, C M x N binary64.
//
// Bound by the matrix cores: v_mfma_f64_16x16x4_f64, 67 TFLOP/s in a loop of nothing else (59 with
// one wave per SIMD).  As the binary32 GEMM: tiles of 16-64 rows x 64 columns, whole rounds of 256
// unsplit and the rest split over K, both operands by 16-byte loads to LDS some 32-k stages
// ahead, swizzled, one barrier per K tile in the middle of its MFMAs, fragments read half a tile
// ahead.  W is converted as its fragments leave LDS.  Before, each 16-k tile went through
// registers into rows padded by one element, with four MFMAs per barrier and k.
// Llama-3.2-3B Down through the fused call: 128 tokens 190 -> 117 us (55 TFLOP/s), 256 tokens 365 -> 220,
// one token 100 -> 26; 250 x 700 x 1024 28.2 -> 19.4 us.
//
// An accumulator chain runs over 96 or 128 k and is then added into a second set of registers, as in the binary32
// GEMM.  Distance from the 64-bit result at noise of 1.66e8, mean over 1-250 tokens x 300-3072 columns, with
// the former K splits, with chains of 384 k and so: K = 264 7.6e-8, 1.03e-7, 7.4e-8; 768 7.7e-8, 9.3e-8, 7.5e-8;
// 9728 1.6e-7, 1.2e-7, 8.0e-8.  The additions run under the next chain's first MFMAs and cost nothing (384-k
// chains added at their end: 119 us for the 117 above).
#include "gemm_dev.hpp"

#include <algorithm>
#include <type_traits>

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

constexpr int D_NW = 4;           // waves of a workgroup, side by side along N
constexpr int D_NT = D_NW * WAVE;
constexpr int D_BK = 32;          // k of one stage: 256 bytes of an A row
constexpr int D_BN = 64;          // columns of a tile
constexpr int D_MAX_TM = 4;       // 16-row blocks of a tile
constexpr int D_CHAIN = 4;        // K tiles that one accumulator chain runs over at most

__device__ __attribute__((aligned(16))) const double f64_zeros[2] = {0.0, 0.0};

typedef const __attribute__((address_space(1))) void* glb_ptr_t;

template <int I, int BYTES>
__device__ __forceinline__ unsigned char* f64_stage()
{
    __shared__ __attribute__((aligned(16))) unsigned char buf[BYTES];
    return buf;
}

constexpr int f64_stage_bytes(int tm, bool wbf16) { return 16 * tm * 256 + D_BN * (wbf16 ? 64 : 128); }
// Stages: as many as let two workgroups share a CU's 160 KB, up to 4.
constexpr int f64_stages(int tm, bool wbf16) { return std::min(4, 78 * 1024 / f64_stage_bytes(tm, wbf16)); }

// Blocks 0 .. nfull - 1: whole tiles, Out = acc - C (C may be null), as binary64 (OUT64) or rounded
// to binary32.  Then rem tiles in splits of ktps K tiles: part gets each split's sums.
template <int TM, bool WBF16, bool OUT64>
__global__ void __launch_bounds__(D_NT, 2)
gemm_f64_kernel(const double* __restrict__ A, int64_t lda, const void* __restrict__ Wv, int64_t ldw,
                const double* __restrict__ C, int64_t ldc, void* __restrict__ Out, int64_t ldo, double* __restrict__ part,
                int M, int N, int K, int mtiles, int nfull, int ktps, int rem)
{
    constexpr int BM = 16 * TM;
    constexpr int S = f64_stages(TM, WBF16);
    constexpr int AB = BM * 256, SB = f64_stage_bytes(TM, WBF16);
    constexpr int LA = TM;                                // 1 KB loads to LDS per wave and stage: A
    constexpr int LW = WBF16 ? 1 : 2;                     // and W
    static_assert(S >= 3 && (S - 1) * (LA + LW) < 64, "stages");
    const int tid = threadIdx.x, lane = tid % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int ktiles = (K + D_BK - 1) / D_BK;
    const int b = blockIdx.x;
    const bool whole = b < nfull;
    const int split = whole ? 0 : (b - nfull) / rem, tt = whole ? 0 : (b - nfull) % rem;
    const int tile = whole ? (int)splitee::xcd_logical_block((uint32_t)b, (uint32_t)nfull) : nfull + tt;
    const int m0 = (tile % mtiles) * BM, n0 = (tile / mtiles) * D_BN;
    const int kt0 = whole ? 0 : split * ktps;
    const int nk = (whole ? ktiles : min(kt0 + ktps, ktiles)) - kt0;

    // A: load t of this wave fills stage rows 4 j .. 4 j + 3, j = wave + 4 t; lane l writes slot
    // l % 16 of row l / 16, holding the row's 16-byte chunk slot ^ (row % 16)
    const double* ap[LA];
    int ak[LA]; // columns of the row left at the load's first K tile (none for a row past M)
#pragma unroll
    for (int t = 0; t < LA; ++t) {
        const int row = 4 * (wave + D_NW * t) + lane / 16, gm = m0 + row;
        const int k = kt0 * D_BK + 2 * ((lane % 16) ^ (row & 15));
        const bool ok = gm < M;
        ap[t] = A + (ok ? (int64_t)gm * lda + k : 0);
        ak[t] = ok ? K - k : 0;
    }
    // W: 4 chunks of a 64-byte bfloat16 row at slot chunk ^ ((row / 4) % 4), 16 rows per load, or
    // 8 chunks of a 128-byte float32 row at slot chunk ^ (row % 8)
    constexpr int WR = WBF16 ? 16 : 8, WC = WBF16 ? 4 : 8, WES = WBF16 ? 2 : 4;
    const char* wp[LW];
    int wk[LW];
#pragma unroll
    for (int t = 0; t < LW; ++t) {
        const int row = WR * (wave + D_NW * t) + lane / WC, gn = n0 + row;
        const int chunk = WBF16 ? (lane % 4) ^ ((row >> 2) & 3) : (lane % 8) ^ (row & 7);
        const int k = kt0 * D_BK + chunk * (16 / WES);
        const bool ok = gn < N;
        wp[t] = reinterpret_cast<const char*>(Wv) + (ok ? ((int64_t)gn * ldw + k) * WES : 0);
        wk[t] = ok ? K - k : 0;
    }

    unsigned char* const st[4] = {f64_stage<0, SB>(), f64_stage<1, SB>(), f64_stage<2, SB>(), f64_stage<(S > 3 ? 3 : 0), SB>()};
    // the loads of relative K tile t into stage q (zeros past the split's end and the matrix)
    auto issue = [&](int t, auto sc) {
        constexpr int q = decltype(sc)::value;
        const int k = t < nk ? t * D_BK : K; // past every row's end
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const double* p = k < ak[i] ? ap[i] + k : f64_zeros;
            __builtin_amdgcn_global_load_lds((glb_ptr_t)p, (lds_ptr_t)(st[q] + (wave + D_NW * i) * 1024), 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < LW; ++i) {
            const char* p = k < wk[i] ? wp[i] + (int64_t)k * WES : reinterpret_cast<const char*>(f64_zeros);
            __builtin_amdgcn_global_load_lds((glb_ptr_t)p, (lds_ptr_t)(st[q] + AB + (wave + D_NW * i) * 1024), 16, 0, 0);
        }
    };

    f64x4 acc[TM], sum[TM]; // acc is added into sum every ring turn (3 or 4 K tiles)
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[i] = sum[i] = f64x4{0.0, 0.0, 0.0, 0.0};

    // lane (r, g) of the MFMA operands: row r of a 16-row block, k = 8 g + e in instruction e of the K
    // tile's eight (the same assignment for A and W)
    const int fr = lane % 16, fg = lane / 16;
    f64x2 a0[TM][2], a1[TM][2];
    f32x4_t wr[2];
    double w[2][4];
    auto read_a = [&](const unsigned char* s, int h, f64x2 (&a)[TM][2]) { // k = 8 g + 4 h .. + 3
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                a[i][c] = *reinterpret_cast<const f64x2*>(s + (16 * i + fr) * 256 + (((4 * fg + 2 * h + c) ^ fr) << 4));
    };
    auto read_w = [&](const unsigned char* s) { // raw: one 16-byte word (bfloat16) or two
        const int row = 16 * wave + fr;
        if (WBF16) {
            wr[0] = *reinterpret_cast<const f32x4_t*>(s + AB + row * 64 + ((fg ^ ((row >> 2) & 3)) << 4));
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                wr[h] = *reinterpret_cast<const f32x4_t*>(s + AB + row * 128 + (((2 * fg + h) ^ (row & 7)) << 4));
        }
    };
    auto widen_w = [&](int h) { // this half's four k
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (WBF16) {
                const uint32_t d = __float_as_uint(wr[0][2 * h + e / 2]);
                w[h][e] = (double)__uint_as_float(e % 2 ? d & 0xFFFF0000u : d << 16);
            } else {
                w[h][e] = (double)wr[h][e];
            }
        }
    };
    auto mul = [&](const f64x2 (&a)[TM][2], int h) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
                acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][e / 2][e % 2], w[h][e], acc[i], 0, 0, 0);
    };
    // K tile t in stage q, its W and the first half of its A in registers.  First half: multiply
    // while the second half of A is read.  Then every wave is done with stage q, and tile t + 1
    // (this wave's loads of it: all but the S - 2 younger tiles') is in everywhere behind the
    // barrier.  Second half: multiply while tile t + 1's first fragments are read and
    // tile t + S goes into stage q.
    auto step = [&](int t, auto sc) {
        constexpr int q = decltype(sc)::value;
        read_a(st[q], 1, a1);
        mul(a0, 0);
#pragma unroll
        for (int i = 0; i < 2 * TM; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * TM, 0);
        __builtin_amdgcn_sched_barrier(0);
        wait_vmem<(S - 2) * (LA + LW)>();
        __builtin_amdgcn_s_waitcnt((0 << 8) | (7 << 4) | 15 | (3 << 14)); // lgkmcnt(0): a1 is in
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        widen_w(1);
        read_w(st[(q + 1) % S]);
        read_a(st[(q + 1) % S], 0, a0);
        issue(t + S, sc);
        mul(a1, 1);
#pragma unroll
        for (int i = 0; i < 2 * TM + LW; ++i) {
            if (i < 2 * TM) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int i = 0; i < LA + LW; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * TM, 0);
        __builtin_amdgcn_sched_barrier(0);
        widen_w(0);
    };
    auto flush = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            sum[i] += acc[i];
            acc[i] = f64x4{0.0, 0.0, 0.0, 0.0};
        }
    };

#define D_IC(I) std::integral_constant<int, I>{}
    issue(0, D_IC(0));
    issue(1, D_IC(1));
    issue(2, D_IC(2));
    if constexpr (S > 3) issue(3, D_IC(3));
    wait_vmem<(S - 1) * (LA + LW)>();
    __builtin_amdgcn_s_barrier();
    read_w(st[0]);
    read_a(st[0], 0, a0);
    widen_w(0);
    // a turn: the chains' flush, in one block with the MFMAs that begin the next chain (from zero, so acc is
    // not cleared, and the additions run under them), then the ring's K tiles
    static_assert(S <= D_CHAIN, "chains too long");
    int t = 0;
    for (; t + S <= nk; t += S) {
        flush();
        step(t, D_IC(0));
        step(t + 1, D_IC(1));
        step(t + 2, D_IC(2));
        if constexpr (S > 3) step(t + 3, D_IC(3));
    }
    // the last, partial turn
    flush();
    if (t < nk) step(t, D_IC(0));
    if (t + 1 < nk) step(t + 1, D_IC(1));
    if constexpr (S > 3) if (t + 2 < nk) step(t + 2, D_IC(2));
#undef D_IC
    wait_vmem<0>(); // loads past the last tile (zeros) have landed before the workgroup ends
    flush();

    if (!whole) { // element e of block i of lane l at ((i 4 + e) 64 + l)
        double* mp = part + ((int64_t)(b - nfull) * D_NW + wave) * (TM * 256);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) mp[(4 * i + e) * 64 + lane] = sum[i][e];
        return;
    }
    // accumulator element e of lane l: row l / 16 + 4 e, column l % 16 of its 16 x 16 block
    // (v_mfma_f64_16x16x4_f64 on gfx950, checked against a binary64 reference); every C load before the
    // first subtraction, elements outside M x N load C[0] and store nothing
    const int col = n0 + 16 * wave + fr;
    double cv[TM][4];
    if (C) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = m0 + 16 * i + fg + 4 * e;
                cv[i][e] = C[row < M && col < N ? (int64_t)row * ldc + col : 0];
            }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = m0 + 16 * i + fg + 4 * e;
            if (row >= M || col >= N) continue;
            const double y = C ? sum[i][e] - cv[i][e] : sum[i][e];
            if (OUT64)
                reinterpret_cast<double*>(Out)[(int64_t)row * ldo + col] = y;
            else
                reinterpret_cast<float*>(Out)[(int64_t)row * ldo + col] = (float)y;
        }
}

// The split tiles' partials added in split order, minus C when it is given.  Thread u handles one
// element of one wave's partial, in the order they were written in.
constexpr int D_MAX_KS = 16;

template <int TM, bool OUT64>
__global__ void __launch_bounds__(256)
f64_sum_kernel(const double* __restrict__ part, int ksplit, const double* __restrict__ C, int64_t ldc,
               void* __restrict__ Out, int64_t ldo, int M, int N, int mtiles, int nfull, int rem)
{
    constexpr int PER = TM * 256, TILE = D_NW * PER; // elements of a wave's and a tile's partial
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= rem * TILE) return;
    const int tt = u / TILE, e = u - tt * TILE, wave = e / PER, f = e - wave * PER;
    const int lane = f % 64, ie = f / 64, tile = nfull + tt;
    const int row = (tile % mtiles) * 16 * TM + 16 * (ie / 4) + lane / 16 + 4 * (ie % 4);
    const int col = (tile / mtiles) * D_BN + 16 * wave + lane % 16;
    if (row >= M || col >= N) return;
    const double cv = C ? C[(int64_t)row * ldc + col] : 0.0;
    // every split's partial in flight together (one past ksplit loads the first again and is not added)
    double v[D_MAX_KS];
#pragma unroll
    for (int q = 0; q < D_MAX_KS; ++q) v[q] = part[((int64_t)(q < ksplit ? q : 0) * rem + tt) * TILE + e];
    double y = v[0];
#pragma unroll
    for (int q = 1; q < D_MAX_KS; ++q)
        if (q < ksplit) y += v[q];
    if (C) y -= cv;
    if (OUT64)
        reinterpret_cast<double*>(Out)[(int64_t)row * ldo + col] = y;
    else
        reinterpret_cast<float*>(Out)[(int64_t)row * ldo + col] = (float)y;
}

struct F64Plan {
    int tm, mtiles;
    int nfull, rem, ksplit, ktps; // whole tiles, split tiles, their splits and K tiles per split
    size_t part_bytes;
};

constexpr size_t F64_MAX_PART = size_t(128) << 20;

// The tile height and the split of the tiles that fill no whole round of 256 workgroups, by the
// launch's modelled time, as plan_f32: a K tile takes 0.24 tm + 0.06 us of a CU (measured unsplit at 128
// tokens x 3072 columns: 0.33, 0.54, 0.77 and 1.02), more with one workgroup alone on it, a workgroup 1 us
// besides, the sum 4 us and its partials' traffic at 5 TB/s.
F64Plan plan_f64(int64_t M, int64_t N, int64_t K)
{
    const int ktiles = (int)((K + D_BK - 1) / D_BK);
    F64Plan best{};
    double best_cost = -1.0;
    for (int tm = 1; tm <= D_MAX_TM && 16 * (tm - 1) < M; ++tm) {
        const int64_t mtiles = (M + 16 * tm - 1) / (16 * tm), tiles = mtiles * ((N + D_BN - 1) / D_BN);
        const int64_t full = tiles / 256 * 256, rem = tiles - full;
        const double ktile = 0.24 * tm + 0.06;
        for (int ks = 1; ks <= D_MAX_KS; ++ks) {
            if (ks > 1 && (rem == 0 || ktiles / ks < 4)) break;
            const int ktps = ktiles > 0 ? (ktiles + ks - 1) / ks : 1;
            if (ks > 1 && (ktiles + ktps - 1) / ktps != ks) continue;
            const size_t pb = ks > 1 ? (size_t)rem * ks * tm * 16 * D_BN * 8 : 0;
            if (pb > F64_MAX_PART) break;
            const int64_t wgs = rem * ks, rounds = (wgs + 255) / 256;
            const double alone = full == 0 && wgs <= 256 ? 1.0 + 0.25 / tm : 1.0;
            const double cost = (double)(full / 256) * (ktiles * ktile + 1.0) +
                                (double)rounds * (ktps * ktile * alone + 1.0) + (ks > 1 ? 4.0 + (double)pb * 2 / 5.0e6 : 0.0);
            if (best_cost >= 0 && cost >= best_cost) continue;
            best_cost = cost;
            best.tm = tm;
            best.mtiles = (int)mtiles;
            best.ksplit = ks;
            best.ktps = ktps;
            best.rem = (int)(ks > 1 ? rem : 0);
            best.nfull = (int)(ks > 1 ? full : tiles);
            best.part_bytes = pb;
        }
    }
    return best;
}

}  // namespace

namespace splitee_host {

size_t f64_gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) { return M > 0 && N > 0 ? plan_f64(M, N, K).part_bytes : 0; }

int launch_gemm_f64(const double* A, int64_t lda, const void* W, int w_type, int64_t ldw, const double* C,
                    int64_t ldc, void* Out, bool out64, int64_t ldo, int64_t M, int64_t N, int64_t K, void* ws,
                    size_t ws_bytes, hipStream_t s)
{
    if (M == 0 || N == 0) return SPLITEE_OK;
    const F64Plan p = plan_f64(M, N, K);
    if (ws_bytes < p.part_bytes || (p.part_bytes && !ws)) return SPLITEE_ERR_WORKSPACE;
    double* part = reinterpret_cast<double*>(ws);
    const dim3 grid((unsigned)(p.nfull + (int64_t)p.rem * p.ksplit));
    const dim3 g2((unsigned)((int64_t)p.rem * p.tm * 4));
    const bool bf16 = w_type == SPLITEE_BF16;
#define D_RUN2(TM, WB, O64)                                                                                        \
    do {                                                                                                           \
        hipLaunchKernelGGL((gemm_f64_kernel<TM, WB, O64>), grid, dim3(D_NT), 0, s, A, lda, W, ldw, C, ldc, Out, ldo, \
                           part, (int)M, (int)N, (int)K, p.mtiles, p.nfull, p.ktps, p.rem);                        \
        if (p.ksplit > 1)                                                                                          \
            hipLaunchKernelGGL((f64_sum_kernel<TM, O64>), g2, dim3(256), 0, s, part, p.ksplit, C, ldc, Out, ldo,   \
                               (int)M, (int)N, p.mtiles, p.nfull, p.rem);                                          \
    } while (0)
#define D_RUN(TM)                                                                                                  \
    do {                                                                                                           \
        if (bf16) { if (out64) D_RUN2(TM, true, true); else D_RUN2(TM, true, false); }                             \
        else { if (out64) D_RUN2(TM, false, true); else D_RUN2(TM, false, false); }                                \
    } while (0)
    switch (p.tm) {
    case 1: D_RUN(1); break;
    case 2: D_RUN(2); break;
    case 3: D_RUN(3); break;
    default: D_RUN(4); break;
    }
#undef D_RUN
#undef D_RUN2
    return hipGetLastError() == hipSuccess ? SPLITEE_OK : SPLITEE_ERR_HIP;
}

}  // namespace splitee_host

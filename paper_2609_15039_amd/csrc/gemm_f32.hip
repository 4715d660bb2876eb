// binary32 MFMA GEMM (gfx950): Out = A . W^T (- C), A float32 M x K, W float32 or
// bfloat16 (widened exactly) N x K row-major.
//
// Bound by the matrix cores: v_mfma_f32_16x16x4_f32, 154 TFLOP/s in a loop of nothing else.
// What cost the most before was the shape of the work: 128 x 128 tiles, 300 of them on 256
// CUs, and two barriers around each 32-k tile's trip through registers.  Now
//  - tiles of 16-128 rows x 64 or 128 columns, chosen so that the rows are hardly padded, whole
//    rounds of 256 tiles unsplit and only the rest split over K (plan_f32);
//  - both operands go to LDS by 16-byte loads, two to five 32-k stages ahead, swizzled so that
//    the fragment reads are free of bank conflicts; the four waves lie side by side along N (two
//    by two reads less LDS and measured the same);
//  - one barrier per K tile, in the middle of its MFMAs: the fragments of the next half tile are
//    read under the MFMAs of this one.
// The matrix cores are then busy 77% of the cycles on gate/up at 333 tokens and 70-71% on the smaller
// projections, at 2.2 GHz (profiles/counters_f32_qwen3-4b-m333.md).  An accumulator chain runs over 96 or 128 k
// and is then added into a second set of registers, so the rounding error no longer grows with
// K: 2.0e-7 to 2.5e-7 of the result at K = 9728 where one chain has 1.7e-6, and 8e-7 before (five splits).
// Chains of 192 k lost to the former splits at K = 256-1024 (2.5e-7 against 2.1e-7, now 2.1e-7) and are
// as fast within 1% on most shapes.
//
// bfloat16 W, Qwen3-4B: 333 tokens QKV 181 -> 92 us, O 124 -> 68, gate/up 357 -> 277 (120 TFLOP/s), Down
// 268 -> 149; 1024 tokens Down 635 -> 389 (131 TFLOP/s); one token O 30.6 -> 10.6; 32 x 512 x 512 8.4 -> 6.1;
// unsplit (splitee_masked_linear) 128 tokens Llama-3.2-3B Down 595 -> 80 us.
//
// K <= 128 under many tiles is bound by the stores of Out and by a workgroup's latency from first load to store,
// which the ring's loads past K lengthen.  One chain then holds all of K, its sums need no second set of registers,
// so 128 x 128 tiles fit (ONE): 2048 x 4096 x 64 22.8 -> 16.9 us (the former 128 x 128 tiles 17.6), 1280 x 19456 x
// 32 34.9 -> 29.6 (29.2), 8192 x 1024 x 128 29.6 -> 26.7 (25.6).
#include "gemm_dev.hpp"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int F_NW = 4;           // waves of a workgroup, side by side along N
constexpr int F_NT = F_NW * WAVE;
constexpr int F_BK = 32;          // k of one stage: 128 bytes of an A row
constexpr int F_CHAIN = 4;        // K tiles that one accumulator chain runs over at most
constexpr int F_MAX_TM = 8;       // 16-row blocks of a tile
constexpr int f32_max_tn(int tm) { return tm >= 4 && tm < 8 ? 2 : 1; } // 64-column blocks (128 x 128 would spill, but for ONE)

__device__ __attribute__((aligned(16))) const float f32_zeros[4] = {0.f, 0.f, 0.f, 0.f};

typedef const __attribute__((address_space(1))) void* glb_ptr_t;

template <int I, int BYTES>
__device__ __forceinline__ unsigned char* f32_stage()
{
    __shared__ __attribute__((aligned(16))) unsigned char buf[BYTES];
    return buf;
}

// Rows of the A stage: a tile's rows rounded up so that every wave loads as many.
constexpr int f32_stage_rows(int tm) { return (16 * tm + 31) / 32 * 32; }
constexpr int f32_stage_bytes(int tm, int tn, bool wbf16) { return f32_stage_rows(tm) * 128 + 64 * tn * (wbf16 ? 64 : 128); }
// Stages: as many as let two workgroups share a CU's 160 KB (one wave per SIMD reaches 141 TFLOP/s, two
// 154), 2, 3, 4 or 6: numbers that chains of at most F_CHAIN K tiles fit.
constexpr int f32_stages(int tm, int tn, bool wbf16)
{
    const int s = 78 * 1024 / f32_stage_bytes(tm, tn, wbf16);
    return s < 2 ? 2 : s >= 6 ? 6 : s == 5 ? 4 : s;
}

// ONE: K of at most F_CHAIN tiles, unsplit: acc is the result, and nothing past K is loaded.
template <int TM, int TN, bool WBF16, bool ONE = false>
__global__ void __launch_bounds__(F_NT, 2)
gemm_f32_kernel(const float* __restrict__ A, int64_t lda, const void* __restrict__ Wv, int64_t ldw,
                const float* __restrict__ C, int64_t ldc, float* __restrict__ Out, int64_t ldo, int M, int N, int K,
                int mtiles, int nfull, int ktps, int rem, float* __restrict__ part)
{
    constexpr int BM = 16 * TM, BN = 64 * TN;
    constexpr int S = f32_stages(TM, TN, WBF16);
    constexpr int RA = f32_stage_rows(TM), AB = RA * 128, SB = f32_stage_bytes(TM, TN, WBF16);
    constexpr int LA = RA / 8 / F_NW;                    // 1 KB loads to LDS per wave and stage: A
    constexpr int LW = BN * (WBF16 ? 64 : 128) / 1024 / F_NW; // and W
    static_assert((S - 1) * (LA + LW) < 64, "loads in flight exceed the wait counter");
    const int tid = threadIdx.x, lane = tid % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int ktiles = (K + F_BK - 1) / F_BK;
    // tiles 0 .. nfull - 1 whole, then rem tiles in splits of ktps K tiles
    const int b = blockIdx.x;
    const bool whole = b < nfull;
    const int sb0 = whole ? 0 : (b - nfull) / rem, tt = whole ? 0 : (b - nfull) % rem;
    const int tile = whole ? (int)splitee::xcd_logical_block((uint32_t)b, (uint32_t)nfull) : nfull + tt;
    const int m0 = (tile % mtiles) * BM, n0 = (tile / mtiles) * BN;
    const int kt0 = whole ? 0 : sb0 * ktps;
    const int nk = (whole ? ktiles : min(kt0 + ktps, ktiles)) - kt0;

    // A: load t of this wave fills stage rows 8 j .. 8 j + 7, j = wave + 4 t; lane l writes slot
    // l % 8 of row l / 8, holding the row's 16-byte chunk slot ^ (row % 8)
    const float* ap[LA];
    int ak[LA]; // columns of the row left at the load's first K tile (none for a row past M)
#pragma unroll
    for (int t = 0; t < LA; ++t) {
        const int row = 8 * (wave + F_NW * t) + lane / 8, gm = m0 + row;
        const int k = kt0 * F_BK + 4 * ((lane % 8) ^ (row & 7));
        const bool ok = row < BM && gm < M;
        ap[t] = A + (ok ? (int64_t)gm * lda + k : 0);
        ak[t] = ok ? K - k : 0;
    }
    // W: 4 chunks of a 64-byte bfloat16 row at slot chunk ^ ((row / 4) % 4), 16 rows per load, or
    // 8 chunks of a 128-byte float32 row as in A
    constexpr int WR = WBF16 ? 16 : 8, WC = WBF16 ? 4 : 8, WES = WBF16 ? 2 : 4;
    const char* wp[LW];
    int wk[LW];
#pragma unroll
    for (int t = 0; t < LW; ++t) {
        const int row = WR * (wave + F_NW * t) + lane / WC, gn = n0 + row;
        const int chunk = WBF16 ? (lane % 4) ^ ((row >> 2) & 3) : (lane % 8) ^ (row & 7);
        const int k = kt0 * F_BK + chunk * (16 / WES);
        const bool ok = gn < N;
        wp[t] = reinterpret_cast<const char*>(Wv) + (ok ? ((int64_t)gn * ldw + k) * WES : 0);
        wk[t] = ok ? K - k : 0;
    }

    unsigned char* const st[6] = {f32_stage<0, SB>(), f32_stage<1, SB>(), f32_stage<(S > 2 ? 2 : 0), SB>(),
                                  f32_stage<(S > 3 ? 3 : 0), SB>(), f32_stage<(S > 4 ? 4 : 0), SB>(), f32_stage<(S > 5 ? 5 : 0), SB>()};
    // the loads of relative K tile t into stage q (zeros past the split's end and the matrix)
    auto issue = [&](int t, auto sc) {
        constexpr int q = decltype(sc)::value;
        if (ONE && t >= nk) return; // (every wait is then for all loads)
        const int k = t < nk ? t * F_BK : K; // past every row's end
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const float* p = k < ak[i] ? ap[i] + k : f32_zeros;
            __builtin_amdgcn_global_load_lds((glb_ptr_t)p, (lds_ptr_t)(st[q] + (wave + F_NW * i) * 1024), 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < LW; ++i) {
            const char* p = k < wk[i] ? wp[i] + (int64_t)k * WES : reinterpret_cast<const char*>(f32_zeros);
            __builtin_amdgcn_global_load_lds((glb_ptr_t)p, (lds_ptr_t)(st[q] + AB + (wave + F_NW * i) * 1024), 16, 0, 0);
        }
    };

    // acc is added into sum every 3 or 4 K tiles
    f32x4_t acc[TM][TN], sum[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = sum[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // lane (r, g) of the MFMA operands: row r of a 16-row block, k = 8 g + e in instruction e of the
    // K tile's eight (any assignment of k to instructions and lane groups serves, the same for A and W)
    const int fr = lane % 16, fg = lane / 16;
    f32x4_t a0[TM], a1[TM], w[2][TN], wn[2][TN];
    auto read_a = [&](const unsigned char* s, int h, f32x4_t (&a)[TM]) { // k = 8 g + 4 h .. + 3
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = 16 * i + fr;
            a[i] = *reinterpret_cast<const f32x4_t*>(s + row * 128 + (((2 * fg + h) ^ (row & 7)) << 4));
        }
    };
    auto read_w = [&](const unsigned char* s) { // raw: one 16-byte word per block (bfloat16) or two
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int row = 16 * (wave * TN + j) + fr;
            if (WBF16) {
                wn[0][j] = *reinterpret_cast<const f32x4_t*>(s + AB + row * 64 + ((fg ^ ((row >> 2) & 3)) << 4));
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    wn[h][j] = *reinterpret_cast<const f32x4_t*>(s + AB + row * 128 + (((2 * fg + h) ^ (row & 7)) << 4));
            }
        }
    };
    auto widen_w = [&]() {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (WBF16) { // bfloat16 -> float32 is exact: the 16 bits become the upper half
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t d = __float_as_uint(wn[0][j][e / 2]);
                    w[e / 4][j][e % 4] = __uint_as_float(e % 2 ? d & 0xFFFF0000u : d << 16);
                }
            } else {
                w[0][j] = wn[0][j];
                w[1][j] = wn[1][j];
            }
        }
    };
    auto mul = [&](const f32x4_t (&a)[TM], int h) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], w[h][j][e], acc[i][j], 0, 0, 0);
    };
    // K tile t in stage q, its W and the first half of its A in registers.  First half: multiply
    // while the second half of A is read.  Then every wave is done with stage q, and tile t + 1
    // (this wave's loads of it: all but the S - 2 younger tiles') is in everywhere behind the
    // barrier.  Second half: multiply while tile t + 1's first fragments are read and
    // tile t + S goes into stage q.  The fences keep reads and loads in their half, the groups
    // spread them between its MFMAs.
    auto step = [&](int t, auto sc) {
        constexpr int q = decltype(sc)::value;
        read_a(st[q], 1, a1);
        mul(a0, 0);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, TN, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 3 * TM * TN, 0);
        __builtin_amdgcn_sched_barrier(0);
        wait_vmem<ONE ? 0 : (S - 2) * (LA + LW)>();
        __builtin_amdgcn_s_waitcnt((0 << 8) | (7 << 4) | 15 | (3 << 14)); // lgkmcnt(0): a1 is in
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        read_w(st[(q + 1) % S]);
        read_a(st[(q + 1) % S], 0, a0);
        issue(t + S, sc);
        mul(a1, 1);
#pragma unroll
        for (int i = 0; i < TM + TN * (WBF16 ? 1 : 2); ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
#pragma unroll
        for (int i = 0; i < LA + LW; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * TM * TN, 0);
        __builtin_amdgcn_sched_barrier(0);
        widen_w();
    };
    auto flush = [&](bool end = false) {
        if (ONE && !end) return;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                sum[i][j] += acc[i][j];
                acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
    };

#define F_IC(I) std::integral_constant<int, I>{}
    issue(0, F_IC(0));
    issue(1, F_IC(1));
    if constexpr (S > 2) issue(2, F_IC(2));
    if constexpr (S > 3) issue(3, F_IC(3));
    if constexpr (S > 4) issue(4, F_IC(4));
    if constexpr (S > 5) issue(5, F_IC(5));
    wait_vmem<ONE ? 0 : (S - 1) * (LA + LW)>();
    __builtin_amdgcn_s_barrier();
    read_w(st[0]);
    read_a(st[0], 0, a0);
    widen_w();
    // a turn: the chains' flush, in one block with the MFMAs that begin the next chain (from zero, so acc is
    // not cleared, and the additions run under them), and 3, 4 or 6 K tiles, with a flush between the halves of 6
    constexpr int TURN = S == 2 ? 4 : S;
    constexpr bool HALF = TURN > F_CHAIN;
    static_assert((HALF ? TURN / 2 : TURN) <= F_CHAIN, "chains too long");
    int t = 0;
    for (; t + TURN <= nk; t += TURN) {
        flush();
        step(t, F_IC(0));
        step(t + 1, F_IC(1));
        step(t + 2, F_IC(2 % S));
        if constexpr (HALF) flush();
        if constexpr (TURN > 3) step(t + 3, F_IC(3 % S));
        if constexpr (TURN > 4) step(t + 4, F_IC(4 % S));
        if constexpr (TURN > 5) step(t + 5, F_IC(5 % S));
    }
    // the last, partial turn
    flush();
    if (t < nk) step(t, F_IC(0));
    if (t + 1 < nk) step(t + 1, F_IC(1));
    if constexpr (TURN > 3) if (t + 2 < nk) step(t + 2, F_IC(2 % S));
    if constexpr (HALF) flush();
    if constexpr (TURN > 4) if (t + 3 < nk) step(t + 3, F_IC(3 % S));
    if constexpr (TURN > 5) if (t + 4 < nk) step(t + 4, F_IC(4 % S));
#undef F_IC
    wait_vmem<0>(); // loads past the last tile (zeros) have landed before the workgroup ends
    flush(true);

    if (!whole && part) { // float4 (i, j) of lane l at ((i TN + j) 64 + l): rows 4 (l / 16) .. + 3, column l % 16
        f32x4_t* mp = reinterpret_cast<f32x4_t*>(part) + ((int64_t)(b - nfull) * F_NW + wave) * (TM * TN * 64);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) mp[(i * TN + j) * 64 + lane] = sum[i][j];
        return;
    }
    // every C load of the wave tile before the first subtraction (one wait, not one per element);
    // elements outside M x N load C[0] and store nothing
    const int r0 = m0 + 4 * fg, c0 = n0 + 16 * wave * TN + fr;
    float cv[TM][TN][4];
    if (C) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = r0 + 16 * i + r, col = c0 + 16 * j;
                    cv[i][j][r] = C[row < M && col < N ? (int64_t)row * ldc + col : 0];
                }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = r0 + 16 * i + r, col = c0 + 16 * j;
                if (row < M && col < N) Out[(int64_t)row * ldo + col] = C ? sum[i][j][r] - cv[i][j][r] : sum[i][j][r];
            }
}

// The split tiles' partials added in split order, minus C.  Thread u handles one float4 of one
// wave's partial, in the register order they were written in.
constexpr int F_MAX_KS = 16;

template <int TM, int TN>
__global__ void __launch_bounds__(256)
f32_sum_kernel(const float* __restrict__ part, int ksplit, const float* __restrict__ C, int64_t ldc,
               float* __restrict__ Out, int64_t ldo, int M, int N, int mtiles, int nfull, int rem)
{
    constexpr int PER = TM * TN * 64, TILE = F_NW * PER; // float4 of a wave's and a tile's partial
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= rem * TILE) return;
    const int tt = u / TILE, e = u - tt * TILE, wave = e / PER, f = e - wave * PER;
    const int ij = f / 64, lane = f % 64, tile = nfull + tt;
    const int row0 = (tile % mtiles) * 16 * TM + 16 * (ij / TN) + 4 * (lane / 16);
    const int col = (tile / mtiles) * 64 * TN + 16 * (wave * TN + ij % TN) + lane % 16;
    float cv[4] = {0.f, 0.f, 0.f, 0.f};
    if (C) {
#pragma unroll
        for (int r = 0; r < 4; ++r) cv[r] = C[row0 + r < M && col < N ? (int64_t)(row0 + r) * ldc + col : 0];
    }
    // every split's partial in flight together: one past ksplit reads zeros and is not added
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(part, (uint32_t)((int64_t)rem * ksplit * TILE * 16));
    f32x4_t v[F_MAX_KS];
#pragma unroll
    for (int q = 0; q < F_MAX_KS; ++q)
        v[q] = __builtin_bit_cast(f32x4_t, load16(rp, q < ksplit ? (uint32_t)((q * rem + tt) * TILE + e) * 16 : OOB));
    f32x4_t sum = v[0];
#pragma unroll
    for (int q = 1; q < F_MAX_KS; ++q)
        if (q < ksplit) sum += v[q];
    if (col >= N) return;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (row0 + r < M) Out[(int64_t)(row0 + r) * ldo + col] = C ? sum[r] - cv[r] : sum[r];
}

struct F32Plan {
    int tm, tn, mtiles;
    int nfull, rem, ksplit, ktps; // whole tiles, split tiles, their splits and K tiles per split
    size_t part_bytes;
};

constexpr size_t F32_SCRATCH = SPLITEE_NOALLOC_SCRATCH_BYTES; // partials and the masked input together

// The tile (16 tm rows x 64 tn columns) and the split of the tiles that fill no whole round of 256
// workgroups, by the launch's modelled time.  Measured over tm 1-8, tn 1-2 and 1-16 splits at
// 1-1024 tokens on the Qwen3-4B and Llama-3.2-3B projections: a K tile takes 0.121 tm tn + 0.06
// us of a CU whatever the number of workgroups on it (a twentieth more with one alone), a
// workgroup 1 us besides, the sum 4 us and its partials' traffic at 5 TB/s.  The model's choice
// is within 5% of the best there.  E.g. 333 tokens x 6144 columns x 2560: 288 tiles of 112 x 64, 256
// whole and 32 in eight splits, 92 us; 240 tiles of 80 x 128 unsplit 108; 288 unsplit 147.
F32Plan plan_f32(int64_t M, int64_t N, int64_t K, bool allow_split)
{
    const int ktiles = (int)((K + F_BK - 1) / F_BK);
    const size_t xt = ((size_t)M * K * 4 + 255) / 256 * 256;
    F32Plan best{};
    // K in one chain and 128 x 128 tiles that nearly fill one to three rounds of two per CU: their count decides.  512
    // tiles, 2048 x 4096 x 64: 16.9 us, with the tiles below 22.8; 480 (3000 x 2560 x 64) 15.6 and 19.2; 1520 (1280 x
    // 19456 x 32) 29.6 and 34.9.  But 288 (1100 x 4096 x 64) 15.0 and 12.1, 1064 (777 x 19456 x 64) 34.9 and 28.9,
    // 4096 (16384 x 4096 x 64) 120 and 113.
    const int64_t m128 = (M + 127) / 128, t128 = m128 * ((N + 127) / 128), r128 = (t128 + 511) / 512;
    if (ktiles <= F_CHAIN && r128 >= 1 && r128 <= 3 && t128 * 10 >= r128 * 512 * 9) {
        best.tm = 8;
        best.tn = 2;
        best.mtiles = (int)m128;
        best.nfull = (int)t128;
        best.ksplit = best.ktps = 1;
        return best;
    }
    double best_cost = -1.0;
    // (rows that one more 16-row block would only pad are not tried: the planning costs host time)
    for (int tm = 1; tm <= F_MAX_TM && 16 * (tm - 1) < M; ++tm)
        for (int tn = 1; tn <= f32_max_tn(tm); ++tn) {
            const int64_t mtiles = (M + 16 * tm - 1) / (16 * tm), tiles = mtiles * ((N + 64 * tn - 1) / (64 * tn));
            const int64_t full = tiles / 256 * 256, rem = tiles - full;
            const double ktile = 0.121 * tm * tn + 0.06;
            for (int ks = 1; ks <= F_MAX_KS; ++ks) {
                // a split has at least four K tiles, and partials and masked input fit the scratch of the
                // call without a workspace, whose bits are those of the call with one (so nothing is split from about
                // 1700 x 9728 up; 1800 and 2048 rows are faster there than with the former splits all the same)
                if (ks > 1 && (!allow_split || rem == 0 || ktiles / ks < 4)) break;
                const int ktps = ktiles > 0 ? (ktiles + ks - 1) / ks : 1;
                if (ks > 1 && (ktiles + ktps - 1) / ktps != ks) continue;
                const size_t pb = ks > 1 ? (size_t)rem * ks * tm * tn * 4096 : 0;
                if (ks > 1 && pb + xt + 512 > F32_SCRATCH) break;
                const int64_t wgs = rem * ks, rounds = (wgs + 255) / 256;
                const double alone = full == 0 && wgs <= 256 ? 1.05 : 1.0;
                const double cost = (double)(full / 256) * (ktiles * ktile + 1.0) +
                                    (double)rounds * (ktps * ktile * alone + 1.0) + (ks > 1 ? 4.0 + (double)pb * 2 / 5.0e6 : 0.0);
                if (best_cost >= 0 && cost >= best_cost) continue;
                best_cost = cost;
                best.tm = tm;
                best.tn = tn;
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

size_t f32_gemm_workspace_bytes(int64_t M, int64_t N, int64_t K)
{
    return M > 0 && N > 0 ? plan_f32(M, N, K, true).part_bytes : 0;
}

int launch_gemm_f32(const float* A, int64_t lda, const void* W, int w_type, int64_t ldw, const float* C, int64_t ldc,
                    float* Out, int64_t ldo, int64_t M, int64_t N, int64_t K, void* ws, size_t ws_bytes, hipStream_t s)
{
    if (M == 0 || N == 0) return SPLITEE_OK;
    const F32Plan p = plan_f32(M, N, K, ws != nullptr);
    if (p.ksplit > 1 && ws_bytes < splitee::WS_COUNTER_BYTES + p.part_bytes) return SPLITEE_ERR_WORKSPACE;
    float* part = p.ksplit > 1 ? ws_partials(ws) : nullptr;
    const dim3 grid((unsigned)(p.nfull + (int64_t)p.rem * p.ksplit));
    const dim3 g2((unsigned)(((int64_t)p.rem * p.tm * p.tn * 256 + 255) / 256));
    const bool bf16 = w_type == SPLITEE_BF16;
    if (p.tm == 8 && p.tn == 2) {
        if (bf16)
            hipLaunchKernelGGL((gemm_f32_kernel<8, 2, true, true>), grid, dim3(F_NT), 0, s, A, lda, W, ldw, C, ldc, Out, ldo, (int)M,
                               (int)N, (int)K, p.mtiles, p.nfull, p.ktps, p.rem, part);
        else
            hipLaunchKernelGGL((gemm_f32_kernel<8, 2, false, true>), grid, dim3(F_NT), 0, s, A, lda, W, ldw, C, ldc, Out, ldo, (int)M,
                               (int)N, (int)K, p.mtiles, p.nfull, p.ktps, p.rem, part);
        return hipGetLastError() == hipSuccess ? SPLITEE_OK : SPLITEE_ERR_HIP;
    }
#define F_RUN(TM, TN)                                                                                                  \
    do {                                                                                                               \
        if (bf16)                                                                                                      \
            hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, true>), grid, dim3(F_NT), 0, s, A, lda, W, ldw, C, ldc, Out,   \
                               ldo, (int)M, (int)N, (int)K, p.mtiles, p.nfull, p.ktps, p.rem, part);                   \
        else                                                                                                           \
            hipLaunchKernelGGL((gemm_f32_kernel<TM, TN, false>), grid, dim3(F_NT), 0, s, A, lda, W, ldw, C, ldc, Out,  \
                               ldo, (int)M, (int)N, (int)K, p.mtiles, p.nfull, p.ktps, p.rem, part);                   \
        if (p.ksplit > 1)                                                                                              \
            hipLaunchKernelGGL((f32_sum_kernel<TM, TN>), g2, dim3(256), 0, s, part, p.ksplit, C, ldc, Out, ldo,        \
                               (int)M, (int)N, p.mtiles, p.nfull, p.rem);                                              \
    } while (0)
    switch (p.tm * 10 + p.tn) {
    case 11: F_RUN(1, 1); break;
    case 21: F_RUN(2, 1); break;
    case 31: F_RUN(3, 1); break;
    case 41: F_RUN(4, 1); break;
    case 42: F_RUN(4, 2); break;
    case 51: F_RUN(5, 1); break;
    case 52: F_RUN(5, 2); break;
    case 61: F_RUN(6, 1); break;
    case 62: F_RUN(6, 2); break;
    case 71: F_RUN(7, 1); break;
    case 72: F_RUN(7, 2); break;
    default: F_RUN(8, 1); break;
    }
#undef F_RUN
    return hipGetLastError() == hipSuccess ? SPLITEE_OK : SPLITEE_ERR_HIP;
}

}  // namespace splitee_host

// bfloat16 MFMA GEMM for few tokens without a split of K over workgroups (gfx950):
// splitee_masked_linear, the untrusted GPU's product, has no workspace for one.
//
//   Out = A . W^T,  A as one or three bfloat16 planes, W row-major or tiled
//
// What bounds it: W read once from HBM, and the masked input, which every workgroup reads
// whole from L2.  A 64-row tile per workgroup (the streamed kernel) leaves most of the chip
// idle here: 24 workgroups for 3072 columns.  So a workgroup owns a narrow tile, 16 rows x
// 16 TN columns, and its eight waves split K: wave w takes the 64-k tiles w, w + 8, .., and
// the waves' sums meet in LDS and are added in wave order (the result does not depend on
// timing).  A wave's masked input goes to LDS by 1 KB loads, 8 rows of whole 128-byte lines
// each, in a swizzled order that its own fragment reads find free of bank conflicts: loading the
// 16-row fragments straight into registers touches every line twice, and the vector L1
// serves a line every other clock (Llama-3.2-3B O and Down at 15 tokens 12.3 and 27.4 us so,
// 9.9 and 21.6 this way).  The stage belongs to one wave: no barrier in the loop.  W goes
// straight to MFMA operand registers.  Two K tiles in flight; three were as fast or slower.
//
// 15 tokens, Llama-3.2-3B, tiled W, against the streamed kernel's unsplit tiles: QKV 31.9 ->
// 12.5 us, O 31.4 -> 9.9, gate/up 47.5 -> 22.4 (18.1 alone: 5.7 TB/s,
// profiles/counters_product_llama3b-m15.md), Down 76.3 -> 21.6; row-major W
// at 32 tokens 93 -> 19, 92 -> 14, 94 -> 46 and 204 -> 31 us.
#include "gemm_dev.hpp"

namespace {

constexpr int WS_NW = 8;                // waves of a workgroup
constexpr int WS_NT = WS_NW * WAVE;
constexpr int WS_MAX_TN = 6;            // 16-column blocks of a workgroup

template <int I, int BYTES>
__device__ __forceinline__ unsigned char* ws_stage()
{
    __shared__ __attribute__((aligned(16))) unsigned char buf[BYTES];
    return buf;
}

template <int NPL, int TN, bool TILED>
__global__ void __launch_bounds__(WS_NT)
wsplit_kernel(const uint16_t* __restrict__ A, int64_t lda, int64_t pstride, const uint16_t* __restrict__ W, int64_t ldw,
              float* __restrict__ Out, int64_t ldo, int M, int N, int K, int mtiles)
{
    constexpr int BM = 16, BN = 16 * TN;
    constexpr int LA = NPL * BM / 8;    // 1 KB loads to LDS per wave and K tile (8 rows of 128 bytes each)
    constexpr int LW = 2 * TN;          // W loads per wave and K tile
    constexpr int SB = LA * 1024;       // LDS bytes of one wave's stage
    constexpr int LDR = BN + 4;         // padded row of the reduction tile
    constexpr int EPT = (BM * BN + WS_NT - 1) / WS_NT; // output elements per thread
    constexpr int R = 2;                // K tiles in flight per wave
    constexpr int RB = WS_NW * BM * LDR * 4; // bytes of the reduction tile
    const int tid = threadIdx.x, lane = tid % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int lb = (int)splitee::xcd_logical_block(blockIdx.x, gridDim.x);
    const int m0 = (lb % mtiles) * BM, n0 = (lb / mtiles) * BN;
    const int ktiles = (K + BK - 1) / BK;
    const int ng = ktiles > wave ? (ktiles - wave + WS_NW - 1) / WS_NW : 0; // this wave's K tiles: wave, wave + 8, ..
    const int fr = lane % 16, fq = lane / 16;

    // W: lane (r, q) takes column n0 + 16 j + r, 16 bytes at k = 32 s + 8 q of step s of the K tile
    const __amdgpu_buffer_rsrc_t rw =
        make_rsrc(W, (uint32_t)(TILED ? (int64_t)((N + 31) / 32) * ktiles * 4096 : (int64_t)N * ldw * 2));
    uint32_t woff[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int gn = n0 + 16 * j + fr;
        woff[j] = gn >= N ? OOB
                  : TILED ? (uint32_t)((int64_t)(gn / 32) * ktiles * 4096 + (fq / 2) * 1024 + ((fq % 2) * 32 + gn % 32) * 16)
                          : (uint32_t)((int64_t)gn * ldw * 2 + fq * 16);
    }
    // masked input: load t fills stage rows 8 t .. 8 t + 7 (row 16 p + r of plane p); lane l writes
    // slot l % 8 of row 8 t + l / 8, which holds k chunk slot ^ ((row / 2) % 8)
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, (uint32_t)(((NPL - 1) * pstride + (int64_t)M * lda) * 2));
    uint32_t aoff[LA];
    int akc[LA];
#pragma unroll
    for (int t = 0; t < LA; ++t) {
        const int row = 8 * t + lane / 8, p = row / BM, gm = m0 + row % BM;
        akc[t] = ((lane % 8) ^ ((row >> 1) & 7)) * 8;
        aoff[t] = gm < M ? (uint32_t)((p * pstride + (int64_t)gm * lda + akc[t]) * 2) : OOB;
    }

    unsigned char* const st0 = ws_stage<0, WS_NW * SB>();
    unsigned char* const st1 = ws_stage<1, WS_NW * SB>();
    auto stage = [&](int u) { return (u == 0 ? st0 : st1) + wave * SB; };

    uint4 wr[R][2][TN];
    // K tile g of this wave into ring slot u (zeros past its last).  An operand offset at or past
    // OOB stays there whatever k adds (the matrices are below 2 GB), so no load needs a branch.
    auto issue = [&](int g, int u) {
        const int kt = wave + WS_NW * g, k = kt * BK;
        const uint32_t dead = g < ng ? 0u : OOB;
#pragma unroll
        for (int t = 0; t < LA; ++t) {
            const uint32_t off = (aoff[t] + (uint32_t)k * 2) | dead;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr_t)(stage(u) + t * 1024), 16,
                                                     (int)(k + akc[t] < K ? off : OOB), 0, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const uint32_t off = (woff[j] + (uint32_t)(TILED ? kt * 4096 + s * 2048 : (k + 32 * s) * 2)) | dead;
                wr[u][s][j] = load16(rw, TILED || k + 32 * s + 8 * fq < K ? off : OOB); // tiled W: zeros past K
            }
        __builtin_amdgcn_sched_barrier(0);
    };

#pragma unroll
    for (int u = 0; u < R; ++u) issue(u, u);

    f32x4_t acc[2][TN];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[s][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto consume = [&](int u) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            uint4 a[NPL];
#pragma unroll
            for (int p = 0; p < NPL; ++p) {
                const int row = p * BM + fr;
                a[p] = *reinterpret_cast<const uint4*>(stage(u) + row * 128 + (((4 * s + fq) ^ ((row >> 1) & 7)) << 4));
            }
#pragma unroll
            for (int p = 0; p < NPL; ++p)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[s][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a[p]), as_bf16x8(wr[u][s][j]), acc[s][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int g = 0;
    for (; g + R <= ng; g += R) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            wait_vmem<(R - 1) * (LA + LW)>(); // this slot's loads are in; the younger slot's may be in flight
            consume(u);
            issue(g + u + R, u);
        }
    }
    wait_vmem<0>(); // the last tile of an odd count, and the loads past it (zeros)
    if (g < ng) consume(0);

    // the waves' sums meet in LDS (in the first stage where it holds them: every wave is done
    // with it) and are added in wave order; a thread adds elements tid, tid + 512, .. of the tile
    float* const red = reinterpret_cast<float*>(RB <= WS_NW * SB ? st0 : ws_stage<2, RB <= WS_NW * SB ? 16 : RB>());
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const f32x4_t v = acc[0][j] + acc[1][j];
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(wave * BM + 4 * fq + r) * LDR + 16 * j + fr] = v[r];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int f = tid + e * WS_NT, row = m0 + f / BN, col = n0 + f % BN;
        if (f >= BM * BN || row >= M || col >= N) continue;
        float y = red[(f / BN) * LDR + f % BN];
#pragma unroll
        for (int v = 1; v < WS_NW; ++v) y += red[(v * BM + f / BN) * LDR + f % BN];
        Out[(int64_t)row * ldo + col] = y;
    }
}

}  // namespace

namespace splitee_host {

// Columns per workgroup (16 TN) and the cost of the launch in microseconds per 64-k tile:
// rounds of 256 workgroups (the stages leave room for one per CU) times a round's time, which
// grows with the masked input and with TN.  Fitted to 3072-9728 wide K at 4-64 tokens: 0.040
// (4.2 + TN) us with three planes on tiled W, 0.042 (2.4 + TN) with one; row-major W, whose
// 16-column loads touch half lines, 0.073 (2 + TN).
WsplitPlan plan_wsplit(int64_t M, int64_t N, int prec, int w_type)
{
    const int64_t mtiles = (M + 15) / 16;
    WsplitPlan best{0, 0.0};
    for (int tn = 1; tn <= WS_MAX_TN; ++tn) {
        const int64_t wgs = mtiles * ((N + 16 * tn - 1) / (16 * tn));
        const double round = w_type != SPLITEE_BF16_TILED ? 0.073 * (2.0 + tn)
                             : prec == SPLITEE_PREC_BF16X3 ? 0.040 * (4.2 + tn)
                                                           : 0.042 * (2.4 + tn);
        const double cost = (double)((wgs + 255) / 256) * round;
        if (best.tn == 0 || cost < best.cost) best = WsplitPlan{tn, cost};
    }
    return best;
}

int launch_wsplit(const void* A, int prec, int64_t lda, int64_t pstride, const void* W, int w_type, int64_t ldw,
                  float* Out, int64_t ldo, int64_t M, int64_t N, int64_t K, hipStream_t s)
{
    const int tn = plan_wsplit(M, N, prec, w_type).tn;
    const int64_t mt = (M + 15) / 16, wgs = mt * ((N + 16 * tn - 1) / (16 * tn));
    const bool tiled = w_type == SPLITEE_BF16_TILED;
    const uint16_t *w = reinterpret_cast<const uint16_t*>(W), *a = reinterpret_cast<const uint16_t*>(A);
#define WS(NP, TN_, T)                                                                                               \
    hipLaunchKernelGGL((wsplit_kernel<NP, TN_, T>), dim3((unsigned)wgs), dim3(WS_NT), 0, s, a, lda, pstride, w, ldw, \
                       Out, ldo, (int)M, (int)N, (int)K, (int)mt)
#define WS_TN(NP, T)                                                                       \
    switch (tn) {                                                                          \
    case 1: WS(NP, 1, T); break;                                                           \
    case 2: WS(NP, 2, T); break;                                                           \
    case 3: WS(NP, 3, T); break;                                                           \
    case 4: WS(NP, 4, T); break;                                                           \
    case 5: WS(NP, 5, T); break;                                                           \
    default: WS(NP, 6, T); break;                                                          \
    }
    if (prec == SPLITEE_PREC_BF16) { if (tiled) { WS_TN(1, true) } else { WS_TN(1, false) } }
    else { if (tiled) { WS_TN(3, true) } else { WS_TN(3, false) } }
#undef WS_TN
#undef WS
    return hipGetLastError() == hipSuccess ? SPLITEE_OK : SPLITEE_ERR_HIP;
}

}  // namespace splitee_host

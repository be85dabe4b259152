// Which tiling of ago_gemm_dma.hpp a product takes, and the launch.
#include "ago_gemm_dma.hpp"

namespace ago {

namespace {
// Time model per tiling: T tiles on 256 compute units, n = ceil(T / 256) on the busiest one, k = K / 32 steps a tile,
//   us = c0 + c1 n + c2 n k + c3 k (n = 1 only) + c4 T k / 256
// (launch and first loads; start and end of a tile; its steps; steps that nothing overlaps; what the whole chip pulls
// through the L2s).  Coefficients: non-negative least squares over 100 products, M 16 .. 16384, K 256 .. 4096, N 512 ..
// 4096, bf16, on an MI355X (mean error 3 - 6 % per tiling; the tiling picked is 2 % behind the best one on average).
struct TilingModel { int bm, bn; float c[5]; };
constexpr TilingModel kModel[kGemmTilings] = {
    {128, 256, {2.026f, 3.551f, 0.174f, 0.1081f, 0.2319f}},
    {128, 256, {0.2497f, 5.033f, 0.2173f, 0.0233f, 0.2484f}},
    {128, 192, {2.356f, 2.585f, 0.1869f, 0.0494f, 0.1489f}},
    {128, 128, {2.054f, 2.064f, 0.158f, 0.0286f, 0.0885f}},
    {64, 128, {2.448f, 0.7838f, 0.1235f, 0.0221f, 0.0398f}},
    {64, 96, {1.245f, 3.874f, 0.0533f, 0.0134f, 0.0862f}},
    {64, 64, {1.735f, 2.541f, 0.0513f, 0.0015f, 0.0551f}},
    {64, 32, {1.464f, 2.498f, 0.0311f, 0.0f, 0.0546f}},
    {32, 32, {1.801f, 1.829f, 0.0193f, 0.0f, 0.0359f}},
    {32, 64, {1.531f, 2.212f, 0.04f, 0.0f, 0.0256f}},
};
// threads of a workgroup
#define AGO_GEMM_SHARED(ID, BM, BN, WM, WN, NST) WM * WN * 64,
#define AGO_GEMM_SPLIT(ID, BM, BN, WAVES, NST) WAVES * 64,
constexpr int kThreads[kGemmTilings] = {AGO_GEMM_TILINGS(AGO_GEMM_SHARED, AGO_GEMM_SPLIT)};
#undef AGO_GEMM_SHARED
#undef AGO_GEMM_SPLIT
}  // namespace

double gemm_dma_predict(int M, int K, int N, int siblings, int* tiling) {
    const double k = K / 32;
    double best = 0;
    int pick = 0;
    for (int i = 0; i < kGemmTilings; ++i) {
        const TilingModel& m = kModel[i];
        const long tiles = ((long)M + m.bm - 1) / m.bm * (((long)N + m.bn - 1) / m.bn) * siblings;
        const double n = (double)((tiles + 255) / 256);
        const double us = m.c[0] + m.c[1] * n + m.c[2] * n * k + (n == 1 ? m.c[3] * k : 0) + m.c[4] * (double)tiles * k / 256;
        if (i == 0 || us < best) { best = us; pick = i; }
    }
    if (tiling) *tiling = pick;
    return best;
}

bool gemm_dma_ok(int K, int N, bool packed) { return K % 32 == 0 && N % (packed ? 16 : 8) == 0; }

hipError_t gemm_dma(const void* a, const void* w, bool packed, const float* bias, const void* res, void* c, int M, int K, int N, int act,
                    hipStream_t s) {
    GemmDmaParams p = {};
    p.a = (const bf16_t*)a; p.w0 = (const bf16_t*)w; p.b0 = bias; p.r = (const bf16_t*)res; p.c0 = (bf16_t*)c;
    p.M = M; p.K = K; p.N = N; p.siblings = 1; p.act = act;
    int tiling = 0;
    gemm_dma_predict(M, K, N, 1, &tiling);
    if (packed) return res ? hipErrorInvalidValue : gemm_dma_packed(tiling, p, s);
    return res ? gemm_dma_special(tiling, p, false, s) : gemm_dma_rows(tiling, p, s);
}

// q / k / v = x w* + b*: three siblings side by side in one grid
hipError_t gemm_dma_qkv(const void* x, const void* const w[3], const float* const b[3], void* const o[3], int B, int S, int K, int Hh, int D,
                        bool head_major, hipStream_t s) {
    GemmDmaParams p = {};
    p.a = (const bf16_t*)x;
    p.w0 = (const bf16_t*)w[0]; p.w1 = (const bf16_t*)w[1]; p.w2 = (const bf16_t*)w[2];
    p.b0 = b[0]; p.b1 = b[1]; p.b2 = b[2];
    p.c0 = (bf16_t*)o[0]; p.c1 = (bf16_t*)o[1]; p.c2 = (bf16_t*)o[2];
    p.M = B * S; p.K = K; p.N = Hh * D; p.siblings = 3; p.act = kNone;
    p.S = S; p.Hh = Hh; p.D = D;
    int tiling = 0;
    gemm_dma_predict(p.M, K, p.N, 3, &tiling);
    return head_major ? gemm_dma_special(tiling, p, true, s) : gemm_dma_rows(tiling, p, s);
}

// matmul -> activation -> matmul as two products.  The fused kernels keep the hidden tensor on chip but exchange fp32 partial
// sums of the output instead, one per 384 hidden units, and a workgroup's 64 rows read every weight through one compute
// unit; against the products above they lose at every measured row count with more than one hidden slice (768 -> 3072
// -> 768, row-major: 128 rows 26.6 -> 11.7 us, 2048 rows 39 -> 34 us; packed 2048 rows 37 -> 32 us).
bool ffn_two_products_pay(int M, int K, int F, int K2, bool packed, size_t ws_bytes, double fused_us) {
    return gemm_dma_ok(K, F, packed) && gemm_dma_ok(F, K2, packed) && (size_t)M * F * 2 <= ws_bytes &&
           gemm_dma_predict(M, K, F, 1, nullptr) + gemm_dma_predict(M, F, K2, 1, nullptr) < fused_us;
}

hipError_t ffn_two_products(const void* x, const void* w1, const float* b1, const void* w2, const float* b2, void* y, int M, int K,
                            int F, int K2, int act, bool packed, void* workspace, hipStream_t s) {
    int tiling = 0;
    gemm_dma_predict(M, K, F, 1, &tiling);
    const TilingModel& m = kModel[tiling];
    prof_start(2, s);      // no split: either product is a part of the chain only
    prof_shape(2, (unsigned)((((long)M + m.bm - 1) / m.bm) * (((long)F + m.bn - 1) / m.bn)), (unsigned)kThreads[tiling]);
    hipError_t e = gemm_dma(x, w1, packed, b1, nullptr, workspace, M, K, F, act, s);
    if (e == hipSuccess) e = gemm_dma(workspace, w2, packed, b2, nullptr, y, M, F, K2, kNone, s);
    prof_stop(2, s);
    return e;
}

// sizes ago_gemm_packed takes
bool gemm_packed_ok(int K, int N) { return (N % 192 == 0 && K % 128 == 0) || (N % 96 == 0 && K % 512 == 0); }

}  // namespace ago

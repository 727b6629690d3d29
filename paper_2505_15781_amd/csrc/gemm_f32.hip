// fp32 projection of few rows: one 16x16 tile of the product per workgroup, the K range dealt to its four wavefronts.
//
// The fp32 mode serves small models, where a projection is a handful of megaflops and only its latency counts: with the
// 64x64 tiles of gemm_simt a 64 x 128 x 512 product ran on 2 workgroups that walked K in 32 dependent steps. Here the
// same product runs on 32 workgroups, every lane has its whole share of K in flight at once (float4 loads straight
// into MFMA operands: a lane's four consecutive K elements feed four 16x16x4 fp32 MFMAs, the order of K inside a sum is
// free), and the four partial tiles meet in LDS. 64 x 128 x 512: 46.9 -> 7.5 us per call; inside the 2-layer fp32 toy
// model the projections of a step take 3-5 us each instead of 12-42.
#include "common.h"

namespace {

// SWIGLU: W rows interleave gate_j, up_j and out[m][j] = silu(gate_j) * up_j, N / 2 columns.
template <bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_f32_few_rows(const float *__restrict__ A, const float *__restrict__ W,
                                                         float *__restrict__ out, int m_upper,
                                                         const int *__restrict__ m_dev, int N, int K) {
    __shared__ float red[4][16][17];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4;
    const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
    // rows are clamped to the launch's bound, not to the count on the device: its load overlaps the others, and rows in
    // between only feed outputs that are not stored
    const float *a = A + (size_t)min(m0 + (lane & 15), m_upper - 1) * K, *w = W + (size_t)min(n0 + (lane & 15), N - 1) * K;
    const int M = m_dev ? min(*m_dev, m_upper) : m_upper;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int k0 = wave * 16; k0 < K; k0 += 64) {
        const int k = k0 + 4 * g, kc = min(k, K - 4);
        f32x4 x = *reinterpret_cast<const f32x4 *>(a + kc);
        const f32x4 y = *reinterpret_cast<const f32x4 *>(w + kc);
        if (k >= K) x = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], y[j], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][4 * g + v][lane & 15] = acc[v];
    __syncthreads();
    if (!SWIGLU) {
        const int r = tid >> 4, c = tid & 15;
        const float y = (red[0][r][c] + red[1][r][c]) + (red[2][r][c] + red[3][r][c]);
        if (m0 + r < M && n0 + c < N) out[(size_t)(m0 + r) * N + n0 + c] = y;
    } else if (tid < 128) {
        const int r = tid >> 3, c = (tid & 7) * 2;
        const float gate = (red[0][r][c] + red[1][r][c]) + (red[2][r][c] + red[3][r][c]);
        const float up = (red[0][r][c + 1] + red[1][r][c + 1]) + (red[2][r][c + 1] + red[3][r][c + 1]);
        if (m0 + r < M && n0 + c < N) out[(size_t)(m0 + r) * (N >> 1) + ((n0 + c) >> 1)] = gate / (1.0f + expf(-gate)) * up;
    }
}

}  // namespace

// Few rows: up to 512 tiles of 64x64. Every tile of 16x16 reads its rows of A and W itself, which costs more than the
// idle units of gemm_simt from then on: 512 x 896 x 1024 28 against 98 us, 1024 x 2048 x 1024 (512 tiles) 119 against
// 142, 2048 x 2048 x 1024 (1024 tiles) 226 against 171.
bool dkv_gemm_f32_few_rows(int dtype, int m, int n, int k) {
    return dtype == DKV_FP32 && k % 4 == 0 && (long)ceil_div(m, 64) * ceil_div(n, 64) <= 512;
}

int dkv_launch_gemm_f32_few_rows(const float *A, const float *W, float *out, int m_upper, const int *m_dev, int n, int k,
                                 bool swiglu, hipStream_t stream) {
    if (m_upper <= 0) return DKV_OK;
    const dim3 grid(ceil_div(n, 16), ceil_div(m_upper, 16));
    if (swiglu) hipLaunchKernelGGL((gemm_f32_few_rows<true>), grid, dim3(256), 0, stream, A, W, out, m_upper, m_dev, n, k);
    else hipLaunchKernelGGL((gemm_f32_few_rows<false>), grid, dim3(256), 0, stream, A, W, out, m_upper, m_dev, n, k);
    DKV_LAUNCH_CHECK();
    return DKV_OK;
}

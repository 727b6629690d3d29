// fp32 projection of few rows: one 16x16 tile of the product per workgroup, one output per thread.
//
// The fp32 mode serves small models, where a projection is a handful of megaflops and only its latency counts: with the
// 64x64 tiles of gemm_simt a 64 x 128 x 512 product ran on 2 workgroups that waited for memory in each of 32 dependent
// steps of K. Here the same product runs on 32 workgroups, K comes in pieces of 128 with the next piece already on its
// way, and a thread needs two 16-byte LDS reads for four FMAs: 64 x 128 x 512 47.1 -> 8.5 us per call, a generation of the
// 2-layer toy model (32 steps) 8.18 -> 2.78 ms. What bounds it is launch and memory latency. Every sum is formed as gemm_simt forms it, one FMA per
// element of K in ascending order, so the choice between the two does not change a bit of the result: in fp32 two
// candidates of a step can be equal but for a rounding, and another order of the sums would commit the other one.
#include "common.h"

namespace {

// SWIGLU: W rows interleave gate_j, up_j and out[m][j] = silu(gate_j) * up_j, N / 2 columns.
template <bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_f32_few_rows(const float *__restrict__ A, const float *__restrict__ W,
                                                         float *__restrict__ out, int m_upper,
                                                         const int *__restrict__ m_dev, int N, int K) {
    constexpr int KC = 128, ROW = KC + 4, V = 16 * KC / 4 / 256;     // + 4: the 16 rows of a read start in different banks
    __shared__ __attribute__((aligned(16))) float As[16][ROW], Ws[16][ROW];
    const int tid = threadIdx.x, r = tid >> 4, c = tid & 15;
    const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
    // rows are clamped to the launch's bound, not to the count on the device: its load overlaps the others, and rows in
    // between only feed outputs that are not stored
    const int M = m_dev ? min(*m_dev, m_upper) : m_upper;
    f32x4 ra[V], rw[V];
    auto fetch = [&](int kb) {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int e = tid + 256 * i, row = e / (KC / 4), k = kb + e % (KC / 4) * 4, kc = min(k, K - 4);
            ra[i] = *reinterpret_cast<const f32x4_el *>(A + (size_t)min(m0 + row, m_upper - 1) * K + kc);
            rw[i] = *reinterpret_cast<const f32x4_el *>(W + (size_t)min(n0 + row, N - 1) * K + kc);
        }
    };
    float acc = 0.f;
    fetch(0);
    for (int kb = 0; kb < K; kb += KC) {
        if (kb) __syncthreads();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int e = tid + 256 * i, row = e / (KC / 4), k = e % (KC / 4) * 4;
            *reinterpret_cast<f32x4 *>(&As[row][k]) = ra[i];
            *reinterpret_cast<f32x4 *>(&Ws[row][k]) = rw[i];
        }
        __syncthreads();
        if (kb + KC < K) fetch(kb + KC);
        auto four = [&](int k) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(&As[r][k]), y = *reinterpret_cast<const f32x4 *>(&Ws[c][k]);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = fmaf(x[j], y[j], acc);
        };
        if (K - kb >= KC) {
#pragma unroll 16
            for (int k = 0; k < KC; k += 4) four(k);
        } else {
            for (int k = 0; k < K - kb; k += 4) four(k);
        }
    }
    if (!SWIGLU) {
        if (m0 + r < M && n0 + c < N) out[(size_t)(m0 + r) * N + n0 + c] = acc;
    } else {
        const float up = __shfl_xor(acc, 1, 64);
        if (!(c & 1) && m0 + r < M && n0 + c < N)
            out[(size_t)(m0 + r) * (N >> 1) + ((n0 + c) >> 1)] = acc / (1.0f + expf(-acc)) * up;
    }
}

}  // namespace

// Few rows: up to 128 tiles of 64x64. Every tile of 16x16 reads its rows of A and W itself, so the time grows with their
// number while gemm_simt's is that of one tile until every unit has one: 512 x 1024 x 128 (128 tiles) 8.6 against 19.8
// us, 128 x 4096 x 256 (128) 12.3 / 25.3, 256 x 2048 x 512 (128) 22.9 / 47.2, 512 x 1024 x 1024 (128) 44 / 91; by the same
// growth the two meet at about 256 tiles.
bool dkv_gemm_f32_few_rows(int dtype, int m, int n, int k) {
    return dtype == DKV_FP32 && k % 4 == 0 && (long)ceil_div(m, 64) * ceil_div(n, 64) <= 128;
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

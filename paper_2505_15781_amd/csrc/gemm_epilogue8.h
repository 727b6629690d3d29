// Epilogues of the 8-wavefront loop (included by gemm_pingpong.h). Same outputs as gemm_epilogue.h on the other
// accumulator layout: acc[h][b][i][j][v] is the element at row 32 MT wm + 16 MT h + 16 i + (lane & 15), column
// 32 NT wn + 16 NT b + 16 j + 4 (lane >> 4) + v of the workgroup's tile: a lane holds four consecutive columns of a row,
// so gate / up pairs are in one lane and the fp32 product leaves in 16-byte stores.
#pragma once

// fp32 product of one wavefront whose part of the tile starts at (row0, col0)
template <int MT, int NT>
__device__ __forceinline__ void store_tile8(const f32x4 (&acc)[2][2][MT][NT], float *out, int row0, int col0, int M, int N,
                                            int lane) {
    const bool vec = (N & 3) == 0;             // four columns of a row or none
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int m = row0 + (h * MT + i) * 16 + (lane & 15);
            float *row = out + (size_t)m * N;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int n = col0 + (b * NT + j) * 16 + 4 * (lane >> 4);
                    if (m >= M) continue;
                    if (vec) {
                        if (n < N) *reinterpret_cast<f32x4_el *>(row + n) = acc[h][b][i][j];
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (n + v < N) row[n + v] = acc[h][b][i][j][v];
                    }
                }
        }
}

template <int EPI, int MT, int NT, int WM, int WN>
__device__ __forceinline__ void run_epilogue8(const f32x4 (&acc)[2][2][MT][NT], const GemmEpilogue &ep, unsigned char *lds,
                                              int m0, int n0, int M, int N, int tile_n, int wm, int wn) {
    constexpr int BM = 32 * MT * WM, BN = 32 * NT * WN, NTHREADS = 512;
    const int tid = threadIdx.x, lane = tid & 63;
    if constexpr (EPI == EPI_SWIGLU) {
        // The activations of the tile go through LDS so that they leave as whole 16-byte pieces of consecutive columns
        // (from the accumulators a store would write 16 bytes of each of 16 rows).
        constexpr int STRIDE = BN + 16;        // bytes per row of BN / 2 bf16; + 16 spreads the 16 rows over the banks
        static_assert(BM * STRIDE <= 2 * (BM + BN) * 128, "fits the tile stages");
        bf16_t *f = static_cast<bf16_t *>(ep.out);
        const int F = N >> 1;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                unsigned char *row = lds + (wm * 32 * MT + (h * MT + i) * 16 + (lane & 15)) * STRIDE;
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int j = 0; j < NT; ++j) {
                        const f32x4 x = acc[h][b][i][j];     // gate, up, gate, up
                        const float y0 = x[0] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x[0])) * x[1];
                        const float y1 = x[2] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x[2])) * x[3];
                        const int col = wn * 32 * NT + (b * NT + j) * 16 + 4 * (lane >> 4);
                        *reinterpret_cast<uint32_t *>(row + col) = (uint32_t)f2bf(y0) | ((uint32_t)f2bf(y1) << 16);
                    }
            }
        __syncthreads();
        constexpr int CH = BN / 16;            // 16-byte pieces per row
        for (int e = tid; e < BM * CH; e += NTHREADS) {
            const int r = e / CH, ch = e % CH, m = m0 + r, c = (n0 >> 1) + ch * 8;
            if (m >= M) continue;
            const unsigned char *src = lds + r * STRIDE + ch * 16;
            bf16_t *dst = f + (size_t)m * F + c;
            if ((F & 7) == 0) {
                if (c < F) *reinterpret_cast<bf16x8_el *>(dst) = *reinterpret_cast<const u32x4 *>(src);
            } else {
                for (int v = 0; v < 8; ++v)
                    if (c + v < F) dst[v] = reinterpret_cast<const bf16_t *>(src)[v];
            }
        }
    } else {   // EPI_HEAD
        EpiSmem<BM, WN> &sm = *reinterpret_cast<EpiSmem<BM, WN> *>(lds);
        float *logits = static_cast<float *>(ep.out);
        bool nan = false;
        if (logits) store_tile8<MT, NT>(acc, logits, m0 + wm * 32 * MT, n0 + wn * 32 * NT, M, N, lane);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int r = wm * 32 * MT + (h * MT + i) * 16 + (lane & 15);
                float x[2 * NT * 4];
                float mx = -INFINITY;
#pragma unroll
                for (int q = 0; q < 2 * NT; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int n = n0 + wn * 32 * NT + q * 16 + 4 * (lane >> 4) + v;
                        float y = acc[h][q / NT][i][q % NT][v];
                        if (n >= N || n == ep.mask_id) y = -INFINITY;      // MASK can never be predicted
                        nan |= (y != y) && m0 + r < M;
                        x[4 * q + v] = y;
                        mx = fmaxf(mx, y);
                    }
                // the four lanes of a row: lane, lane ^ 16, lane ^ 32, lane ^ 48
                mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                float sum = 0.f;
                int best = 0x7fffffff;
#pragma unroll
                for (int q = 0; q < 2 * NT; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float y = x[4 * q + v];
                        if (y > -INFINITY) sum += __expf(y - mx);
                        if (y == mx && mx > -INFINITY) best = min(best, n0 + wn * 32 * NT + q * 16 + 4 * (lane >> 4) + v);   // lowest id on ties
                    }
                sum += __shfl_xor(sum, 16, 64);
                sum += __shfl_xor(sum, 32, 64);
                best = min(best, __shfl_xor(best, 16, 64));
                best = min(best, __shfl_xor(best, 32, 64));
                if (lane < 16) {
                    sm.red[r][wn] = mx;
                    sm.red2[r][wn] = sum;
                    sm.redi[r][wn] = best;
                }
            }
        if (__any(nan) && lane == 0) atomicOr(ep.status, 1 /* STATUS_NAN */);
        __syncthreads();
        merge_head_columns<BM, WN, NTHREADS>(sm, ep, m0, M, tile_n);
    }
}

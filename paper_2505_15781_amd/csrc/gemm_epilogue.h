// Epilogues of the projection kernel: what a row kernel would do after re-reading the product happens on the
// accumulators instead (included by gemm_kernel.h inside its namespace). Only epilogues without loads are here (see
// the note at GemmEpilogue).
//
// Accumulator layout (MFMA 32x32x16, wave (wm, wn) of the workgroup tile at (m0, n0)): acc[i][j][v] is the
// element at column n0 + (wn NT + j) 32 + (lane & 31), row m0 + (wm MT + i) 32 + 8 (v >> 2) + 4 (lane >> 5) + (v & 3).
// So the 32 lanes of a half-wave hold 32 consecutive columns of one row, neighbouring lanes neighbouring columns.
#pragma once

// value of the neighbouring lane (lane ^ 1)
__device__ __forceinline__ float lane_swap1(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));
}
// Reductions over the 32 lanes that hold one row, every lane getting the result: partners one, two, four, eight and 16 lanes
// apart, by data-parallel primitives and gfx950's row swap. Behind the first two steps the lanes of a quad agree, so that a
// mirrored half row and row hand over the value of the lane four and eight apart. The epilogue of the vocabulary projection is
// bound by these chains (three per row, 16 MT rows per wavefront): LDS permutes for the five steps against these, the whole launch
// on the same tiles: 126464 x 4096 at 33 rows 211 and 180 us (162 since those tiles have three stages of LDS), at 93 rows 204 and
// 189, 32000 x 2048 at 48 rows 38 and 31; the launch's floor, the weights once at 6 TB/s, is 173 and 22 us. (152064 x 3584 at 93
// rows, 128x256 tiles, 263 and 240; planned there are 192x256 tiles of 8 wavefronts, level with them, whose epilogue in
// gemm_epilogue8.h still permutes through LDS.)
template <int CTRL> __device__ __forceinline__ int dpp_move(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true); }
template <typename F> __device__ __forceinline__ int half_reduce(int x, F combine) {
    x = combine(x, dpp_move<0xB1>(x));        // quad_perm 1 0 3 2
    x = combine(x, dpp_move<0x4E>(x));        // quad_perm 2 3 0 1
    x = combine(x, dpp_move<0x141>(x));       // row_half_mirror
    x = combine(x, dpp_move<0x140>(x));       // row_mirror
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
    return combine((int)r[0], (int)r[1]);
}
__device__ __forceinline__ float as_f(int x) { return __builtin_bit_cast(float, x); }
__device__ __forceinline__ float half_sum(float v) {
    return as_f(half_reduce(__builtin_bit_cast(int, v), [](int a, int b) { return __builtin_bit_cast(int, as_f(a) + as_f(b)); }));
}
__device__ __forceinline__ float half_max(float v) {
    return as_f(half_reduce(__builtin_bit_cast(int, v), [](int a, int b) { return __builtin_bit_cast(int, fmaxf(as_f(a), as_f(b))); }));
}
__device__ __forceinline__ int half_min(int v) {
    return half_reduce(v, [](int a, int b) { return min(a, b); });
}

// LDS scratch of the epilogues, carved out of the (now idle) tile stages.
template <int BM, int WN> struct EpiSmem {
    float red[BM][WN];       // EPI_HEAD: maxima of a row over each wavefront's columns
    float red2[BM][WN];      //           sums of exp(x - max)
    int redi[BM][WN];        //           arg maxima
};

// The column statistics that the WN wavefronts of a row left in LDS, merged into the tile's record of the row.
template <int BM, int WN, int NTHREADS>
__device__ __forceinline__ void merge_head_columns(const EpiSmem<BM, WN> &sm, const GemmEpilogue &ep, int m0, int M, int tile_n) {
    for (int r = threadIdx.x; r < BM; r += NTHREADS) {
        const int m = m0 + r;
        if (m < M) {
            float mx = sm.red[r][0], sum = sm.red2[r][0];
            int best = sm.redi[r][0];
#pragma unroll
            for (int w = 1; w < WN; ++w) {      // ascending columns: ties keep the lower id
                const float om = sm.red[r][w], os = sm.red2[r][w];
                if (om > mx) {
                    sum = sum * __expf(mx - om) + os;      // mx == -inf only with sum == 0
                    mx = om;
                    best = sm.redi[r][w];
                } else if (om > -INFINITY) {
                    sum += os * __expf(om - mx);
                }
            }
            ep.head_part[(size_t)m * ep.head_tiles + tile_n] = HeadPartial{mx, sum, best, 0};
        }
    }
}

template <int EPI, int MT, int NT, int WM, int WN>
__device__ __forceinline__ void run_epilogue(f32x16 (&acc)[MT][NT], const GemmEpilogue &ep, void *smem_raw,
                                             int m0, int n0, int M, int N, int tile_n, int tiles_n) {
    constexpr int BM = 32 * MT * WM, NW = WM * WN, NTHREADS = 64 * NW;
    EpiSmem<BM, WN> &sm = *reinterpret_cast<EpiSmem<BM, WN> *>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int col = lane & 31, rsub = 4 * (lane >> 5);

    if constexpr (EPI == EPI_SWIGLU) {
        // columns 2j (gate_j) and 2j+1 (up_j) sit in neighbouring lanes; even lanes finish accumulator elements
        // 0..7 and odd lanes 8..15, so every lane runs half of the activations
        bf16_t *f = static_cast<bf16_t *>(ep.out);
        const int F = N >> 1;
        const bool odd = lane & 1;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = (wm * MT + i) * 32 + 8 * (v >> 2) + rsub + (v & 3), m = m0 + r;
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int n = n0 + (wn * NT + j) * 32 + col;
                    const float own = acc[i][j][v];
                    const float other = lane_swap1(own);
                    if ((v < 8) != odd) {
                        const float g = odd ? other : own, u = odd ? own : other;
                        const float y = g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g)) * u;
                        if (m < M && n < N) f[(size_t)m * F + (n >> 1)] = f2bf(y);
                    }
                }
            }
    } else {   // EPI_HEAD
        float *logits = static_cast<float *>(ep.out);
        bool nan = false;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = (wm * MT + i) * 32 + 8 * (v >> 2) + rsub + (v & 3), m = m0 + r;
                float x[NT];
                float mx = -INFINITY;
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int n = n0 + (wn * NT + j) * 32 + col;
                    x[j] = acc[i][j][v];
                    if (logits && m < M && n < N) logits[(size_t)m * N + n] = x[j];
                    if (n >= N || n == ep.mask_id) x[j] = -INFINITY;      // MASK can never be predicted
                    nan |= (x[j] != x[j]) && m < M;
                    mx = fmaxf(mx, x[j]);
                }
                mx = half_max(mx);
                float sum = 0.f;
                int best = 0x7fffffff;
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int n = n0 + (wn * NT + j) * 32 + col;
                    if (x[j] > -INFINITY) sum += __expf(x[j] - mx);
                    if (x[j] == mx && mx > -INFINITY) best = min(best, n);      // lowest id on ties
                }
                sum = half_sum(sum);
                best = half_min(best);
                if (col == 0) {
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

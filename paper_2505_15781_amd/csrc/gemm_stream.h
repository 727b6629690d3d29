// Projection kernel for one row of tiles of 256 rows (129 to 256 rows): 12 wavefronts, of which four multiply, four fetch
// the activations and four the weights (included by gemm_kernel.h inside its namespace).
//
// What bounds these launches is what a compute unit can have under way: about 180 lines of 128 bytes, returned in order, so
// that every line costs what the slowest around it does: 410 ns for weights from HBM, 113 ns for activations from L2.
// Fills alone, 256 x 24576 x 4096: 128x192 tiles, whose weights two workgroups fetch, 54 us; 256x96 tiles, whose weights
// enter one unit only and come with the non-temporal hint, 48 us with both operands issued tile by tile, 41 us (18 TB/s) with
// the weights issued two K tiles at a time by wavefronts of their own, which leaves stretches of the queue that hold only
// activations. (Three stages of activations: with two 53 us. All 8 wavefronts of a workgroup fetching and multiplying,
// K dealt to two groups: 63 us against 55 for the whole kernel; two fetching wavefronts per operand instead of four: 63.)
// With its consumer, cold weights, same card: 256 x 24576 x 4096 with SwiGLU 65.1 -> 53.0 us, 256 x 4096 x 12288
// 44.2 -> 40.4, 192 x 3584 x 18944 61.2 -> 46.4, 256 x 22016 x 4096 with SwiGLU 0.80 of the time. Per K tile the fills take
// 0.61 us, the products 0.57 (MFMAs 0.37: one wavefront per SIMD waits for its fragments), both together 0.66. Counted inside
// steps of 250 to 256 rows, the launches fetch the weights once and the activations once per XCD that works on their K slice:
// 1.05 to 1.07 of the bytes they cannot do without.
#pragma once

struct StreamTile {
    static constexpr int BM = 256, RA = 3, BURST = 2, RW = 2 * BURST;    // rows; stages of activations; K tiles of weights issued together; stages
};

template <int EPI, int NT>
__global__ __launch_bounds__(768) void gemm_stream(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W, float *__restrict__ P,
                                                   int m_upper, int m_cap, const int *__restrict__ m_dev, int N, int K,
                                                   int kt_per_split, const GemmEpilogue ep) {
    constexpr int MT = 2, BM = StreamTile::BM, BN = 32 * NT, RA = StreamTile::RA, B = StreamTile::BURST, RW = StreamTile::RW;
    constexpr int A_STAGE = BM * 128, W_STAGE = BN * 128, W_BASE = RA * A_STAGE;
    constexpr int IA = BM / 32, IW = NT;              // load instructions (8 rows) of a fetching wavefront per K tile
    static_assert((RA - 1) * IA < 64 && B * IW < 64, "vmcnt is a 6-bit counter");
    extern __shared__ __attribute__((aligned(16))) uint4 lds[];

    const int M = m_dev ? min(*m_dev, m_upper) : m_upper;
    const int kt_total = K / BK, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // XCD x runs the workgroups x, x + 8, ...: they take neighbouring places of the order (K slice, column of tiles), so that an
    // XCD reads few slices of the activations
    const int gx = gridDim.x, total = gx * gridDim.z, id = blockIdx.x + gx * blockIdx.z;
    const int pos = (id & 7) * (total >> 3) + min(id & 7, total & 7) + (id >> 3);
    const int bz = pos / gx, bx = pos - bz * gx;
    const int n0 = bx * BN, kt0 = bz * kt_per_split, nk = min(kt_total, kt0 + kt_per_split) - kt0;
    if (M <= 0) return;
    const int rot = (int)((unsigned)(bx * 5) % (unsigned)nk);     // first K tile: not all workgroups sweep the same columns
    const uint32_t lds_base = (uint32_t)(size_t)(lds_ptr_t)lds;

    // One barrier per K tile, at which tile k has landed (the fetching wavefronts have waited for it) and tile k - 1 has been
    // read; behind it the stages of tile k - 1 and, for the weights, of the pair before are filled again.
    if (wave >= 4) {
        const int w = wave & 3;
        const bool is_w = wave >= 8;
        uint32_t off[IA];
        const int r0 = is_w ? n0 : 0, last = (is_w ? N : M) - 1;
#pragma unroll
        for (int i = 0; i < IA; ++i) {
            // LDS row r holds the chunk (16 bytes) c of the K tile in slot c ^ ((r >> 1) & 7); rows past the end are clamped
            const int row = (4 * i + w) * 8 + (lane >> 3);
            off[i] = (uint32_t)(min(r0 + row, last) - r0) * (uint32_t)(2 * K) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
        }
        const char *base = reinterpret_cast<const char *>((is_w ? W : A) + (size_t)r0 * K + (size_t)kt0 * BK);
        auto k_at = [&](int t) {
            int k = t + rot;
            if (k >= nk) k -= nk;
            return base + (size_t)k * (BK * 2);
        };
        if (is_w) {
            auto burst = [&](int t0) {
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    if (t0 + j >= nk) break;
                    const char *src = k_at(t0 + j);
                    const uint32_t dst = lds_base + W_BASE + ((t0 + j) % RW) * W_STAGE + w * 1024;
#pragma unroll
                    for (int i = 0; i < IW; ++i) dma16_at_nt(off[i], src, dst + i * 4096);
                }
            };
            burst(0);
            for (int k = 0; k < nk; ++k) {
                if (k % B == 0) __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (k % B == 0) burst(k + B);
            }
        } else {
            auto fetch = [&](int t, int stage) {
                const char *src = k_at(t);
                const uint32_t dst = lds_base + stage * A_STAGE + w * 1024;
#pragma unroll
                for (int i = 0; i < IA; ++i) dma16_at(off[i], src, dst + i * 4096);
            };
#pragma unroll
            for (int t = 0; t < RA - 1; ++t)
                if (t < nk) fetch(t, t);
            int stage = RA - 1;
            for (int k = 0; k < nk; ++k) {
                if (k + RA - 2 < nk) __builtin_amdgcn_s_waitcnt(waitcnt_imm((RA - 2) * IA, false));
                else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, false));
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (k + RA - 1 < nk) fetch(k + RA - 1, stage);
                stage = stage + 1 == RA ? 0 : stage + 1;
            }
        }
        return;
    }
    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    bf16x8 af[2][MT], wf[2][NT];
    const unsigned char *ra = reinterpret_cast<const unsigned char *>(lds) + (wave * MT * 32 + (lane & 31)) * 128;
    const unsigned char *rw = reinterpret_cast<const unsigned char *>(lds) + W_BASE + (lane & 31) * 128;
    const int sw = (lane >> 1) & 7;                    // the swizzle of a row: bands of 32 rows do not change it
    auto ldfrag = [&](int sa, int sb, int ks, int fb) {
        const int chunk = ((2 * ks + (lane >> 5)) ^ sw) << 4;
        // in the order in which the products need them
        af[fb][0] = *reinterpret_cast<const bf16x8 *>(ra + sa * A_STAGE + chunk);
#pragma unroll
        for (int j = 0; j < NT; ++j) wf[fb][j] = *reinterpret_cast<const bf16x8 *>(rw + sb * W_STAGE + j * 4096 + chunk);
#pragma unroll
        for (int i = 1; i < MT; ++i) af[fb][i] = *reinterpret_cast<const bf16x8 *>(ra + sa * A_STAGE + i * 4096 + chunk);
    };
    auto next_tile = [&]() {
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    int sa = 0, sb = 0;
    next_tile();
    ldfrag(0, 0, 0, 0);
    for (int t = 0; t < nk; ++t) {
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            if (ks + 1 < BK / 16) {
                ldfrag(sa, sb, ks + 1, (ks + 1) & 1);
            } else if (t + 1 < nk) {
                next_tile();
                sa = sa + 1 == RA ? 0 : sa + 1;
                sb = sb + 1 == RW ? 0 : sb + 1;
                ldfrag(sa, sb, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks & 1][i], wf[ks & 1][j], acc[i][j], 0, 0, 0);
        }
    }
    if constexpr (EPI == EPI_STORE) {
        float *out = P + (size_t)bz * m_cap * N;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int n = n0 + j * 32 + (lane & 31);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int m = (wave * MT + i) * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                    if (m < M && n < N) out[(size_t)m * N + n] = acc[i][j][v];
                }
            }
    } else {
        static_assert(EPI != EPI_HEAD, "the fetching wavefronts have left: no barriers in the epilogue");
        run_epilogue<EPI, MT, NT, 4, 1>(acc, ep, lds, 0, n0, M, N, n0 / BN, 0);
    }
}

template <int EPI, int NT>
int launch_stream(const void *A, const void *W, float *P, int m_upper, int m_cap, const int *m_dev, int n, int k, int split,
                  const GemmEpilogue &ep, hipStream_t s) {
    constexpr int BN = 32 * NT, smem = (StreamTile::RA * StreamTile::BM + StreamTile::RW * BN) * 128;
    static_assert(smem <= 160 * 1024, "LDS of a compute unit");
    if (m_upper > StreamTile::BM) {
        dkv_set_error("this kernel has one row of tiles of %d rows, not %d", StreamTile::BM, m_upper);
        return DKV_E_UNSUPPORTED;
    }
    const int kt_total = k / BK, kps = ceil_div(kt_total, split);
    const dim3 grid(ceil_div(n, BN), 1, ceil_div(kt_total, kps));
    if (EPI != EPI_STORE && grid.z != 1) {
        dkv_set_error("a fused epilogue needs one K slice");
        return DKV_E_INVALID_ARG;
    }
    if (EPI == EPI_SWIGLU && (n & 1)) {
        dkv_set_error("the fused SwiGLU epilogue pairs neighbouring columns: their number must be even");
        return DKV_E_INVALID_ARG;
    }
    // set once per process; the call is idempotent, so threads that race here only repeat it
    static std::atomic<bool> attr_set{false};
    if (!attr_set.load(std::memory_order_acquire)) {
        DKV_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_stream<EPI, NT>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, smem));
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((gemm_stream<EPI, NT>), grid, dim3(768), smem, s, (const bf16_t *)A, (const bf16_t *)W, P, m_upper, m_cap,
                       m_dev, n, k, kps, ep);
    DKV_LAUNCH_CHECK();
    return DKV_OK;
}

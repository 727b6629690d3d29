// Main loop of the projection kernel for the large tiles: 8 wavefronts in two groups of four that alternate between
// fetching operands and multiplying (included by gemm_kernel.h inside its namespace).
//
// Why: with thousands of rows the projections are bound by the matrix pipes under the card's power limit, and by how
// many cycles those pipes wait. Measured on registers only, with random operands: MFMA 32x32x16 runs at 1.88 PFLOP/s,
// 16x16x32 at 2.12-2.14 (2.41-2.48 with operands of zeros). So the tile is multiplied with 16x16x32, by 8 wavefronts, two
// per SIMD, one of each group, of which one fetches while the other multiplies. Fragment reads of all 8 wavefronts move
// 192 KB through LDS per 256x256x64 step, 37 % of its 2048 MFMA cycles at the 256 B/cycle that conflict-free 16-byte reads reach
// (a loop of these reads alone), beside the fills' writes: they have to be spread evenly under the MFMAs, which the alternation does.
//
// Schedule: a wavefront's 32 MT x 32 NT part of the tile is worked on as 2 x 2 quarters (row half A0 / A1, column half
// B0 / B1), one quarter (2 MT NT MFMAs) per phase. A phase is a fetch slot (LDS reads of the fragments it needs, the
// DMA of one quarter-tile region for a later K tile) and a multiply slot, with a barrier after each. Group 1 runs one
// barrier behind group 0, so in every slot one group multiplies while the other fetches, and each SIMD's matrix pipe
// always has a wavefront with operands in registers.
//   phase        1            2            3            4
//   LDS reads    A0(t)        B1(t)        A1(t)        B0(t+1)
//   DMA          A1(t+1)      A0(t+2)      B0(t+2)      B1(t+2)
//   multiplies   A0 B0        A0 B1        A1 B1        A1 B0
// A region is refilled as soon as both groups have read it (one barrier later), so with two LDS stages a load has 6
// to 7 phases, 3000 cycles and more, to land: longer than a miss under load, which one tile of lookahead (2048 cycles)
// is not. At 6144 rows a K step of 256x256x64 takes 2460 cycles of which its MFMAs need 2048, 192x256x64 2240-2270 and
// 256x192x64 2450-2470 of 1536 each; over whole launches the matrix pipes are busy 60-69 % of the cycles. Against the
// 4-wavefront loop that these tiles had before (one wavefront per SIMD, 32x32x16, one K tile ahead), same box:
//   6144 x 24576 x 4096 with SwiGLU   1112 -> 872 us (1.42 PFLOP/s)      6144 x 12288 x 4096   566 -> 489 us
//   6144 x 4096 x 12288 (192x256)      592 -> 475 us                     4096 x 37888 x 3584   1078 -> 825 us
// (on other cards 872-939, 489-564, 472-484 and 800-860 us)
#pragma once

// all but the newest VM vector memory operations of this wavefront are done, and all its LDS operations
template <int VM> __device__ __forceinline__ void wait_all_but() {
    static_assert(VM >= 0 && VM < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | 0x0070);
}
__device__ __forceinline__ void slot_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

template <int V> struct IntC { static constexpr int value = V; };

#include "gemm_epilogue8.h"

template <int EPI, int MT, int NT, int WM, int WN>
__device__ __forceinline__ void pingpong_tiles(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W,
                                               float *__restrict__ P, int m_upper, int m_cap,
                                               const int *__restrict__ m_dev, int N, int K, int kt_per_split,
                                               int frac_units, int flags, const GemmEpilogue &ep, unsigned char *lds) {
    static_assert(WM * WN == 8, "two wavefronts per SIMD");
    constexpr int BM = 32 * MT * WM, BN = 32 * NT * WN, STAGE = (BM + BN) * 128;
    // DMA instructions (8 rows of 128 B each) of a half of the A / W tile: two per wavefront, or two for group 0 and
    // one for group 1
    constexpr int IA = 2 * MT * WM, IB = 2 * NT * WN;
    static_assert(IA % 4 == 0 && IB % 4 == 0 && IA > 8 && IB > 8 && IA <= 16 && IB <= 16, "one or two per wavefront");
    constexpr int CA0 = 2, CA1 = IA == 16 ? 2 : 1, CB0 = 2, CB1 = IB == 16 ? 2 : 1;    // per wavefront of group 0 / 1

    const int M = m_dev ? min(*m_dev, m_upper) : m_upper;
    const int kt_total = K / BK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), group = wave >> 2;
    const int wm = wave / WN, wn = wave % WN;
    const uint32_t lds_base = (uint32_t)(size_t)(lds_ptr_t)lds;
    const int tiles_n = (N + BN - 1) / BN;
    int unit = frac_units ? blockIdx.x * frac_units : 0;
    const int unit_end = frac_units ? min(unit + frac_units, tiles_n * ((m_upper + BM - 1) / BM) * kt_total) : 0;
  for (;;) {
    const TileWork w = next_tile_work<BM, BN>(unit, unit_end, frac_units, kt_total, kt_per_split, tiles_n, flags);
    if (w.m0 < M) {
    const int nk = w.nk, m0 = w.m0, n0 = w.n0;
    const int kt_rot = (flags & GEMM_FLAG_STAGGER) ? (int)((unsigned)(n0 / BN * 5 + m0 / BM * 3) % (unsigned)nk) : 0;

    // Region h (half) of the A tile: rows [32 MT b + 16 MT h, + 16 MT) of every band b < WM, likewise for W with NT
    // and WN. LDS row r holds the chunk (16 bytes) c of the K tile in slot c ^ ((r >> 1) & 7), as in the other loop.
    // Rows past the end are clamped: they only feed outputs that are never stored.
    uint32_t va[2][2], vw[2][2], la[2][2], lw[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = (i * 8 + wave) * 8, sub = lane >> 3;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ra = q / (16 * MT) * (32 * MT) + h * 16 * MT + q % (16 * MT), rw = q / (16 * NT) * (32 * NT) + h * 16 * NT + q % (16 * NT);
            const int a = ra + sub, b = rw + sub;
            va[h][i] = (uint32_t)(min(m0 + a, M - 1) - m0) * (uint32_t)(2 * K) + (((lane & 7) ^ ((a >> 1) & 7)) << 4);
            vw[h][i] = (uint32_t)(min(n0 + b, N - 1) - n0) * (uint32_t)(2 * K) + (((lane & 7) ^ ((b >> 1) & 7)) << 4);
            la[h][i] = lds_base + ra * 128;
            lw[h][i] = lds_base + (BM + rw) * 128;
        }
    }
    const char *Ab = reinterpret_cast<const char *>(A + (size_t)m0 * K + (size_t)w.kt0 * BK);
    const char *Wb = reinterpret_cast<const char *>(W + (size_t)n0 * K + (size_t)w.kt0 * BK);
    auto k_offset = [&](int t) {
        int tt = min(t, nk - 1) + kt_rot;       // past the end only with one K tile: a second fetch that nobody reads
        if (tt >= nk) tt -= nk;
        return (size_t)tt * (BK * 2);
    };
    auto dma_a = [&](int h, int t, int stage) {
        const char *base = Ab + k_offset(t);
        dma16_at(va[h][0], base, la[h][0] + stage * STAGE);
        if (IA == 16 || group == 0) dma16_at(va[h][1], base, la[h][1] + stage * STAGE);
    };
    auto dma_w = [&](int h, int t, int stage) {
        const char *base = Wb + k_offset(t);
        dma16_at(vw[h][0], base, lw[h][0] + stage * STAGE);
        if (IB == 16 || group == 0) dma16_at(vw[h][1], base, lw[h][1] + stage * STAGE);
    };
    // wait until at most `a` A regions and `b` W regions issued by this wavefront are still on their way
    auto wait_regions = [&](auto a, auto b) {
        constexpr int v0 = decltype(a)::value * CA0 + decltype(b)::value * CB0, v1 = decltype(a)::value * CA1 + decltype(b)::value * CB1;
        if (v0 == v1 || group == 0) wait_all_but<v0>();
        else wait_all_but<v1>();
    };

    f32x4 acc[2][2][MT][NT];      // [row half][column half][16-row tile][16-column tile]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[h][b][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // fragments: lane l holds row l & 15, K elements 8 (l >> 4) + [0, 8) of each 32-element K step
    bf16x8 af[MT][2], w0[2][NT][2], w1[NT][2];
    const int kc0 = ((lane >> 4) ^ ((lane & 15) >> 1)) << 4, kc1 = ((4 + (lane >> 4)) ^ ((lane & 15) >> 1)) << 4;
    const unsigned char *ra = lds + (wm * 32 * MT + (lane & 15)) * 128, *rw = lds + (BM + wn * 32 * NT + (lane & 15)) * 128;
    auto read_a = [&](int h, int stage) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const unsigned char *p = ra + stage * STAGE + (h * MT + i) * (16 * 128);
            af[i][0] = *reinterpret_cast<const bf16x8 *>(p + kc0);
            af[i][1] = *reinterpret_cast<const bf16x8 *>(p + kc1);
        }
    };
    auto read_w = [&](bf16x8 (&d)[NT][2], int h, int stage) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const unsigned char *p = rw + stage * STAGE + (h * NT + j) * (16 * 128);
            d[j][0] = *reinterpret_cast<const bf16x8 *>(p + kc0);
            d[j][1] = *reinterpret_cast<const bf16x8 *>(p + kc1);
        }
    };
    // the weights are the first operand: a lane then holds four consecutive output columns of one row
    auto multiply = [&](f32x4 (&c)[MT][NT], const bf16x8 (&b)[NT][2]) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][ks], af[i][ks], c[i][j], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
        slot_barrier();
    };
    // K tile t out of stage S. The waits count the regions issued after the one that the next phase of either group
    // reads; the last two tiles, which fetch less, have counts of their own. The branches are scalar and hold no
    // register writes, so that the tile stays one stretch of code (peeled tails made the compiler spill).
    auto k_tile = [&](int t, auto stage) {
        constexpr int S = decltype(stage)::value;
        const bool more1 = t + 1 < nk, more2 = t + 2 < nk;
        read_a(0, S);
        if (more1) {
            dma_a(1, t + 1, S ^ 1);
            wait_regions(IntC<3>{}, IntC<2>{});               // B1(t) has landed
        } else {
            wait_regions(IntC<1>{}, IntC<0>{});
        }
        slot_barrier();
        multiply(acc[0][0], w0[S]);
        read_w(w1, 1, S);
        if (more2) {
            dma_a(0, t + 2, S);
            wait_regions(IntC<3>{}, IntC<2>{});               // A1(t)
        } else if (more1) {
            wait_regions(IntC<2>{}, IntC<2>{});
        } else {
            wait_regions(IntC<0>{}, IntC<0>{});
        }
        slot_barrier();
        multiply(acc[0][1], w1);
        read_a(1, S);
        if (more2) {
            dma_w(0, t + 2, S);
            wait_regions(IntC<2>{}, IntC<2>{});               // A0(t+1), B0(t+1)
        } else {
            wait_regions(IntC<1>{}, IntC<1>{});
        }
        slot_barrier();
        multiply(acc[1][1], w1);
        read_w(w0[S ^ 1], 0, S ^ 1);                          // after the last tile: read, never used
        if (more2) dma_w(1, t + 2, S);
        wait_all_but<63>();
        slot_barrier();
        multiply(acc[1][0], w0[S]);
    };

    dma_a(0, 0, 0); dma_w(0, 0, 0); dma_w(1, 0, 0); dma_a(1, 0, 0);
    dma_a(0, 1, 1); dma_w(0, 1, 1); dma_w(1, 1, 1);
    wait_regions(IntC<2>{}, IntC<3>{});                       // A0(0), B0(0)
    slot_barrier();
    read_w(w0[0], 0, 0);
    wait_all_but<63>();
    slot_barrier();
    if (group == 1) slot_barrier();                           // group 1 runs one slot behind
    for (int t = 0; t < nk; t += 2) {
        k_tile(t, IntC<0>{});
        if (t + 1 < nk) k_tile(t + 1, IntC<1>{});
    }
    if (group == 0) slot_barrier();                           // level again: every LDS read of the tile is done

    if constexpr (EPI == EPI_STORE) {
        float *out = P + (size_t)w.slot * m_cap * N;
        store_tile8<MT, NT>(acc, out, m0 + wm * 32 * MT, n0 + wn * 32 * NT, M, N, lane);
    } else {
        run_epilogue8<EPI, MT, NT, WM, WN>(acc, ep, lds, m0, n0, M, N, n0 / BN, wm, wn);
    }
    }   // m0 < M
    if (!frac_units || unit >= unit_end) break;
    // stores count in vmcnt: the waits of the next part start from zero; every wavefront is done with LDS
    wait_all_but<0>();
    __syncthreads();
  }
}

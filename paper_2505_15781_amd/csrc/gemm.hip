// Projection kernels: partial[s][m][n] = A[m, k-slice s] * W[n, k-slice s]^T, fp32 accumulation.
//
// The active rows of a denoising step (Algorithm 1 line 3: the transformer runs on x[M_{t-1}] only)
// are the M dimension; their count lives on the device, so kernels bound M by *m_dev.
//
// bf16, K a multiple of 64 (every model shape): `gemm_dma`. Tiles of 192 rows or columns and more by 256 take the
// 8-wavefront loop of gemm_pingpong.h; what follows is about the 4-wavefront loop of the others. MFMA 32x32x16 tiles; the A and W tiles of
// a K step travel from global memory straight into LDS (global_load_lds_dwordx4: 16 bytes per lane, lane i
// lands at base + 16 i) through a ring of STAGES buffers, so up to STAGES-1 tiles are in flight without
// holding registers. The LDS layout XOR-swizzles the 16-byte chunks of a 128-byte row with (row >> 1)
// so a fragment read of 16 consecutive rows touches every bank once; the swizzle is applied by choosing
// which global chunk each lane fetches. Fragment reads run one K sub-step ahead of the MFMAs, across tile
// boundaries. Measured on MI355X a compute unit sustains 50-60 GB/s of such fills whatever the depth,
// so the tile shapes below are chosen to keep the bytes each workgroup pulls (W tile + A tile) small
// relative to its MFMA work, and K is split across workgroups only as far as needed to fill 256 CUs.
// Two launch options, both measured: `stagger` starts each workgroup's K loop at a different tile (unsplit
// launches otherwise sweep the same columns of A and W in step and crowd a few memory channels: up to 25 %
// on the widest projection at <= 128 rows); `xcd_group` renumbers workgroups so that the 32 that run
// together on one XCD (hardware sends workgroup i to XCD i mod 8) cover a compact block of tiles, 6 rows high, and
// share their A and W tiles through that XCD's L2 (heights 3 to 12 are within 4 % of each other at 6144 rows, 1 and 24
// cost 5-15 %).
// bf16, other K (multiple of 8): `gemm_reg`, register-staged tiles. fp32 mode / anything else: `gemm_simt`.
#include <atomic>

#include "common.h"

namespace {

constexpr int BK = 64;   // K elements per LDS tile (8 chunks of 8 bf16)

// Register-staged variant for K that is a multiple of 8 but not of 64 (zero-fills the K tail).
__global__ __launch_bounds__(256) void gemm_reg(const bf16_t *__restrict__ A, const bf16_t *__restrict__ W,
                                                float *__restrict__ P, int m_upper, int m_cap,
                                                const int *__restrict__ m_dev, int N, int K, int kt_per_split) {
    constexpr int MT = 2, BM = 64, BN = 128, CA = 2, CW = 4;
    __shared__ uint4 lds[2][(BM + BN) * 8];
    const int M = m_dev ? min(*m_dev, m_upper) : m_upper;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    if (m0 >= M) return;
    const int kt_total = (K + BK - 1) / BK;
    const int kt0 = blockIdx.z * kt_per_split, kt1 = min(kt_total, kt0 + kt_per_split);
    const int tid = threadIdx.x, lane = tid & 63, wn = tid >> 6;
    uint4 ra[CA], rw[CW];
    auto load_global = [&](int kt) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            int c = tid + 256 * i, row = c >> 3, kc = c & 7, gm = m0 + row, gk = kt * BK + kc * 8;
            ra[i] = (gm < M && gk < K) ? *reinterpret_cast<const uint4 *>(A + (size_t)gm * K + gk) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < CW; ++i) {
            int c = tid + 256 * i, row = c >> 3, kc = c & 7, gn = n0 + row, gk = kt * BK + kc * 8;
            rw[i] = (gn < N && gk < K) ? *reinterpret_cast<const uint4 *>(W + (size_t)gn * K + gk) : make_uint4(0, 0, 0, 0);
        }
    };
    auto store_lds = [&](int buf) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            int c = tid + 256 * i, row = c >> 3, kc = c & 7;
            lds[buf][row * 8 + (kc ^ ((row >> 1) & 7))] = ra[i];
        }
#pragma unroll
        for (int i = 0; i < CW; ++i) {
            int c = tid + 256 * i, row = c >> 3, kc = c & 7;
            lds[buf][(BM + row) * 8 + (kc ^ ((row >> 1) & 7))] = rw[i];
        }
    };
    f32x16 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    if (kt0 < kt1) {
        load_global(kt0);
        store_lds(0);
    }
    __syncthreads();
    for (int kt = kt0; kt < kt1; ++kt) {
        const int buf = (kt - kt0) & 1;
        if (kt + 1 < kt1) load_global(kt + 1);
        const bf16x8 *tile = reinterpret_cast<const bf16x8 *>(lds[buf]);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int chunk = 2 * ks + (lane >> 5);
            const int wrow = wn * 32 + (lane & 31);
            const bf16x8 wfr = tile[(BM + wrow) * 8 + (chunk ^ ((wrow >> 1) & 7))];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int row = i * 32 + (lane & 31);
                const bf16x8 afr = tile[row * 8 + (chunk ^ ((row >> 1) & 7))];
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afr, wfr, acc[i], 0, 0, 0);
            }
        }
        if (kt + 1 < kt1) store_lds(buf ^ 1);
        __syncthreads();
    }
    float *out = P + (size_t)blockIdx.z * m_cap * N;
    const int n = n0 + wn * 32 + (lane & 31);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = m0 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (m < M && n < N) out[(size_t)m * N + n] = acc[i][v];
        }
}

// Plain FMA tile kernel: 64x64 outputs per workgroup, 4x4 per thread.
template <typename T>
__global__ __launch_bounds__(256) void gemm_simt(const T *__restrict__ A, const T *__restrict__ W,
                                                 float *__restrict__ P, int m_upper,
                                                 const int *__restrict__ m_dev, int N, int K) {
    constexpr int TM = 64, TN = 64, TK = 16;
    __shared__ float As[TK][TM + 4], Ws[TK][TN + 4];
    const int M = m_dev ? min(*m_dev, m_upper) : m_upper;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    if (m0 >= M) return;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    float acc[4][4] = {};
    for (int kb = 0; kb < K; kb += TK) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int e = tid + 256 * i, row = e >> 4, kk = e & 15;
            int gk = kb + kk;
            As[kk][row] = (m0 + row < M && gk < K) ? El<T>::ld(A + (size_t)(m0 + row) * K + gk) : 0.f;
            Ws[kk][row] = (n0 + row < N && gk < K) ? El<T>::ld(W + (size_t)(n0 + row) * K + gk) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < TK; ++kk) {
            float a[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = Ws[kk][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int m = m0 + ty * 4 + i, n = n0 + tx * 4 + j;
            if (m < M && n < N) P[(size_t)m * N + n] = acc[i][j];
        }
}

struct KindInfo {
    int bm, bn;
};
constexpr KindInfo kKinds[] = {
    {32, 128},    // GEMM_DMA_32x128   <1,1,1,4> 4 stages
    {64, 128},    // GEMM_DMA_64x128   <2,1,1,4> 4 stages (vocabulary statistics: <1,2,2,2> 3 stages)
    {128, 128},   // GEMM_DMA_128x128  <2,2,2,2> 3 stages
    {128, 256},   // GEMM_DMA_128x256  <2,4,2,2> 3 stages
    {256, 256},   // GEMM_DMA_256x256  <4,2,2,4> 2 stages, 8 wavefronts
    {128, 96},    // GEMM_DMA_128x96   <1,3,4,1> 4 stages
    {128, 192},   // GEMM_DMA_128x192  <2,3,2,2> 3 stages
    {256, 192},   // GEMM_DMA_256x192  <2,3,4,2> 2 stages, 8 wavefronts
    {192, 256},   // GEMM_DMA_192x256  <3,2,2,4> 2 stages, 8 wavefronts
};
static_assert(sizeof(kKinds) / sizeof(kKinds[0]) == GEMM_DMA_LAST + 1, "one entry per gemm_dma kind");
static_assert(GEMM_DMA_192x256 == DKV_GEMM_DMA_192x256 && GEMM_REG_64x128 == DKV_GEMM_REG_64x128 &&
                  GEMM_SIMT == DKV_GEMM_SIMT && GEMM_KINDS == DKV_PROF_ATTN,
              "the kinds of the public header are these");

// Number of K slices that is really launched for a requested split (no empty slice).
int effective_split(int k, int split) {
    const int kt_total = ceil_div(k, BK), kps = ceil_div(kt_total, split < 1 ? 1 : split);
    return ceil_div(kt_total, kps);
}

}  // namespace

GemmPlan dkv_gemm_plan(int dtype, int m_upper, int n, int k, int slices_go_to) {
    GemmPlan p;
    p.split_k = 1;
    p.frac_units = 0;
    p.flags = 0;
    if (dtype != DKV_BF16 || (k % 8) != 0) {
        p.kind = GEMM_SIMT;
        return p;
    }
    if (k % BK != 0) {
        p.kind = GEMM_REG_64x128;
        return p;
    }
    // Tile shape and K split: the candidate with the smallest predicted launch time. The prediction is a
    // small model of these kernels on MI355X, its constants fitted to two sweeps of the (tile shape, split) pairs
    // over the layer and vocabulary shapes of the 8B and 7B models at 31 row counts from 16 to 12288 (beyond 2048 rows
    // unsplit only), each launch timed together with the row kernel that consumes it, on weights that no cache holds
    // (mean loss against the best measured candidate 1.1 %, worst 14 %; with the constants of the 4-wavefront kernels for
    // all tiles 5.8 % and 70 %). A third sweep, of splits 1 to 8 at 2048 to 8192 rows over six layer shapes and seven narrow
    // ones (512 to 3072 columns), was not fitted to: mean loss 0.7 %, worst 14 %. Slices pay there too: 3584 x 18944 at 2049
    // rows 313 -> 248 us, 512 x 4096 at 2049 rows 41 -> 25, 1024 x 8192 at 3072 rows 83 -> 63, 4096 x 12288 at 4352 rows
    // 471 -> 421 us.
    //   a workgroup of the 4-wavefront tiles needs, per K tile, the longer of filling its LDS stage (52 GB/s per compute
    //   unit, 14.5 TB/s over all workgroups in flight) and its MFMAs (5.7 TFLOP/s per compute unit);
    //   a workgroup of the 8-wavefront tiles needs the times of kPingPong, alone and with the whole chip at work;
    //   128x256 tiles have no second workgroup on the compute unit that would work in a round's first fills and epilogue, and
    //   lose that time with every further round where the epilogue computes (SwiGLU, vocabulary statistics); one that only stores
    //   the fp32 product is shorter with them than with the 8-wavefront tiles (24576 x 4096 at 640 rows, 128x256 / 192x256 tiles: SwiGLU 150 /
    //   144 us, product 139 / 160; 37888 x 3584 at 384 rows 148 / 136 and 145 / 152; up to K = 6144: beyond, 8-wavefront tiles in K slices
    //   are ahead for products too, 22016 x 11008 at 608 rows 439 / 361, 37888 x 8192 at 288 rows 317 / 305);
    //   workgroups run in rounds of 256 (one per compute unit), a partly filled round costs a full one;
    //   no launch beats streaming its operands and results once;
    //   every further K slice adds the write and re-read of its partial sums by the consumer; a reduction of its own also
    //   reads the first slice and is a launch more (fitted with dkv_gemm over 12 shapes at 8 to 5000 rows: mean loss 1.3 %;
    //   charged like the consumer's, 400 x 4608 x 3584 took 36.6 us in 4 slices against 29.2 in one).
    // The times of 256x256 tiles and of a further round of 128x256 tiles are those of a chip that has been busy for 12 ms and
    // more, as it is inside a step. Against the constants of single launches, over 1440 launches (27 layer shapes, 65 to 6144 rows; stored
    // products with and without a reduction of their own, SwiGLU): 0.999 of the time on average. Planned differently are 37888 x
    // 3584 at 257 to 384 rows with SwiGLU, 192x256 for 128x256 tiles, 148 -> 133-140 us; 24576 x 4096 at 513 to 640 rows, the same,
    // 150 -> 144; 4096 x 12288 at 410 to 512 rows, 256x256 in 6 slices for 128x256 in 4, 70 -> 67; 24576 x 4096 at 3072 rows, 256x256 for
    // 192x256, 506 -> 489; 152064 x 3584 at 65 to 128 candidates, 192x256 for 128x256, level; and, the one that loses more than
    // 3 %, 8192 x 8192 at 413 to 512 rows, 256x256 in 3 slices for 4, 76 -> 84 (rows 16 KB apart; a time that repairs it takes the gain
    // of 4096 x 12288 away).
    // Tiles of 96 and 192 columns or rows exist because 12288 / 96 = 128 and 24576 / 192 = 128 column tiles make
    // exactly one or two full rounds where 128- and 256-column tiles leave a quarter of the chip idle, and 129..192 or
    // 257..384 rows fill one or two 192-row tiles (320 rows of the 8B vocabulary: 821 -> 393 us).
    // Products of more than 768 tiles are not sliced: a last round that is nearly empty is a small part of theirs (4096 x
    // 12288 at 9217 rows, 592 tiles: 2 slices 865 against 896 us; 3584 x 18944 at 14017 rows, 770: 1725 against 1788).
    // The planner runs for every row count that a run can have when the run is set up, so divisions are kept out of the
    // inner loop.
    constexpr double kFillPerCu = 52032.0, kFlopsPerCu = 5698686.0, kFillAll = 14478510.0;   // bytes, flops per us
    constexpr double kPerStream = 1.0 / 7841520.0, kPerReduce = 1.0 / 1849696.0;                // us per byte
    constexpr double kLaunch = 3.5, kPipeFill = 0.7, kPipeFill8 = 0.16, kReduceFixed = 3.2, kNextRound128x256 = 14.0;     // us
    struct PingPong { double alone, full; };                                                    // us per K tile
    constexpr PingPong kPingPong[] = {{}, {}, {}, {}, {1.130, 1.290}, {}, {}, {1.041, 1.092}, {0.980, 1.078}};
    static_assert(GEMM_DMA_256x256 == 4 && GEMM_DMA_256x192 == 7 && GEMM_DMA_192x256 == 8 && GEMM_DMA_LAST == 8, "order of kPingPong");
    const int kt_total = k / BK;
    const bool store_only = (slices_go_to == SLICES_LAUNCH || slices_go_to == SLICES_PRODUCT) && kt_total <= 96;
    struct { int s, nk; } slices[6];       // K slices worth trying, K tiles of each
    int n_slices = 0;
    for (int s : {1, 2, 3, 4, 6, 8}) {
        const int nk = ceil_div(kt_total, s);
        if (s == 1 || (slices_go_to != SLICES_NONE && nk >= 8 && ceil_div(kt_total, nk) == s)) slices[n_slices++] = {s, nk};
    }
    const double product = 4.0 * m_upper * (double)n, operands = 2.0 * n * k + 2.0 * m_upper * (double)k;
    double best = 0.0, best_work = 0.0;
    p.kind = -1;
    for (int kind = 0; kind <= GEMM_DMA_LAST; ++kind) {
        const KindInfo &ki = kKinds[kind];
        if (ki.bm > 32 && ki.bm >= 4 * m_upper) continue;       // mostly padding
        if (ki.bm < 128 && m_upper > 4 * ki.bm) continue;       // W re-read too often
        const int tiles = ceil_div(m_upper, ki.bm) * ceil_div(n, ki.bn);
        const double fill = (ki.bm + ki.bn) * 128.0, flops = 2.0 * ki.bm * ki.bn * BK;
        const double t_cu = fill / kFillPerCu > flops / kFlopsPerCu ? fill / kFillPerCu : flops / kFlopsPerCu;
        const double t_all = fill / kFillAll;                   // per workgroup in flight
        const PingPong &pp = kPingPong[kind];
        const bool eight = pp.full > 0.0;
        for (int i = 0; i < n_slices && (i == 0 || tiles <= 768); ++i) {
            const int s = slices[i].s;
            const long wgs = (long)tiles * s, rounds = (wgs + 255) / 256;
            double t_rounds;                   // per K tile, over all rounds
            if (eight) {
                const double last = pp.full * (double)(wgs - (rounds - 1) * 256) * (1.0 / 256.0);
                t_rounds = (rounds - 1) * pp.full + (last > pp.alone ? last : pp.alone);
            } else {
                const double all = (double)(wgs < 256 ? wgs : 256) * t_all;
                t_rounds = rounds * (all > t_cu ? all : t_cu);
            }
            double t = slices[i].nk * t_rounds + rounds * (eight ? kPipeFill8 : kPipeFill);
            if (kind == GEMM_DMA_128x256 && !store_only) t += (rounds - 1) * kNextRound128x256;
            const double stream = (operands + s * product) * kPerStream, work = t;
            if (stream > t) t = stream;
            t += kLaunch;
            if (s > 1) t += (s - (slices_go_to == SLICES_LAUNCH ? 0 : 1)) * product * kPerReduce + kReduceFixed;
            // level where only the stream counts: of two 8-wavefront tiles the one with less work (padding)
            if (p.kind < 0 || t < best || (t == best && eight && kPingPong[p.kind].full > 0.0 && work < best_work)) {
                best = t;
                best_work = work;
                p.kind = kind;
                p.split_k = s;
            }
        }
    }
    // One row of tiles of 256 rows, inside a step: the kernels of gemm_stream.h, by the same model with a time per K tile and a
    // fixed part of their own. Fitted to 162 launches with their consumers (129 to 256 rows, 18 layer shapes of 1024 to 37888
    // columns, cold weights): the choice loses 0.4 % on average and 6 % at worst against the best of either, and gains 3.6 %
    // over the plan without them: 7-20 % where the tiles make whole rounds of a long K (24576 x 4096, 22016 x 4096,
    // 3584 x 18944, 4096 x 12288), nothing where K is short (4096 x 4096: 1.06-1.11 of the time) or the rounds do not fit
    // (37888 x 3584: 1.13-1.21). Over 93 launches of 30 layer shapes whose plan they change, against that plan: 0.88 of the time, 0.99
    // at worst; with only half of the bound's rows live 0.93, 1.12 at worst (8192 x 8192). dkv_gemm on its own does not get them: it
    // goes through dkv_gemm_with, which takes the public kernel numbers, and no launch of its own was measured. With up to 128 rows the 128-row tiles are level (24576 x 4096 at 128 rows 43.3 against 51.6 us).
    if ((slices_go_to == SLICES_CONSUMER || slices_go_to == SLICES_PRODUCT) && m_upper > 128 && m_upper <= 256) {
        struct Stream { int kind, bn; double alone, full; };                                    // us per K tile
        constexpr Stream kStream[] = {{GEMM_STREAM_256x96, 96, 0.52, 0.56}, {GEMM_STREAM_256x64, 64, 0.44, 0.44}};
        constexpr double kPipeFillStream = 6.5;
        for (const Stream &st : kStream) {
            const int tiles = ceil_div(n, st.bn);
            for (int i = 0; i < n_slices && (i == 0 || tiles <= 768); ++i) {
                const int s = slices[i].s;
                const long wgs = (long)tiles * s, rounds = (wgs + 255) / 256;
                const double last = st.full * (double)(wgs - (rounds - 1) * 256) * (1.0 / 256.0);
                double t = slices[i].nk * ((rounds - 1) * st.full + (last > st.alone ? last : st.alone)) + rounds * kPipeFillStream;
                const double stream = (operands + s * product) * kPerStream;
                if (stream > t) t = stream;
                t += kLaunch;
                if (s > 1) t += (s - 1) * product * kPerReduce + kReduceFixed;
                if (t < best) {
                    best = t;
                    p.kind = st.kind;
                    p.split_k = s;
                }
            }
        }
        if (dkv_gemm_is_stream(p.kind)) return p;
    }
    // Launch options, from the same sweeps: a staggered K start pays when there is one row of tiles
    // (all workgroups of a K slice would otherwise read the same A columns at once), and with two or three rows of tiles
    // and several rounds of workgroups where the rows are a multiple of 4 KB apart, so that equal columns sit in the same
    // memory channels (14 % less time at K = 4096 over 1000 workgroups, none at K = 3584 or with one round); weights that
    // are read once (one row of tiles) are streamed with the non-temporal hint by the 4-wavefront tiles (in the 8-wavefront
    // loop, which has no such loads, the hint measured 0-13 % slower with K slices and between 5 % faster and 4 % slower
    // without); the XCD-grouped order
    // pays once there are enough tile rows to form groups, for the largest tiles everywhere, for every tile on wide
    // products. With it against without, 400 to 2048 rows: 128x128 1.0-1.08 of the time at 8192 columns, 0.95-1.03 at 12288
    // and 16384, 0.89-0.98 at 20480 and 24576, 0.83-0.91 at 32768; 128x256 0.96-1.03 from 12288 to 20480, 0.94-1.0 at 24576,
    // 0.92-0.99 at 32768; 128x192 0.85-1.0 except at 12288 (1.0-1.06) and 24576 (0.97-1.04). Between 12288 and 24576 columns
    // the tiles planned with four rows and more are 128x256 and the 8-wavefront ones, so the line costs nothing there; below
    // 12288 it leaves out 128x192 tiles, which would gain.
    const int tiles_m = ceil_div(m_upper, kKinds[p.kind].bm);
    const long wgs = (long)tiles_m * ceil_div(n, kKinds[p.kind].bn) * p.split_k;
    if (tiles_m == 1 || (tiles_m <= 3 && p.split_k == 1 && wgs > 512 && k % 2048 == 0)) p.flags |= GEMM_FLAG_STAGGER;
    // (not for matrices small enough to stay in the 256 MB last-level cache from one step to the next)
    if (tiles_m == 1 && kPingPong[p.kind].full == 0.0 && (size_t)n * k * 2 >= ((size_t)32 << 20)) p.flags |= GEMM_FLAG_STREAM_W;
    if (tiles_m >= 4 && (n >= 24576 || p.kind == GEMM_DMA_256x256 || p.kind == GEMM_DMA_256x192 || p.kind == GEMM_DMA_192x256 ||
                         (p.kind == GEMM_DMA_128x256 && tiles_m >= 6)))
        p.flags |= GEMM_FLAG_XCD_GROUP;
    // Giving 256 workgroups 3/4 of a tile's K range each (frac_units, kept for experiments through
    // dkv_gemm_with) was measured to take the same time as two full slices, so it is never planned.
    return p;
}

bool dkv_gemm_can_fuse_swiglu(int dtype, int n, int k, const GemmPlan &p) {
    return dtype == DKV_BF16 && (p.kind <= GEMM_DMA_LAST || dkv_gemm_is_stream(p.kind)) && p.split_k == 1 && p.frac_units == 0 &&
           (k % BK) == 0 && (n & 1) == 0;
}

int dkv_gemm_plan_valid(int dtype, int k, GemmPlan p) {
    if (p.split_k < 1 || p.kind < 0 || (p.kind >= GEMM_KINDS && !dkv_gemm_is_stream(p.kind)) || p.frac_units < 0) return 0;
    if (p.frac_units) {
        // a 3/4 share: every tile is covered by exactly two workgroups
        if (p.kind > GEMM_DMA_LAST || dtype != DKV_BF16 || (k % BK) != 0) return 0;
        return p.split_k == 2 && (k / BK) % 4 == 0 && p.frac_units == (k / BK) * 3 / 4;
    }
    if (p.kind == GEMM_SIMT) return p.split_k == 1;
    if (dtype != DKV_BF16 || (k % 8) != 0) return 0;
    if (p.kind != GEMM_REG_64x128 && (k % BK) != 0) return 0;
    return effective_split(k, p.split_k) == p.split_k;
}

bool dkv_gemm_can_fuse_head(int dtype, int k, const GemmPlan &p) {
    return dtype == DKV_BF16 && p.kind >= 0 && p.kind <= GEMM_DMA_LAST && p.split_k == 1 && p.frac_units == 0 &&
           (k % BK) == 0;
}

int dkv_gemm_tiles_n(const GemmPlan &p, int n) {
    return p.kind >= 0 && p.kind <= GEMM_DMA_LAST ? ceil_div(n, kKinds[p.kind].bn) : 0;
}

int dkv_launch_gemm_head(const void *A, const void *W, int m_upper, const int *m_dev, int n, int k, GemmPlan p,
                         const GemmEpilogue &ep, hipStream_t stream) {
    if (m_upper <= 0) return DKV_OK;
    if (ep.kind != EPI_HEAD || !dkv_gemm_can_fuse_head(DKV_BF16, k, p) || !dkv_gemm_plan_valid(DKV_BF16, k, p)) {
        dkv_set_error("projection plan (kind %d, split %d) cannot run the vocabulary epilogue at K %d", p.kind, p.split_k, k);
        return DKV_E_UNSUPPORTED;
    }
    p.flags &= ~GEMM_FLAG_SWIGLU;
    return dkv_dispatch_dma_head(A, W, nullptr, m_upper, m_upper, m_dev, n, k, p, ep, stream);
}

int dkv_launch_gemm(int dtype, const void *A, const void *W, float *partial, int m_upper, int m_cap,
                    const int *m_dev, int n, int k, GemmPlan p, hipStream_t stream) {
    if (m_upper <= 0) return DKV_OK;
    if (!dkv_gemm_plan_valid(dtype, k, p)) {
        dkv_set_error("projection plan (kind %d, split %d) does not fit dtype %d, K %d", p.kind, p.split_k, dtype, k);
        return DKV_E_UNSUPPORTED;
    }
    if (p.kind <= GEMM_DMA_LAST || dkv_gemm_is_stream(p.kind)) {
        GemmEpilogue ep;
        if (p.flags & GEMM_FLAG_SWIGLU) {
            if (p.split_k != 1 || p.frac_units) {
                dkv_set_error("the fused SwiGLU epilogue of a plain launch needs one K slice");
                return DKV_E_INVALID_ARG;
            }
            ep.kind = EPI_SWIGLU;
            ep.out = partial;
            return dkv_dispatch_dma_swiglu(A, W, partial, m_upper, m_cap, m_dev, n, k, p, ep, stream);
        }
        return dkv_dispatch_dma_store(A, W, partial, m_upper, m_cap, m_dev, n, k, p, ep, stream);
    }
    switch (p.kind) {
        case GEMM_REG_64x128: {
            const int kt_total = ceil_div(k, BK), kps = ceil_div(kt_total, p.split_k);
            dim3 grid(ceil_div(n, 128), ceil_div(m_upper, 64), p.split_k);
            hipLaunchKernelGGL(gemm_reg, grid, dim3(256), 0, stream, (const bf16_t *)A, (const bf16_t *)W, partial,
                               m_upper, m_cap, m_dev, n, k, kps);
            break;
        }
        default: {
            if (dkv_gemm_f32_few_rows(dtype, m_upper, n, k))
                return dkv_launch_gemm_f32_few_rows((const float *)A, (const float *)W, partial, m_upper, m_dev, n, k, false,
                                                    stream);
            dim3 grid(ceil_div(n, 64), ceil_div(m_upper, 64), 1);
            if (dtype == DKV_BF16)
                hipLaunchKernelGGL((gemm_simt<bf16_t>), grid, dim3(256), 0, stream, (const bf16_t *)A,
                                   (const bf16_t *)W, partial, m_upper, m_dev, n, k);
            else
                hipLaunchKernelGGL((gemm_simt<float>), grid, dim3(256), 0, stream, (const float *)A,
                                   (const float *)W, partial, m_upper, m_dev, n, k);
        }
    }
    DKV_LAUNCH_CHECK();
    return DKV_OK;
}

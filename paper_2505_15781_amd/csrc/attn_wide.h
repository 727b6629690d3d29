// Attention kernel for active sets of hundreds of query rows: 32 query rows per wavefront, 32x32x16 MFMA, head_dim 128.
// Included by attention.hip (uses its helpers).
//
// Work item = (sequence, kv head, block of 128 query rows). Keys stream in tiles of 64 through two LDS stages that the
// memory system fills directly (global_load_lds: no staging registers, no LDS stores); each of the four wavefronts
// multiplies its 32 query rows against the shared tile, so a K or V fragment read from LDS feeds 32 queries.
//
// Why: with 16-row tiles the loop was a chain product -> softmax -> product in every wavefront, and the two wavefronts of a
// SIMD did the same part at the same time: matrix pipes busy 33 %, vector issue 48 %, their sum and little overlap (here 45
// and 53 %). Here
// a wavefront works on half tiles of 32 keys in a skewed order: one stretch holds the scores of half tile j + 1, the output
// products of half tile j - 1 and the exponentials of half tile j, which do not depend on each other, and the schedule
// deals them out one MFMA, one or two LDS reads, three vector instructions at a time. The running sum is a product with a
// row of ones (v_dot2 costs 11 cycles each next to MFMAs, unpacking and adding on the vector units 2 % of the time). Two
// workgroups share a compute unit and cover each other's barrier (one per tile).
// Per call, with the scatter launch, before and after (same card): 8 sequences x 32 heads x 1024 keys, 512 rows 127.4 ->
// 119.0 us; 4 x 32 heads x 1536 keys, 1536 rows 231 -> 218 us; 16 x 4 kv heads of 7, 768 keys, up to 129 rows 41.5 -> 35.3
// us. What bounds it: the energy of its instructions. Over a launch of 1.1 ms (4 x 32 heads, 4096 keys and rows) the chip holds 1.92
// GHz of its 2.4, with the matrix pipes busy 57 % and vector issue 56 % of those cycles and 18 % of the wavefronts' time
// waiting; the 512-row launch takes 83 us alone and 89-94 behind others of its kind. So neither port is full, and schedules that
// only move instructions gain nothing; fewer instructions do: of 278 vector ones per wavefront and tile, next to 37 MFMAs, 105
// rescale the output, which some query of the 32 needs at 26 of 32 half tiles (independent scores). A reference that lags the
// maximum by up to 2^8 saves those (8-14 % less time), but then the largest probability is no longer exactly 1 and the error
// against float64 grows by up to 10 %: not done.
#pragma once

typedef __attribute__((address_space(3))) void *lds_ptr_t;
template <int V> struct StageC { static constexpr int value = V; };

// LDS rows of 256 bytes (one key); the 16-byte chunk c of row r sits in place c ^ wide_swizzle(r): 16 consecutive rows put
// a chunk into 16 different places (score operands: one chunk of 32 rows), and 4 consecutive rows put a 64-byte group into
// 4 different groups (transposing reads: 32 bytes of 4 rows each).
__device__ __forceinline__ int wide_swizzle(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }

// Work item of this workgroup in launches of 257 to 511 workgroups, where some compute units get two: as attn_item, but the
// blocks that hold query rows come first. A workgroup without rows leaves at once, and where it stood between others the
// hardware put two busy workgroups on one unit and left others empty (11 sequences x 8 kv heads of 3, 10 to 115 rows: 1024
// keys 35.9 -> 27.3 us, 4096 keys 113 -> 82; with no such sequences level to 1 % slower). With at most 256 workgroups every one
// has a unit; from 512 on, where the first two of every unit may be empty as well, the plain order is kept (the other one is not
// measured there). A lane per (sequence, kv head) pair of the XCD counts its blocks; a prefix sum
// over the lanes finds the pair of this workgroup.
__device__ __forceinline__ bool wide_item_compact(const int *row_off, int pairs, int Hkv, int G, int q_blocks, int &pair, int &qb) {
    const int lane = threadIdx.x & 63, slot = blockIdx.x >> 3, p = lane * 8 + (blockIdx.x & 7), b = min(p, pairs - 1) / Hkv;
    const int n = p < pairs ? min(((row_off[b + 1] - row_off[b]) * G + 127) / 128, q_blocks) : 0;
    int upto = n;                                  // inclusive prefix sum: within rows of 16 lanes, then across the rows
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x111, 0xf, 0xf, true);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x112, 0xf, 0xf, true);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x114, 0xf, 0xf, true);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x118, 0xf, 0xf, true);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x142, 0xa, 0xf, false);
    upto += __builtin_amdgcn_update_dpp(0, upto, 0x143, 0xc, 0xf, false);
    const unsigned long long behind = __builtin_amdgcn_ballot_w64(upto > slot);
    if (!behind) return false;
    const int at = __builtin_ctzll(behind);
    pair = at * 8 + (blockIdx.x & 7);
    qb = slot - (__builtin_amdgcn_readlane(upto, at) - __builtin_amdgcn_readlane(n, at));
    return true;
}

constexpr int WIDE_LDS_BYTES = 4 * 64 * 256;         // K0 K1 V0 V1

__global__ __launch_bounds__(256, 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bf16_wide(
    const bf16_t *__restrict__ Q, const bf16_t *__restrict__ Kc, const bf16_t *__restrict__ Vc,
    const int *__restrict__ row_off, bf16_t *__restrict__ out, int batch, int Hq, int Hkv, int L, int q_blocks,
    int rows_cap, float scale_log2e) {
    constexpr int NW = 4, DH = 128, ROW = DH * 2, KT2 = 64, TILE = KT2 * ROW;     // bytes of a row, of a K or V tile
    constexpr int DI = KT2 / (4 * NW);                          // DMA instructions (4 rows each) per wavefront and tile
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = Hq / Hkv, n_tiles = (L + KT2 - 1) / KT2;
    const int qi = lane & 31, g = lane >> 5, l16 = lane & 15, l4 = lane >> 4;
    const uint32_t lds_base = (uint32_t)(size_t)(lds_ptr_t)smem_raw;
    int pair, qb;
    if (gridDim.x > 256 && gridDim.x < 512) {          // at most 64 pairs on an XCD
        if (!wide_item_compact(row_off, batch * Hkv, Hkv, G, q_blocks, pair, qb)) return;
    } else if (!attn_item(blockIdx.x, batch * Hkv, q_blocks, pair, qb)) {
        return;
    }
    const int kvh = pair % Hkv, b = pair / Hkv;
    const int r0 = row_off[b], nq = (row_off[b + 1] - r0) * G, mb0 = qb * NW * 32;
    if (mb0 >= nq) return;                       // uniform for the workgroup

    // DMA: instruction i of a wavefront fills rows 4 (i NW + wave) + [0, 4) of a tile; lane -> row lane / 16, place lane % 16.
    // Keys past the end are clamped to the last one: their scores are masked, their probabilities zero.
    const char *Kb = reinterpret_cast<const char *>(Kc + (size_t)pair * (size_t)L * DH);
    const char *Vb = reinterpret_cast<const char *>(Vc + (size_t)pair * (size_t)L * DH);
    uint32_t chunk[DI];
#pragma unroll
    for (int i = 0; i < DI; ++i) chunk[i] = (l16 ^ wide_swizzle(4 * (i * NW + wave) + l4)) << 4;
    auto fill = [&](const char *base, int t, uint32_t dst) {
#pragma unroll
        for (int i = 0; i < DI; ++i) {
            const int row = 4 * (i * NW + wave) + l4;
            dma16_at((uint32_t)min(row, L - 1 - t * KT2) * ROW + chunk[i], base + (size_t)t * TILE,
                       lds_base + dst + 4 * (i * NW + wave) * ROW);
        }
    };
    // this lane's query row; rows beyond the host's bound have no slot in Q and out
    const int mq = mb0 + wave * 32 + qi;
    const bool q_ok = mq < nq && r0 + mq / G < rows_cap;
    const size_t q_at = q_ok ? ((size_t)(r0 + mq / G) * Hq + kvh * G + mq % G) * DH : (size_t)(kvh * G) * DH;
    bf16x8 qf[DH / 16];
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(Q + q_at + 8 * g + 16 * ks);
    fill(Kb, 0, 0);
    fill(Vb, 0, 2 * TILE);
    if (n_tiles > 1) fill(Kb, 1, TILE);

    // score operands: row lane & 31, chunk 2 ks + g
    const unsigned char *krow = smem_raw + qi * ROW;
    const int kx = (g ^ wide_swizzle(qi)) << 4;
    // output operand: see vt_operand; block lane / 16 = (g, dims + 16 half), key 4 g + j / 4 (+ 8), dims 4 (j % 4)
    const unsigned char *vrow = smem_raw + 2 * TILE + (4 * g + (l16 >> 2)) * ROW + ((l16 & 1) << 3);
    const int vx = ((2 * (l4 & 1) + ((l16 & 3) >> 1)) ^ (((l16 >> 2) << 2) | g)) << 4;       // keys + 8: swizzle ^ 2

    // lowest finite start: scores of -inf then give probabilities of zero, also where a whole half tile is masked
    float m_run = -3.0e38f, alpha = 1.f;
    bool behind = false;
    // sum of exactly the rounded probabilities of the second product: a product with a tile whose row 0 is ones; element 0
    // of the lanes below 32 is the sum of query qi, everything else stays zero
    f32x16 l_acc;
    bf16x8 ones;
#pragma unroll
    for (int v = 0; v < 16; ++v) l_acc[v] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = qi == 0 ? (__bf16)1.0f : (__bf16)0.0f;
    f32x16 acc[DH / 32], stA, stB;               // stA, stB: scores of the first and the second 32 keys of a tile
    bf16x8 pA[2], pB[2];                         // their probabilities
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) pB[0][e] = pB[1][e] = (__bf16)0.f;

    auto k_operand = [&](int ks, int stage, int half) {
        return *reinterpret_cast<const bf16x8 *>(krow + (kx ^ (ks << 5)) + stage * TILE + half * 32 * ROW);
    };
    // keys of k step ks in operand order: 16 ks + 4 g + {0..3}, 16 ks + 8 + 4 g + {0..3}: as the scores leave the MFMA
    auto v_operand = [&](int mt, int ks, int stage, int half) {
        const unsigned char *p = vrow + stage * TILE + (2 * half + ks) * 16 * ROW;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + (vx ^ (mt << 6))));
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + 8 * ROW + (vx ^ (mt << 6) ^ 32)));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    // One stretch: scores of a half tile (into sn), output products of the half tile before the last (pv), exponentials of
    // the last one (so -> pn). The three are independent of each other.
    auto stretch = [&](f32x16 &sn, int kstage, int khalf, const bf16x8 (&pv)[2], int vstage, int vhalf, const f32x16 &so,
                       bf16x8 (&pn)[2]) {
#pragma unroll
        for (int v = 0; v < 16; ++v) sn[v] = 0.f;
        f32x8 p[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) l_acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, pv[ks], l_acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(i, kstage, khalf), qf[i], sn, 0, 0, 0);
            acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(i & 3, i >> 2, vstage, vhalf), pv[i >> 2], acc[i & 3], 0, 0, 0);
#pragma unroll
            for (int e = 2 * i; e < 2 * i + 2; ++e)
                p[e >> 3][e & 7] = __builtin_amdgcn_exp2f(fmaf(so[e], scale_log2e, -m_run));
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) pn[ks] = __builtin_convertvector(p[ks], bf16x8);
        asm volatile("" : "+v"(pn[0]), "+v"(pn[1]));        // here, not behind the branches of maximum()
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);
        }
    };
    // Brings the output up to the reference m_run of the exponentials.
    auto rescale = [&]() {
        if (!behind) return;
#pragma unroll
        for (int mt = 0; mt < DH / 32; ++mt) acc[mt] *= alpha;
        l_acc[0] *= alpha;
    };
    // Maximum of the half tile whose first key is `key`. The running maximum is the reference of the exponentials, so that
    // the largest probability is exactly 1. The probabilities of the half tile before still wait for their product: the
    // output is rescaled to the new reference only behind that product, at the next call.
    auto maximum = [&](f32x16 &st, int key) {
        rescale();
        if (key + 32 > L) {                      // wave-uniform: only the last tile of a sequence has keys past the end
            const int left = L - key - 4 * g;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (8 * (v >> 2) + (v & 3) >= left) st[v] = -INFINITY;
        }
        float mx = st[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, st[v]);
        float u, w;
        swap_rows32(mx, u, w);
        mx = fmaxf(u, w) * scale_log2e;
        const float m_new = fmaxf(m_run, mx);
        behind = __builtin_amdgcn_ballot_w64(m_new > m_run) != 0;       // else the factor is exactly 1 for every query
        alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
    };
    auto tile_barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070);      // vmcnt(0), lgkmcnt(0): this wavefront's fills have landed, its LDS reads returned
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // the first stretch multiplies (zero) probabilities with the second half of V stage 1: no NaN may be there
    for (int i = tid; i < TILE / 32; i += 64 * NW) reinterpret_cast<uint4 *>(smem_raw + 3 * TILE + TILE / 2)[i] = make_uint4(0, 0, 0, 0);
    tile_barrier();
#pragma unroll
    for (int v = 0; v < 16; ++v) stA[v] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) stA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(i, 0, 0), qf[i], stA, 0, 0, 0);
    maximum(stA, 0);
    // Tile t, in stage S; the scores of its first half are formed.
    auto step = [&](int t, auto stage) {
        constexpr int S = decltype(stage)::value;
        stretch(stB, S, 1, pB, S ^ 1, 1, stA, pA);
        maximum(stB, t * KT2 + 32);
        // behind the barrier K(t + 1) and V(t) have landed for everybody, and everybody is done with K(t) and V(t - 1)
        tile_barrier();
        if (t + 2 < n_tiles) fill(Kb, t + 2, S * TILE);
        if (t + 1 < n_tiles) fill(Vb, t + 1, (2 + (S ^ 1)) * TILE);
        stretch(stA, S ^ 1, 0, pA, S, 0, stB, pB);            // behind the last tile: scores of an old tile, never used
        if (t + 1 < n_tiles) maximum(stA, (t + 1) * KT2);
    };
    for (int t = 0; t < n_tiles; t += 2) {
        step(t, StageC<0>{});
        if (t + 1 < n_tiles) step(t + 1, StageC<1>{});
    }
    const int last = (n_tiles - 1) & 1;
    rescale();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) l_acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, pB[ks], l_acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(i & 3, i >> 2, last, 1), pB[i >> 2], acc[i & 3], 0, 0, 0);

    float u, w;
    swap_rows32(l_acc[0], u, w);
    const float inv = 1.f / (u + w);
    if (!q_ok) return;
    bf16_t *op = out + q_at + 8 * g;
#pragma unroll
    for (int mt = 0; mt < DH / 32; ++mt)
#pragma unroll
        for (int c = 0; c < 4; c += 2) {
            // lane qi holds dims 8 c + {0..3} and 8 c + 8 + {0..3}, lane qi + 32 the other four of each: after the swaps the
            // first has the lower 8 dims, the second the upper 8
            uint32_t y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int v = 4 * c + (e >> 1) * 4 + (e & 1) * 2;
                y[e] = (uint32_t)f2bf(acc[mt][v] * inv) | ((uint32_t)f2bf(acc[mt][v + 1] * inv) << 16);
            }
            const auto p0 = __builtin_amdgcn_permlane32_swap(y[0], y[2], false, false);
            const auto p1 = __builtin_amdgcn_permlane32_swap(y[1], y[3], false, false);
            *reinterpret_cast<bf16x8_el *>(op + 32 * mt + 8 * c) = u32x4{p0[0], p1[0], p0[1], p1[1]};
        }
}

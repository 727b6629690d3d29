// Bidirectional attention of the active queries over the full-length, position-indexed K/V cache
// (Eq. 4: softmax(Q^{A_t} K^{I T} / sqrt(d)) V^I, no mask; query heads of one group share a K/V head).
//
// bf16 kernels (attn_ksplit.h, attn_shared.h, attn_wide.h): a "query row" is an (active row, query head of the
// group) pair, handled in tiles of 16 or 32. Keys stream in tiles through LDS (K rows and V rows as they are stored,
// the V operand through transposing reads), the next tiles are on their way while the current one is multiplied. Scores
// are formed transposed (keys x queries) so the probabilities come out of the MFMA already laid out as the
// operand of the second product and never leave registers; the output accumulates transposed
// (head_dim x queries) with a running max / sum per query (online softmax). The key-split kernel deals
// the key tiles to the wavefronts of a workgroup and merges their states in LDS; the other two
// give every wavefront its own query tile over one shared K/V tile. When the key-split kernel also slices the keys
// across workgroups every workgroup writes (max, sum, unnormalised output) and attn_merge combines them.
//
// generic kernel (fp32 mode and odd head sizes): one wavefront per (row, query head), lanes stride
// over the keys, fp32 FMA, exact expf.
#include <atomic>

#include "common.h"

namespace {

constexpr int KT = 32;                 // keys per tile

template <int DH> struct AttnSmem {
    static constexpr int K_STRIDE = DH * 2 + 16;        // bytes per K row (+16 spreads the 16-byte fragment reads)
    static constexpr int V_STRIDE = DH * 2 + 32;        // bytes per V row (+32 spreads the transposing reads)
    static constexpr int K_BYTES = KT * K_STRIDE;
    static constexpr int V_BYTES = KT * V_STRIDE;
    static constexpr int WAVE_BYTES = K_BYTES + V_BYTES;
};

typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((address_space(3))) bf16x4 *lds_bf16x4_ptr;

// MFMA operand V^T[dim 16 mt + (lane & 15)][8 keys] from V rows stored as they are in the cache (row = key).
// ds_read_b64_tr_b16 works on blocks of 16 lanes: lane j points at 4 consecutive 16-bit elements, and lane i
// receives element i % 4 of the pieces of lanes i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12. With lane j pointing
// at dims [16 mt + 4 (j % 4), +4) of key j / 4, lane i gets dim 16 mt + i of four consecutive keys. Two reads
// give the 8 keys of the lane's K group in the order the probabilities come out of the score MFMA:
// keys key0 + 4 g + {0..3} and key0 + 16 + 4 g + {0..3}, g = lane / 16. `vrow0` = address of (key 4 g + j / 4,
// dim 4 (j % 4)) of the tile, precomputed per lane.
__device__ __forceinline__ bf16x8 vt_operand(const unsigned char *vrow0, int mt, int v_stride, int key0) {
    const unsigned char *a = vrow0 + key0 * v_stride + mt * 32;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(a));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(a + 16 * v_stride));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Reductions over the four lanes that hold one query (lane, lane ^ 16, lane ^ 32, lane ^ 48), every lane getting the
// result: gfx950's row swaps (v_permlane16_swap exchanges the odd 16-lane rows of one register with the even rows of
// another, v_permlane32_swap the upper half of one with the lower half of another; applied to two copies of x they
// leave "my value" and "my partner's value" side by side). Two vector instructions per stage instead of an LDS
// round trip (ds_bpermute) with its index arithmetic, on the path between the two products of every key tile.
__device__ __forceinline__ void swap_rows16(float x, float &u, float &v) {
    const unsigned a = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    u = __builtin_bit_cast(float, r0);
    v = __builtin_bit_cast(float, r1);
}
__device__ __forceinline__ void swap_rows32(float x, float &u, float &v) {
    const unsigned a = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    u = __builtin_bit_cast(float, r0);
    v = __builtin_bit_cast(float, r1);
}
__device__ __forceinline__ float query_lanes_max(float x) {
    float u, v;
    swap_rows16(x, u, v);
    x = fmaxf(u, v);
    swap_rows32(x, u, v);
    return fmaxf(u, v);
}
__device__ __forceinline__ float query_lanes_sum(float x) {
    float u, v;
    swap_rows16(x, u, v);
    x = u + v;
    swap_rows32(x, u, v);
    return u + v;
}

// One online-softmax step of a lane over NT sub-tiles of 16 keys (Eq. 4's softmax, streamed): st[jt][i] is the raw
// score of key key_base + 16 jt + i against this lane's query. Updates the running max (log2 domain) and sum,
// rescales the output accumulators, and returns the probabilities as bf16 MFMA operands: operand hh covers
// sub-tiles 2hh and 2hh+1. The running sum is not formed here: the caller multiplies the same operands with a row of
// ones (row_sum_operand) into l_acc, so the matrix pipe adds up exactly the rounded probabilities that enter the
// second product and the vector units are spared sixteen additions per lane and tile; l_acc is only rescaled here.
template <int NT, int NACC>
__device__ __forceinline__ void softmax_step(f32x4 (&st)[NT], float &m_run, f32x4 &l_acc, f32x4 (&acc)[NACC],
                                             bf16x8 (&pb)[NT / 2], int key_base, int L, bool masked,
                                             float scale_log2e) {
    if (masked) {              // wave-uniform: only the last tile of a sequence has keys past the end
#pragma unroll
        for (int jt = 0; jt < NT; ++jt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (key_base + 16 * jt + i >= L) st[jt][i] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int jt = 0; jt < NT; ++jt)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, st[jt][i]);
    mx = query_lanes_max(mx);
    const float m_new = fmaxf(m_run, mx * scale_log2e);
    // Rescale only when some query of the wavefront got a new maximum (rare after the first tiles): for the
    // others the factor would be exactly 1.
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        l_acc *= alpha;
#pragma unroll
        for (int mt = 0; mt < NACC; ++mt) acc[mt] *= alpha;
        m_run = m_new;
    }
#pragma unroll
    for (int hh = 0; hh < NT / 2; ++hh) {
        f32x8 p;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            p[e] = __builtin_amdgcn_exp2f(fmaf(st[2 * hh + (e >> 2)][e & 3], scale_log2e, -m_new));
        pb[hh] = __builtin_convertvector(p, bf16x8);
    }
}

// First operand of the product that sums the probabilities of a query: a 16 x 32 tile whose row 0 is all ones (the
// lanes with lane % 16 == 0 hold that row). mfma(row_sum_operand, pb, l_acc) adds the sum over the 32 keys of pb to
// element 0 of l_acc in the lanes below 16 (row 0, column = query); everything else in l_acc stays zero, so the sum
// over a query's four lanes (query_lanes_sum of element 0) is the running sum.
__device__ __forceinline__ bf16x8 row_sum_operand(int lane) {
    const __bf16 one = (lane & 15) == 0 ? (__bf16)1.0f : (__bf16)0.0f;
    return bf16x8{one, one, one, one, one, one, one, one};
}

// 16 bytes with the non-temporal hint (data that this launch reads once)
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load16_nt(const void *p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Work-item order of the bf16 kernels. The `inner` workgroups of a (sequence, kv head) pair (query groups or blocks
// x key slices) read the same K/V rows, and the hardware sends workgroup i to XCD i mod 8, each with an L2 of its
// own: consecutive ids would have every XCD fetch the pair's K/V once more (measured: 4.2x the K/V bytes from
// memory with four query blocks per pair). So pair p lives on XCD p mod 8: its workgroups take the ids
// p mod 8 + 8 (inner (p / 8) + w), w < inner, which are dispatched within a few ids of each other. The grid is
// padded to a multiple of 8 pairs; returns false for the padding.
__device__ __forceinline__ bool attn_item(unsigned id, int pairs, int inner, int &pair, int &within) {
    const unsigned xcd = id & 7, slot = id >> 3;
    pair = (int)(slot / inner) * 8 + (int)xcd;
    within = (int)(slot % inner);
    return pair < pairs;
}
static inline unsigned attn_grid(long pairs, int inner) { return (unsigned)((pairs + 7) / 8 * 8 * inner); }

#include "attn_shared.h"
#include "attn_ksplit.h"
#include "attn_wide.h"

// Merge the key slices of one (row, head): one wavefront per pair.
template <int DH>
__global__ __launch_bounds__(256) void attn_merge(const float *__restrict__ part, bf16_t *__restrict__ out,
                                                  const int *__restrict__ row_off, int batch, int Hq,
                                                  int splits, int rows_cap) {
    const int lane = threadIdx.x & 63;
    const long pair = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const long n_pairs = (long)min(row_off[batch], rows_cap) * Hq;
    if (pair >= n_pairs) return;
    const float *rec = part + (size_t)pair * splits * (DH + 4);
    float M = -INFINITY;
    for (int s = 0; s < splits; ++s) M = fmaxf(M, rec[(size_t)s * (DH + 4)]);
    float lsum = 0.f;
    float o[DH / 64 > 0 ? DH / 64 : 1] = {};
    for (int s = 0; s < splits; ++s) {
        const float *r = rec + (size_t)s * (DH + 4);
        float w = exp2f(r[0] - M);
        lsum += w * r[1];
#pragma unroll
        for (int i = 0; i < (DH / 64 > 0 ? DH / 64 : 1); ++i) {
            int d = lane + 64 * i;
            if (d < DH) o[i] += w * r[4 + d];
        }
    }
    const float inv = 1.f / lsum;
#pragma unroll
    for (int i = 0; i < (DH / 64 > 0 ? DH / 64 : 1); ++i) {
        int d = lane + 64 * i;
        if (d < DH) out[(size_t)pair * DH + d] = f2bf(o[i] * inv);
    }
}

// Four consecutive elements as they are stored, and as floats.
__device__ __forceinline__ f32x4 raw4(const float *p) { return *reinterpret_cast<const f32x4_el *>(p); }
__device__ __forceinline__ u32x2 raw4(const bf16_t *p) { return *reinterpret_cast<const bf16x4_el *>(p); }
__device__ __forceinline__ f32x4 floats(f32x4 v) { return v; }
__device__ __forceinline__ f32x4 floats(u32x2 v) {
    return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                 __uint_as_float(v.y & 0xffff0000u)};
}
__device__ __forceinline__ void store4(float *p, f32x4 v) { *reinterpret_cast<f32x4_el *>(p) = v; }
__device__ __forceinline__ void store4(bf16_t *p, f32x4 v) {
    *reinterpret_cast<bf16x4_el *>(p) = u32x2{(uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16),
                                              (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16)};
}

// Generic kernel: one wavefront per (row, head), keys in chunks of 64. Scores and softmax state: a lane per key of the
// chunk, each with its own running maximum. Output: DH / 4 lanes per key with four dims each, so the V rows are read
// coalesced; a lane keeps one sum per key place that it serves, and only the last step adds those up and reduces over
// lanes (with a whole output vector per lane that was DH wavefront reductions: 64 rows x 4 heads x 64 keys of 32 floats,
// 11.1 -> 7 us). The sums run in the order of a butterfly over the 64 key places, as with one output vector per lane, so
// that candidates of nearly equal confidence keep their order. What bounds it at few rows is a memory latency per batch of
// loads and chunk: 2 sequences x 4 heads of 64 floats, 23 rows, 1300 keys 135 -> 64 us with whole batches in flight (92 with
// one output vector per lane), 8 x 16 heads of 128, 37 rows, 2500 keys 3008 -> 924 us (2292).
template <typename T, int DH>
__global__ __launch_bounds__(256) void attn_generic(const T *__restrict__ Q, const T *__restrict__ Kc,
                                                    const T *__restrict__ Vc,
                                                    const int *__restrict__ row_off, T *__restrict__ out,
                                                    int batch, int Hq, int Hkv, int L, int rows_cap,
                                                    float scale) {
    constexpr int LPK = DH / 4, KPP = 64 / LPK, NJ = 64 / KPP;      // lanes per key, keys per pass, passes per chunk
    __shared__ float2 state[4][64];                                 // (rescale, probability) of each key place
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long pair = (long)blockIdx.x * 4 + wave;
    const int total_rows = min(row_off[batch], rows_cap);
    if (pair >= (long)total_rows * Hq) return;
    const int row = (int)(pair / Hq), h = (int)(pair % Hq);
    int b = 0;
    while (row >= row_off[b + 1]) ++b;
    const int kvh = h / (Hq / Hkv);
    const T *qp = Q + (size_t)pair * DH;
    const T *Kb = Kc + ((size_t)b * Hkv + kvh) * (size_t)L * DH;
    const T *Vb = Vc + ((size_t)b * Hkv + kvh) * (size_t)L * DH;
    const int kk = lane / LPK, d = (lane % LPK) * 4;
    f32x4 o[NJ];                                                    // key places kk + KPP j
#pragma unroll
    for (int j = 0; j < NJ; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    auto share = [&](float2 x) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        state[wave][lane] = x;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // fp32 queries come through the scalar cache; bf16 ones, which may start at an odd element, stay in registers
    constexpr bool Q_REGS = sizeof(T) == 2;
    f32x4 qr[Q_REGS ? DH / 4 : 1];
    if constexpr (Q_REGS) {
#pragma unroll
        for (int i = 0; i < DH / 4; ++i) qr[i] = floats(raw4(qp + 4 * i));
    }
    // The loads of a batch of K pieces, and of V rows, are all issued before the first is used (left to itself, and behind a
    // branch for the last keys of a sequence, the compiler waited for one or two at a time).
    constexpr int KB = DH / 4 < 16 ? DH / 4 : 16, VB = DH == 128 ? 8 : NJ;
    for (int k0 = 0; k0 < L; k0 += 64) {
        const bool whole = k0 + 64 <= L;
        decltype(raw4(Kb)) vr[VB], kr[KB];
        auto load_v = [&](int j0) {
#pragma unroll
            for (int j = 0; j < VB; ++j) vr[j] = raw4(Vb + (size_t)min(k0 + KPP * (j0 + j) + kk, L - 1) * DH + d);
        };
        const T *kp = Kb + (size_t)min(k0 + lane, L - 1) * DH;
        float s = 0.f;
#pragma unroll
        for (int i0 = 0; i0 < DH / 4; i0 += KB) {
#pragma unroll
            for (int i = 0; i < KB; ++i) kr[i] = raw4(kp + 4 * (i0 + i));
            if (i0 + KB == DH / 4) load_v(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < KB; ++i) {
                const f32x4 q = Q_REGS ? qr[i0 + i] : floats(raw4(qp + 4 * (i0 + i))), k = floats(kr[i]);
#pragma unroll
                for (int v = 0; v < 4; ++v) s = fmaf(q[v], k[v], s);
            }
        }
        s *= scale;
        const float mn = fmaxf(m, s);
        const float a = expf(m - mn), p = expf(s - mn);
        if (k0 + lane < L) {
            l = l * a + p;
            m = mn;
        }
        share(make_float2(a, p));
#pragma unroll
        for (int j0 = 0; j0 < NJ; j0 += VB) {
            if (j0) {
                load_v(j0);
                __builtin_amdgcn_sched_barrier(0);
            }
            auto add = [&](int j) {
                const float2 ap = state[wave][KPP * (j0 + j) + kk];
                const f32x4 v = floats(vr[j]);
                f32x4 x;
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = fmaf(ap.y, v[i], o[j0 + j][i] * ap.x);
                return x;
            };
            if (whole) {
#pragma unroll
                for (int j = 0; j < VB; ++j) o[j0 + j] = add(j);
            } else {
#pragma unroll
                for (int j = 0; j < VB; ++j) {
                    const f32x4 x = add(j);
                    const bool use = k0 + KPP * (j0 + j) + kk < L;
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[j0 + j][i] = use ? x[i] : o[j0 + j][i];
                }
            }
        }
    }
    const float Mx = wave_max(m);
    const float w = (m == -INFINITY) ? 0.f : expf(m - Mx);
    const float lt = wave_sum(l * w), lt_other = __shfl_xor(lt, 32, 64);
    share(make_float2(w, 0.f));
    // The first step of a butterfly over lanes takes one product exactly and the other rounded: of places p and p + 32 the
    // lower one in the lanes below 32, the upper one in the others; so does that of the sum. The result of dim d comes from
    // lane d & 63, as it did when every lane held a whole output vector.
    const bool upper = d & 32;
    const float inv = 1.f / (upper ? lt_other : lt);
#pragma unroll
    for (int j = 0; j < NJ / 2; ++j) {
        const float wl = state[wave][KPP * j + kk].x, wu = state[wave][KPP * (j + NJ / 2) + kk].x;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float lo = o[j][i], up = o[j + NJ / 2][i];
            o[j][i] = fmaf(upper ? up : lo, upper ? wu : wl, (upper ? lo : up) * (upper ? wl : wu));
        }
    }
#pragma unroll
    for (int x = NJ / 4; x > 0; x >>= 1)
#pragma unroll
        for (int j = 0; j < x; ++j) o[j] += o[j + x];
    f32x4 y = o[0];
#pragma unroll
    for (int x = 32; x >= LPK; x >>= 1)
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] += __shfl_xor(y[i], x, 64);
    if (kk == 0) store4(out + (size_t)pair * DH + d, y * inv);
}

template <typename T>
int launch_generic(const void *q, const void *k, const void *v, const int *row_off, void *out, int batch,
                   int Hq, int Hkv, int L, int dh, int rows_upper, hipStream_t s) {
    long pairs = (long)rows_upper * Hq;
    dim3 grid((unsigned)((pairs + 3) / 4));
    float scale = 1.0f / sqrtf((float)dh);
#define GEN(D)                                                                                        \
    hipLaunchKernelGGL((attn_generic<T, D>), grid, dim3(256), 0, s, (const T *)q, (const T *)k,       \
                       (const T *)v, row_off, (T *)out, batch, Hq, Hkv, L, rows_upper, scale)
    if (dh == 32) GEN(32);
    else if (dh == 64) GEN(64);
    else if (dh == 128) GEN(128);
    else {
        dkv_set_error("head_dim %d not supported (32, 64, 128)", dh);
        return DKV_E_UNSUPPORTED;
    }
#undef GEN
    DKV_LAUNCH_CHECK();
    return DKV_OK;
}

}  // namespace

AttnPlan dkv_attn_plan(int dtype, int batch, int n_q_heads, int n_kv_heads, int seq_len, int head_dim,
                       int max_rows_per_seq) {
    return dkv_attn_plan_within(SIZE_MAX, dtype, batch, n_q_heads, n_kv_heads, seq_len, head_dim, max_rows_per_seq);
}

AttnPlan dkv_attn_plan_within(size_t partial_bytes, int dtype, int batch, int n_q_heads, int n_kv_heads, int seq_len, int head_dim,
                              int max_rows_per_seq) {
    AttnPlan p;
    p.use_mfma = (dtype == DKV_BF16 && (head_dim == 64 || head_dim == 128)) ? 1 : 0;
    p.shared = 0;
    p.wide = 0;
    p.q_blocks = 0;
    p.ksplit_nq = 0;
    p.ksplit_waves = 0;
    p.q_groups = 0;
    int G = n_q_heads / n_kv_heads;
    p.q_tiles = ceil_div(max_rows_per_seq * G, 16);
    if (p.q_tiles < 1) p.q_tiles = 1;
    if (!p.use_mfma) {
        p.splits = 1;
        p.tiles_per_split = ceil_div(seq_len, KT);
        return p;
    }
    // Blocks of 128 query rows that share K/V tiles (head_dim 128, more than four query tiles) from 192 workgroups on; below,
    // or with fewer rows, the key-split kernel: at 128 workgroups the two are within 5 % of each other (1 x 32 heads, 512
    // keys, 512 rows 19.7 against 19.9 us, 4 x 32 heads, 1024 keys, 128 rows 29.4 against 30.4), at 64 it is 9 % ahead.
    // Where a pair has one block and its K/V is long, the stream of K/V bounds the launch and attn_shared.h, with two
    // tiles on their way, is ahead of attn_wide.h: 8 x 32 heads, 128 rows, 1024 keys 40.3 against 43.0 us; 512 keys 25.4
    // against 24.8, and several blocks per pair (4 x 32 heads, 1024 keys, 256 rows) 38.6 against 36.2.
    const int blocks = ceil_div(p.q_tiles, 8);
    const long wgs = (long)batch * n_kv_heads * blocks;
    if (head_dim == 128 && p.q_tiles >= 5 && wgs >= 192) {
        // fewer than two workgroups per compute unit: 8 wavefronts
        p.shared = blocks > 1 || seq_len < 768 ? 0 : wgs < 512 ? 8 : 4;
        p.wide = !p.shared;
        p.q_blocks = blocks;
        p.splits = 1;
        p.tiles_per_split = ceil_div(seq_len, 64);
        return p;
    }
    // Key-split kernel: query tiles per item (one or two) and key slices by a small model of the fullest XCD. attn_item puts all
    // workgroups of a pair on XCD pair % 8, so an XCD has ceil(pairs / 8) pairs and 32 compute units for them, whatever the other
    // XCDs do. In steps of one key tile and one query tile of a wavefront (about 2 us with 128 dims, half of it with 64):
    //   a workgroup costs kFixed and the key tiles of a wavefront; a second query tile makes a step half as long again, but the
    //   items half as many;
    //   workgroups have 8 wavefronts, one on a compute unit, where all items of an XCD fit at once or keys are sliced, otherwise 4
    //   (0.88 of the time of 8 there, median of 347 plans); items of one tile go up to 64 of those (beyond, two tiles take 0.63-1.1 of the time);
    //   slices begin at 24 key tiles of 128 dims, leave two tiles to each wavefront beyond four slices, may run in up to four rounds of
    //   32 workgroups (kRound for each further one: where the keys are many, rounds of short chains beat one of long chains
    //   that leaves units idle; 3 % where a round takes every unit), and cost a merge launch that reads them all.
    // Fitted to 1991 calls (1 to 24 sequences, 1 to 64 K/V heads, 40 to 20000 keys, head_dim 64 and 128; up to 30 plans of each
    // measured, K/V cold): the choice loses 1.2 % on average and 23 % at worst against the best, and takes 0.87 of the time of two tiles
    // always with slices up to 384 workgroups (1.17 at worst), 0.94 of that of lines at numbers of items and key tiles (1.10 at worst);
    // over 700 other calls 0.86 (1.11) and 0.95 (1.16).
    // Those lost where keys are many, which slices of two-tile items then share: 36 pairs, 16384 keys, 64 rows 76.5 us
    // with two tiles in three slices, 135 with one in one; 8192 keys 45 and 70; 8 pairs of 7 query heads, 8192 keys, 48 rows 41 and 57;
    // and on few pairs, where two tiles were taken beyond 1024 keys: 4 pairs of 7 query heads, 1536 keys, 20 rows 12.5 us with one
    // tile in three slices, 14.5 with two; 64 rows 16.6 with one in one, 24.5 with two in three.
    const long pairs = (long)batch * n_kv_heads;
    const long per_xcd = (pairs + 7) / 8;
    const int n_tiles = ceil_div(seq_len, KT);
    constexpr float kFixed = 4.0f, kTwoTiles = 1.56f, kFourWaves = 0.89f, kRound = 5.5f, kMerge = 0.9f, kMergeSlice = 0.36f,
                    kFull = 1.035f;
    const float keys = (head_dim == 64 ? 0.5f : 1.0f) * (float)n_tiles;
    const int most_slices = n_tiles * head_dim < 24 * 128 ? 1 : n_tiles / 16 > 4 ? n_tiles / 16 : 4;
    const size_t slice_bytes = (size_t)batch * ceil_div(p.q_tiles * 16, G) * n_q_heads * (head_dim + 4) * sizeof(float);
    const size_t fit = partial_bytes / slice_bytes;
    float best = 0.f;
    int s = 1;
    for (int nq = 1; nq <= 2 && nq <= p.q_tiles; ++nq) {
        const int groups = ceil_div(p.q_tiles, nq);
        const long items = per_xcd * groups;
        if (nq == 1 && items > 64 && p.q_tiles > 1) continue;
        const float chain = (nq == 2 ? kTwoTiles : 1.0f) * keys;
        for (int slices = 1; slices == 1 || (slices <= most_slices && slices * items <= 128 && (size_t)slices <= fit); ++slices) {
            const int waves = items > 32 && slices == 1 ? 4 : 8;
            const float rounds = waves == 8 ? (float)((slices * items + 31) / 32) : kFourWaves;
            float t = kFixed + rounds * chain / (float)(slices * waves) + (rounds > 1.0f ? (rounds - 1.0f) * kRound : 0.0f);
            if (slices > 1) t += kMerge + kMergeSlice * (float)slices;
            if (slices > 1 && slices * items % 32 == 0) t *= kFull;
            if (best == 0.f || t < best) {
                best = t;
                s = slices;
                p.ksplit_nq = nq;
                p.q_groups = groups;
                p.ksplit_waves = waves;
            }
        }
    }
    p.tiles_per_split = ceil_div(n_tiles, s);
    p.splits = ceil_div(n_tiles, p.tiles_per_split);
    return p;
}

size_t dkv_attn_partial_bytes(const AttnPlan &p, int batch, int n_q_heads, int n_kv_heads, int head_dim) {
    if (!p.use_mfma || p.splits == 1) return 0;
    int G = n_q_heads / n_kv_heads;
    // rows per sequence are at most q_tiles*16/G (rounded up); records are indexed by (row, head, split)
    size_t rows = (size_t)batch * (size_t)ceil_div(p.q_tiles * 16, G);
    return rows * n_q_heads * p.splits * (size_t)(head_dim + 4) * sizeof(float);
}

int dkv_attn_can_fuse_update(const AttnPlan &plan, int max_rows_per_seq) {
    return plan.use_mfma && plan.ksplit_nq > 0 && max_rows_per_seq <= 64;
}

int dkv_launch_attention(int dtype, const void *q, void *k_cache, void *v_cache, const int *row_off, void *out,
                         int batch, int n_q_heads, int n_kv_heads, int seq_len, int head_dim, int rows_upper,
                         AttnPlan plan, void *partial, AttnFusedUpdate fuse, hipStream_t stream) {
    if (rows_upper <= 0) return DKV_OK;
    if (fuse.k_new && !plan.ksplit_nq) {
        dkv_set_error("the cache update can only be fused into the key-split attention kernel");
        return DKV_E_INVALID_ARG;
    }
    if (!plan.use_mfma) {
        if (dtype == DKV_BF16)
            return launch_generic<bf16_t>(q, k_cache, v_cache, row_off, out, batch, n_q_heads, n_kv_heads,
                                          seq_len, head_dim, rows_upper, stream);
        return launch_generic<float>(q, k_cache, v_cache, row_off, out, batch, n_q_heads, n_kv_heads,
                                     seq_len, head_dim, rows_upper, stream);
    }
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)head_dim);
    long pairs = (long)rows_upper * n_q_heads;
    if (plan.ksplit_nq) {
        const unsigned wgs = attn_grid((long)batch * n_kv_heads, plan.q_groups * plan.splits);
#define KSPLIT_F(D, NQ, NW, F)                                                                                 \
    do {                                                                                                       \
        static std::atomic<bool> lds_ok{false};    /* idempotent call: racing threads only repeat it */       \
        const size_t smem = NW * AttnSmem<D>::WAVE_BYTES;                                                      \
        if (!lds_ok.load(std::memory_order_acquire)) {                                                         \
            DKV_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_bf16_ksplit<D, NQ, NW, F>),   \
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));           \
            lds_ok.store(true, std::memory_order_release);                                                     \
        }                                                                                                      \
        hipLaunchKernelGGL((attn_bf16_ksplit<D, NQ, NW, F>), dim3(wgs), dim3(64 * NW), smem, stream,           \
                           (const bf16_t *)q, (bf16_t *)k_cache, (bf16_t *)v_cache, row_off, (bf16_t *)out,    \
                           (float *)partial, batch, n_q_heads, n_kv_heads, seq_len, plan.q_groups,             \
                           plan.splits, plan.tiles_per_split, rows_upper, scale_log2e,                         \
                           (const bf16_t *)fuse.k_new, (const bf16_t *)fuse.v_new, fuse.active_idx);           \
    } while (0)
#define KSPLIT(D, NQ, NW)                                                                                      \
    do {                                                                                                       \
        if (fuse.k_new) KSPLIT_F(D, NQ, NW, true);                                                             \
        else KSPLIT_F(D, NQ, NW, false);                                                                       \
    } while (0)
        if (head_dim == 128) {
            if (plan.ksplit_waves == 8) {
                if (plan.ksplit_nq == 2) KSPLIT(128, 2, 8);
                else KSPLIT(128, 1, 8);
            } else {
                if (plan.ksplit_nq == 2) KSPLIT(128, 2, 4);
                else KSPLIT(128, 1, 4);
            }
        } else {
            if (plan.ksplit_waves == 8) {
                if (plan.ksplit_nq == 2) KSPLIT(64, 2, 8);
                else KSPLIT(64, 1, 8);
            } else {
                if (plan.ksplit_nq == 2) KSPLIT(64, 2, 4);
                else KSPLIT(64, 1, 4);
            }
        }
#undef KSPLIT_F
#undef KSPLIT
        DKV_LAUNCH_CHECK();
        if (plan.splits > 1) {
            if (head_dim == 128)
                hipLaunchKernelGGL((attn_merge<128>), dim3((unsigned)((pairs + 3) / 4)), dim3(256), 0, stream,
                                   (const float *)partial, (bf16_t *)out, row_off, batch, n_q_heads, plan.splits,
                                   rows_upper);
            else
                hipLaunchKernelGGL((attn_merge<64>), dim3((unsigned)((pairs + 3) / 4)), dim3(256), 0, stream,
                                   (const float *)partial, (bf16_t *)out, row_off, batch, n_q_heads, plan.splits,
                                   rows_upper);
            DKV_LAUNCH_CHECK();
        }
    } else if (plan.wide) {
        static std::atomic<bool> lds_ok{false};
        if (!lds_ok.load(std::memory_order_acquire)) {
            DKV_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_bf16_wide),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, WIDE_LDS_BYTES));
            lds_ok.store(true, std::memory_order_release);
        }
        hipLaunchKernelGGL(attn_bf16_wide, dim3(attn_grid((long)batch * n_kv_heads, plan.q_blocks)), dim3(256),
                           WIDE_LDS_BYTES, stream, (const bf16_t *)q, (const bf16_t *)k_cache, (const bf16_t *)v_cache,
                           row_off, (bf16_t *)out, batch, n_q_heads, n_kv_heads, seq_len, plan.q_blocks, rows_upper,
                           scale_log2e);
        DKV_LAUNCH_CHECK();
    } else if (plan.shared) {
        constexpr size_t smem = 2 * 64 * ((128 * 2 + 16) + (128 * 2 + 32));   // two stages of 64 K rows and 64 V rows
        static std::atomic<bool> lds_ok{false};
        if (!lds_ok.load(std::memory_order_acquire)) {
            DKV_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_bf16_shared<1, 8>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
            DKV_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_bf16_shared<2, 4>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
            lds_ok.store(true, std::memory_order_release);
        }
#define SHARED(NQ_, NW_)                                                                                             \
    hipLaunchKernelGGL((attn_bf16_shared<NQ_, NW_>), dim3(attn_grid((long)batch * n_kv_heads, 1)), dim3(64 * NW_), smem, \
                       stream, (const bf16_t *)q, (const bf16_t *)k_cache, (const bf16_t *)v_cache, row_off,         \
                       (bf16_t *)out, batch, n_q_heads, n_kv_heads, seq_len, rows_upper, scale_log2e)
        if (plan.shared == 8) SHARED(1, 8);
        else SHARED(2, 4);
#undef SHARED
        DKV_LAUNCH_CHECK();
    }
    return DKV_OK;
}

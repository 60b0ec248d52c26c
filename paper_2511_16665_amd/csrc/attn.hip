// Tree-masked grouped-query attention over the paged KV cache.
//
// Every active row (b, i) of every query head attends to the seq_len[b] committed cache rows and to
// the provisional rows seq_len[b] + j whose bit j is set in the row's mask (ancestors-or-self of a
// tree node; a causal prefix for chains).
//
// impl 0 ("wave-per-row"): one workgroup of four wavefronts per (row, query head), each wave taking every fourth tile
//   of 64 keys; lanes own keys for the score pass and pieces of value rows for the value pass; online softmax across a wave's
//   tiles, the waves merged at the end.  Any dtype, any head_dim that is a multiple of 64 up to 256.  Used for fp32
//   mode and as a cross-check.  Bound by load latency: a key's elements are requested 64 together, values by rows spread
//   over the lanes, 16 rows of every lane group together (4 heads of 64, 130 keys: 40 us with one wave and 4-byte loads, one
//   after the other; 13.7 with four waves, 16-byte key loads and 16 keys' values at a time; 7.6 this way).
// impl 1 ("MFMA split-KV"): the bf16 / head_dim 128 production kernel, described further down.
#include <algorithm>

#include "dev_common.h"
#include "kernels.h"

namespace tlt {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;   // 16-byte register vector
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
constexpr int kRowWaves = 4;   // waves of impl 0's workgroup (64 * kRowWaves covers the largest head_dim)

__device__ __forceinline__ bool region_visible(const Rows& rows, int r, int i, int j) {
    if (j >= rows.n_region) return false;
    if (!rows.mask) return j <= i;
    uint64_t w = rows.mask[(int64_t)r * rows.mask_words + (j >> 6)];
    return (w >> (j & 63)) & 1ull;
}

// element e of a 16-byte piece
template <typename T>
__device__ __forceinline__ float element(u32x4_t v, int e) {
    if constexpr (sizeof(T) == 4) return __uint_as_float(v[e]);
    else return __uint_as_float((e & 1) ? v[e >> 1] & 0xffff0000u : v[e >> 1] << 16);
}

template <typename T>
__global__ __launch_bounds__(64 * kRowWaves) void attn_wave_per_row_k(Rows rows, KVLayer kv, const T* __restrict__ qkv,
                                                                      T* __restrict__ out, int n_q_heads, float scale) {
    typedef u32x4_t __attribute__((aligned(2))) piece_t;   // (a caller's pool may start at any element: one load all the same)
    constexpr int VEC = 16 / sizeof(T), kU = 16, kGroups = 64 * VEC / 64;   // (groups: at head_dim 64, the smallest)
    __shared__ __align__(16) float q_s[256], o_s[kRowWaves][kGroups][256];
    __shared__ float m_s[kRowWaves], l_s[kRowWaves], p_s[kRowWaves][64];
    __shared__ int64_t base_s[kRowWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x, hq = blockIdx.y, b = blockIdx.z;
    const int r = b * rows.n + i;
    const int d = kv.d;
    const int G = n_q_heads / kv.n_kv, kh = hq / G;
    const int qkv_dim = (n_q_heads + 2 * kv.n_kv) * d;
    T* o = out + ((int64_t)r * n_q_heads + hq) * d;
    if (rows.n_valid && i >= rows.n_valid[b]) {
        if ((int)threadIdx.x < d) o[threadIdx.x] = from_float<T>(0.f);
        return;
    }
    const int ctx = kv.seq_len[b];
    const int total = ctx + rows.n_region;
    if ((int)threadIdx.x < d) q_s[threadIdx.x] = to_float(qkv[(int64_t)r * qkv_dim + hq * d + threadIdx.x]) * scale;
    __syncthreads();
    const T* kc = (const T*)kv.k;
    const T* vc = (const T*)kv.v;
    // values: d / VEC lanes read a key's row in 16-byte pieces, so the wave's lanes hold `groups` keys at a time
    const int lpk = d / VEC, groups = 64 / lpk, grp = lane / lpk, piece = (lane - grp * lpk) * VEC;
    float m = -INFINITY, l = 0.f;
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
    for (int t0 = 64 * wave; t0 < total; t0 += 64 * kRowWaves) {
        const int key = t0 + lane;
        bool vis = key < total && (key < ctx || region_visible(rows, r, i, key - ctx));
        PageRef pr;
        int64_t base = -1;
        if (vis && locate(kv.block_table, kv.max_pages, kv.n_pages, kv.page_size, b, key, pr))
            base = ((pr.page * kv.n_kv + kh) * kv.page_size + pr.row) * d;
        vis = base >= 0;
        if (!vis) base = 0;   // (row 0 of the pool: its weight below is zero)
        float s = 0.f;
        const T* kp = kc + base;
        for (int c0 = 0; c0 < d; c0 += 64) {   // (a key's 64 elements requested together)
            u32x4_t kk[64 / VEC];
#pragma unroll
            for (int c = 0; c < 64 / VEC; ++c) kk[c] = *(const piece_t*)(kp + c0 + c * VEC);
#pragma unroll
            for (int c = 0; c < 64 / VEC; ++c)
#pragma unroll
                for (int e = 0; e < VEC; ++e) s = fmaf(q_s[c0 + c * VEC + e], element<T>(kk[c], e), s);
        }
        if (!vis) s = -INFINITY;
        const float m_new = fmaxf(m, wave_max(s));
        if (m_new == -INFINITY) continue;  // nothing visible so far (uniform across the wave)
        const float corr = expf(m - m_new);      // exp(-inf) = 0 on the first visible tile
        const float p = vis ? expf(s - m_new) : 0.f;
        l = l * corr + wave_sum(p);
        m = m_new;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] *= corr;
        p_s[wave][lane] = p;       // (read back by the same wave only)
        base_s[wave][lane] = base;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int nk = min(64, total - t0);
        for (int k0 = 0; k0 < nk; k0 += kU * groups) {   // (kU rows per lane in flight; keys past nk have weight zero and read row 0)
            u32x4_t vv[kU];
            float pk[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int k = k0 + u * groups + grp;
                const bool on = k < 64 && grp < groups;
                pk[u] = on ? p_s[wave][k] : 0.f;
                vv[u] = *(const piece_t*)(vc + (on ? base_s[wave][k] : 0) + (on ? piece : 0));
            }
#pragma unroll
            for (int u = 0; u < kU; ++u)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] = pk[u] != 0.f ? fmaf(pk[u], element<T>(vv[u], e), acc[e]) : acc[e];
        }
        __builtin_amdgcn_wave_barrier();
    }
    // the partial results, merged in wave and group order
    if (grp < groups)
#pragma unroll
        for (int e = 0; e < VEC; ++e) o_s[wave][grp][piece + e] = acc[e];
    if (lane == 0) {
        m_s[wave] = m;
        l_s[wave] = l;
    }
    __syncthreads();
    if ((int)threadIdx.x >= d) return;
    float mm = m_s[0];
#pragma unroll
    for (int w = 1; w < kRowWaves; ++w) mm = fmaxf(mm, m_s[w]);
    float ll = 0.f, a = 0.f;
#pragma unroll
    for (int w = 0; w < kRowWaves; ++w) {
        const float f = m_s[w] == -INFINITY ? 0.f : expf(m_s[w] - mm);
        ll += f * l_s[w];
        float o_w = 0.f;
        for (int g = 0; g < groups; ++g) o_w += o_s[w][g][threadIdx.x];
        a += f * o_w;
    }
    o[threadIdx.x] = from_float<T>(ll > 0.f ? a / ll : 0.f);
}

// impl 0 on rows that the projection has just left (fp32, few rows per sequence): the rotation and the write of the new keys and values, a kernel of
// their own otherwise, belong to this one.  Every workgroup rotates its query and its kv head's n new keys into LDS (n * d / 2 <= 256: an angle per
// thread) and takes the new rows from there; the first query head of each kv head also leaves row i's key and value in the cache, which
// nobody reads in this launch.  A tiny decoder's step is as long as its launches are many (2.4 us of the host each), and the chain of this one is two
// loads long: lengths, block table and projection together, then keys and values together.  Sums and their order are those of the two kernels.
__global__ __launch_bounds__(64 * kRowWaves) void attn_rope_rows_k(Rows rows, KVLayer kv, const float* __restrict__ qkv, float* __restrict__ out,
                                                                   int n_q_heads, float scale, const float* __restrict__ bias, float theta, RopeTable tab,
                                                                   bool from_table) {
    constexpr int VEC = 4, kU = 16;
    __shared__ __align__(16) float q_s[256], k_s[512 + 4 * 8], v_s[512], o_s[kRowWaves][4][256];
    __shared__ float m_s[kRowWaves], l_s[kRowWaves], p_s[kRowWaves][64];
    __shared__ const float* v_at[kRowWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x, hq = blockIdx.y, b = blockIdx.z, n = rows.n, r = b * n + i;
    const int d = kv.d, half = d >> 1, n_kv = kv.n_kv, G = n_q_heads / n_kv, kh = hq / G;
    const int qkv_dim = (n_q_heads + 2 * n_kv) * d;
    float* o = out + ((int64_t)r * n_q_heads + hq) * d;
    // everything that depends on no other load, requested together: the wave's first block-table entries among it
    const int ctx = kv.seq_len[b];
    const int nv = rows.n_valid ? rows.n_valid[b] : n;
    auto page_of = [&](int slot) {   // -1: no page
        const int lp = slot / kv.page_size;
        const int pg = slot >= 0 && lp < kv.max_pages ? kv.block_table[(int64_t)b * kv.max_pages + lp] : -1;
        return pg >= 0 && pg < kv.n_pages ? pg : -1;
    };
    const int pg_first = page_of(64 * wave + lane);
    const int j = (int)threadIdx.x / half, p = (int)threadIdx.x - j * half;   // this thread's new row and pair
    const bool on = j < n;
    float k_lo = 0.f, k_hi = 0.f, v_lo = 0.f, v_hi = 0.f, q_lo = 0.f, q_hi = 0.f;
    if (on) {
        const float* row = qkv + (int64_t)(b * n + j) * qkv_dim;
        const int ko = (n_q_heads + kh) * d + p, vo = (n_q_heads + n_kv + kh) * d + p, qo = hq * d + p;
        k_lo = row[ko], k_hi = row[ko + half], v_lo = row[vo], v_hi = row[vo + half];
        if (j == i) q_lo = row[qo], q_hi = row[qo + half];
        if (bias) {
            k_lo += bias[ko], k_hi += bias[ko + half], v_lo += bias[vo], v_hi += bias[vo + half];
            if (j == i) q_lo += bias[qo], q_hi += bias[qo + half];
        }
    }
    if (i >= nv) {   // (uniform: the row is not active)
        if ((int)threadIdx.x < d) o[threadIdx.x] = 0.f;
        return;
    }
    if (on) {
        float c, sn;
        const int64_t t = (int64_t)(b * n + j) * d + p;
        if (from_table) {
            c = tab.cs[t], sn = tab.cs[t + half];
        } else {
            const int pos = ctx + rows.pos_base + (rows.pos_off ? rows.pos_off[b * n + j] : rows.pos_stride * j);
            double s64, c64;
            sincos((double)pos * pow((double)theta, -2.0 * (double)p / (double)d), &s64, &c64);
            c = (float)c64, sn = (float)s64;
            if (tab.cs && hq == 0 && j == i) tab.cs[t] = c, tab.cs[t + half] = sn;
        }
        const float kl = k_lo * c - k_hi * sn, kr = k_hi * c + k_lo * sn;
        k_s[j * (d + 4) + p] = kl, k_s[j * (d + 4) + half + p] = kr;
        v_s[j * d + p] = v_lo, v_s[j * d + half + p] = v_hi;
        if (j == i) {
            q_s[p] = (q_lo * c - q_hi * sn) * scale, q_s[half + p] = (q_hi * c + q_lo * sn) * scale;
            if (hq == kh * G) {
                const int slot = ctx + rows.slot_base + i, pg = page_of(slot);
                if (pg >= 0) {
                    const int64_t at = (((int64_t)pg * n_kv + kh) * kv.page_size + slot % kv.page_size) * d + p;
                    ((float*)kv.k)[at] = kl, ((float*)kv.k)[at + half] = kr;
                    ((float*)kv.v)[at] = v_lo, ((float*)kv.v)[at + half] = v_hi;
                }
            }
        }
    }
    __syncthreads();
    const int total = ctx + rows.n_region, first_new = ctx + rows.slot_base;
    const int lpk = d / VEC, groups = 64 / lpk, grp = lane / lpk, piece = (lane - grp * lpk) * VEC;
    float m = -INFINITY, l = 0.f;
    float acc[VEC] = {0.f, 0.f, 0.f, 0.f};
    for (int t0 = 64 * wave; t0 < total; t0 += 64 * kRowWaves) {
        const int key = t0 + lane;
        const int pg = t0 == 64 * wave ? pg_first : page_of(key);
        const bool vis = key < total && pg >= 0 && (key < ctx || region_visible(rows, r, i, key - ctx));
        const int64_t base = vis ? (((int64_t)pg * n_kv + kh) * kv.page_size + key % kv.page_size) * d : 0;   // (row 0 of the pool: its weight below is zero)
        const bool fresh = vis && key >= first_new;
        const float* kp = fresh ? k_s + (key - first_new) * (d + 4) : (const float*)kv.k + base;
        v_at[wave][lane] = fresh ? v_s + (key - first_new) * d : (const float*)kv.v + base;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // (read back by the same wave only)
        __builtin_amdgcn_wave_barrier();
        const int nk = min(64, total - t0);
        f32x4_t vv[kU];
        auto fetch_values = [&](int k0) {   // kU rows of every lane group
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int k = k0 + u * groups + grp;
                vv[u] = *(const f32x4_t*)(v_at[wave][k < 64 && grp < groups ? k : 0] + (grp < groups ? piece : 0));
            }
        };
        float s = 0.f;
        for (int c0 = 0; c0 < d; c0 += 64) {   // (a key's 64 elements requested together, and the first values with the first of them)
            f32x4_t kk[64 / VEC];
#pragma unroll
            for (int c = 0; c < 64 / VEC; ++c) kk[c] = *(const f32x4_t*)(kp + c0 + c * VEC);
            if (c0 == 0) fetch_values(0);
#pragma unroll
            for (int c = 0; c < 64 / VEC; ++c)
#pragma unroll
                for (int e = 0; e < VEC; ++e) s = fmaf(q_s[c0 + c * VEC + e], kk[c][e], s);
        }
        if (!vis) s = -INFINITY;
        const float m_new = fmaxf(m, wave_max(s));
        if (m_new == -INFINITY) continue;  // nothing visible so far (uniform across the wave)
        const float corr = expf(m - m_new);      // exp(-inf) = 0 on the first visible tile
        const float w = vis ? expf(s - m_new) : 0.f;
        l = l * corr + wave_sum(w);
        m = m_new;
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] *= corr;
        p_s[wave][lane] = w;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int k0 = 0; k0 < nk; k0 += kU * groups) {
            if (k0 > 0) fetch_values(k0);
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int k = k0 + u * groups + grp;
                const float pk = k < 64 && grp < groups ? p_s[wave][k] : 0.f;
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] = pk != 0.f ? fmaf(pk, vv[u][e], acc[e]) : acc[e];
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    // the partial results, merged in wave and group order
    if (grp < groups)
#pragma unroll
        for (int e = 0; e < VEC; ++e) o_s[wave][grp][piece + e] = acc[e];
    if (lane == 0) {
        m_s[wave] = m;
        l_s[wave] = l;
    }
    __syncthreads();
    if ((int)threadIdx.x >= d) return;
    float mm = m_s[0];
#pragma unroll
    for (int w = 1; w < kRowWaves; ++w) mm = fmaxf(mm, m_s[w]);
    float ll = 0.f, a = 0.f;
#pragma unroll
    for (int w = 0; w < kRowWaves; ++w) {
        const float f = m_s[w] == -INFINITY ? 0.f : expf(m_s[w] - mm);
        ll += f * l_s[w];
        float o_w = 0.f;
        for (int g = 0; g < groups; ++g) o_w += o_s[w][g][threadIdx.x];
        a += f * o_w;
    }
    o[threadIdx.x] = ll > 0.f ? a / ll : 0.f;
}

// Up to 512 keys, by the bound that the host knows: a key's pointer may be the LDS's or the memory's, and loads through such are slower than the row
// attention's global ones, which shows where the keys are the time.  Us per block of a forward, rotary kernel and row attention against this one, heads of 64,
// one sequence of 8 rows and 32 of them: 20 keys 24.5/22.6 and 34.6/33.4, 130 24.8/23.5 and 38.3/37.3, 500 29.4/28.4 and 53.2/53.2, 1000 37.4/38.2 and
// 73.7/78.4, 4000 77.3/89.2 and 207/228; heads of 128, 4 rows: 500 36.6/36.3 and 63.2/61.6, 1000 48.8/49.3 and 98.6/98.0, 12000 301/317 (one sequence).
constexpr int kRopeMaxKeys = 512;
bool attention_rope_supported(int dtype, const Rows& rows, const KVLayer& kv, const void* qkv, const void* bias) {
    return dtype == F32 && !rows.shared_ctx && (int64_t)kv.seq_len_bound + rows.n_region <= kRopeMaxKeys && kv.d % 64 == 0 && kv.d <= 256 && rows.n * (kv.d / 2) <= 64 * kRowWaves &&
           rows.n_region == rows.slot_base + rows.n && (((uintptr_t)qkv | (uintptr_t)kv.k | (uintptr_t)kv.v | (uintptr_t)bias) & 15) == 0;
}

hipError_t attention_rope(hipStream_t s, const Rows& rows, const KVLayer& kv, const void* qkv, void* out, int n_q_heads, float theta, const void* bias,
                          const RopeTable& tab, bool from_table) {
    if (rows.B * rows.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(attn_rope_rows_k, dim3(rows.n, n_q_heads, rows.B), dim3(64 * kRowWaves), 0, s, rows, kv, (const float*)qkv, (float*)out, n_q_heads,
                       1.0f / sqrtf((float)kv.d), (const float*)bias, theta, tab, from_table);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// impl 1 ("MFMA split-KV"), bf16, head_dim 128.
//
// One workgroup (8 waves, two per SIMD) owns (sequence b, kv head, chunk of CK keys, group of
// query-row tiles).  All G query heads of the kv head and all tree rows form the row set R = n*G,
// row r = i*G + g, cut into tiles of 16 rows dealt round-robin to the waves; a wave keeps its tiles'
// Q fragments and fp32 output accumulators in registers and the whole workgroup streams the chunk's
// K/V pages once through a 4-stage LDS ring in tiles of 64 keys, filled by direct global->LDS loads
// issued two tiles ahead.  A wave runs the instance of the program for the number of row tiles it owns
// (waves of one workgroup share the barriers and the fetches, not the code).
//
// Both products run on v_mfma_f32_16x16x32_bf16 in the transposed orientation:
//   S^T[key][row] = sum_d K[key][d] Q[row][d]      A = K rows from LDS, B = Q fragment
//   O^T[d][row]  += sum_key V^T[d][key] P^T[key][row]   A = V^T read with the LDS transpose load,
//                                                       B = P packed from S^T
// In that orientation a lane's S^T results (4 consecutive keys of its own row l%16) are already the
// k-slots the second product's B operand wants, so P never leaves registers, and the k-slot order
// (slot 4*sub + v of lane group g = key 16*sub + 4*g + v) is matched on the V side by which keys each
// transpose load addresses.  A lane's 32 accumulators all belong to one row, so the online-softmax
// rescale is a per-lane scalar.
// Each workgroup writes unnormalised partial outputs with their running max and sum (fp32); a
// second kernel merges the chunks.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;

// max over the four 16-lane groups of a wave (lanes l, l^16, l^32, l^48) without going through the LDS
// crossbar: v_permlane32_swap / v_permlane16_swap exchange half-waves / odd and even 16-lane rows of
// two registers, so swapping a value with a copy of itself puts the partner's value beside it.
__device__ __forceinline__ float group_max4(float x) {
    const uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const float m = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const uint32_t v = __float_as_uint(m);
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

constexpr int kD = 128;       // head_dim of this kernel
constexpr int kKT = 64;       // keys per LDS tile
constexpr int kStages = 4;                  // LDS ring depth
constexpr int kAhead = 2;                   // tiles of K/V in flight; one more stage stays readable for the late waves (below)
constexpr int kStageElems = 2 * kKT * kD;   // one stage: K tile then V tile, 16 KB each
constexpr float kNegBig = -1e30f;
constexpr int kMaxRows = 128;    // rows per sequence whose visibility bits are kept in LDS
constexpr int kMaxChunk = 4096;  // keys per chunk: bounds the page-id table kept in LDS

// Work decomposition.  A work item is (sequence, key range); each item is run by n_kv * row_groups
// workgroups.  The key ranges are cut ON THE DEVICE from the actual sequence lengths (the host only
// knows an upper bound): a one-workgroup planning kernel picks the item length so that the chip
// gets whole rounds of items (kMinTiles .. 64 tiles of 64 keys), gives every sequence equally long chunks,
// and lists the items longest first.  Workgroups are dispatched in list order, so the long items
// start first and the short ones fill the tail (longest-processing-time-first list scheduling).
struct AttnItem {
    int b, k_begin, k_end, slot;   // slot: index of this item's partial result (slots of a sequence are contiguous)
    int page[kAhead * kKT / 16];   // pages of the first kAhead tiles (-1: none): their fetches need not wait for the block table
};
struct AttnWork {        // lives in the workspace, written by attn_plan_k
    int n_items;
    int pad[3];
    // int slot0[B]; int n_chunks[B]; AttnItem items[max_items];
};

struct AttnPlan {
    int row_tiles;   // ceil(R / 16)
    int row_groups;  // row tiles are cut into groups of at most 8 * tpw = 24
    int tpw;         // row tiles per wave (template instance)
    int r_pad;       // row_tiles * 16
    int heads;       // workgroups per item: n_kv * row_groups
    int max_items;   // upper bound of the item count, from the host-side length bound
};

static AttnPlan plan_attention(int B, int n, int G, int n_kv, int bound_total) {
    AttnPlan p;
    p.row_tiles = (n * G + 15) / 16;
    p.r_pad = p.row_tiles * 16;
    p.row_groups = (p.row_tiles + 23) / 24;
    const int per_group = (p.row_tiles + p.row_groups - 1) / p.row_groups;
    const int per_wave = (per_group + 7) / 8;
    p.tpw = per_wave <= 1 ? 1 : (per_wave <= 2 ? 2 : 3);
    p.heads = n_kv * p.row_groups;
    // items <= sum_b ceil(tiles_b / T) <= total_tiles / T + B, and the planner picks T so that they fill
    // whole rounds of 256 workgroups with T <= 64: items * heads <= 256 * ceil((total_tiles / 64 + B) * heads / 256)
    const int64_t tiles_bound = (int64_t)B * ((bound_total + kKT - 1) / kKT);
    const int64_t a = (256 + p.heads - 1) / p.heads, c = (tiles_bound + 63) / 64;
    p.max_items = 2 * B + (int)(a + c);
    return p;
}

static size_t attn_work_bytes(int B, int max_items) {
    return (sizeof(AttnWork) + (size_t)2 * B * sizeof(int) + (size_t)max_items * sizeof(AttnItem) + 255) / 256 * 256;
}

// Shortest chunk: with one or a few sequences, shorter chunks put more of the CUs to work, but every one adds a partial
// result to the merge (one sequence of 8192, main + merging kernel: 8 tiles 11.1 + 4.8 us, 4 tiles 8.5 + 6.0, 3 and 2 tiles 8.4
// + 6.5; three of 5000, 161 query rows: 22.1 + 5.9, 4 tiles 19.9 + 7.4).
constexpr int kMinTiles = 4;
constexpr int kPlanCached = 4096;   // sequences whose lengths and slots the planning kernel keeps in LDS

// One workgroup, so a chain of latencies: lengths are read once, and the counting, the search for the chunk size, the running
// sums and the sort are spread over its threads (once per forward and drafter level; against one thread walking the sequences, in
// a forward: 1 sequence of 8192 7.2 -> 4.6 us, 16 sequences 9.1 -> 6.0, 64 sequences 20.9 -> 9.4; called by itself again and again,
// everything warm, 1 to 6 sequences of 30 to 250 the same within 0.3 us).  A step of a scan is a trip through the LDS crossbar:
// no scan has more of them than its length needs (0.5 us).
__global__ __launch_bounds__(256) void attn_plan_k(const int32_t* __restrict__ seq_len, int B, int n_region, int heads,
                                                   int max_items, AttnWork* __restrict__ work, int len_bound,
                                                   unsigned int* __restrict__ status, const int32_t* __restrict__ block_table,
                                                   int max_pages, int64_t n_pages, const int32_t* __restrict__ n_valid) {
    extern __shared__ int s_len[];   // [min(B, kPlanCached)] keys of a sequence, then as many first slots
    __shared__ int s_total, s_items, s_hist[66], s_pos[66], s_count[65];
    int* slot0 = (int*)(work + 1);
    int* nch = slot0 + B;
    AttnItem* items = (AttnItem*)(nch + B);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int* s_slot = s_len + min(B, kPlanCached);
    // n_valid (causal rows only): the slots of a sequence's inactive rows are not written and no row sees them
    auto keys_of = [&](int b, int len) { return max(len, 0) + (n_valid ? min(max(n_valid[b], 0), n_region) : n_region); };
    auto total_of = [&](int b) { return b < kPlanCached ? s_len[b] : keys_of(b, seq_len[b]); };
    auto tiles_of = [&](int b) { return (total_of(b) + kKT - 1) / kKT; };
    auto slot_of = [&](int b) { return b < kPlanCached ? s_slot[b] : slot0[b]; };
    if (tid < 66) s_hist[tid] = 0;
    if (tid < 65) s_count[tid] = 0;
    if (tid == 0) s_total = 0;
    __syncthreads();
    int mine = 0;
    for (int b = tid; b < B; b += 256) {
        const int len = seq_len[b], keys = keys_of(b, len);
        if (b < kPlanCached) s_len[b] = keys;
        mine += (keys + kKT - 1) / kKT;
        // the grid and the item list were sized from the caller's length bound: a longer sequence would lose
        // part of its context, which only the device can see
        if (status && len > len_bound) atomicOr(status, 1u);
    }
    if (mine) atomicAdd(&s_total, mine);
    __syncthreads();
    // A workgroup takes a whole CU (248 VGPRs per wave, 131 KB of LDS), so the work items run in rounds of
    // 256.  Measured at the 7B benchmark shape (attention ms per step): one round of 256 items 4.02, two
    // rounds 4.33, four 4.20, and 4.6-4.8 when the count falls between whole rounds (384, 768 items): the
    // fewest whole rounds that the 64-tile cap on a chunk allows are the target, and of the chunk sizes that
    // fit them the smallest (items closest to filling the rounds).  Thread (t, part) counts the items of chunk size t.
    {
        const int t = (tid & 63) + 1;
        int64_t items_t = 0;
        if (t >= kMinTiles)
            for (int b = wave; b < B; b += 4) items_t += (tiles_of(b) + t - 1) / t;
        atomicAdd(&s_count[t], (int)(items_t < 0x7fffffff / 256 ? items_t : 0x7fffffff / 256));
    }
    __syncthreads();
    int T;
    {
        const int t = lane + 1;
        const int rounds0 = (int)max(((int64_t)s_total * heads + 256 * 64 - 1) / (256 * 64), (int64_t)1);
        const int rounds_t = t >= kMinTiles ? (int)(((int64_t)s_count[t] * heads + 255) / 256) : 0x7fffffff;
        // (longer chunks never make more items: the fewest rounds are those of the longest)
        const int r = max(__builtin_amdgcn_readlane(rounds_t, 63), rounds0);
        T = __ffsll((unsigned long long)__builtin_amdgcn_ballot_w64(rounds_t <= r));   // lane t - 1 stands for t
    }
    // chunks of every sequence and the slots they take: running sums, 64 sequences at a time
    if (wave == 0) {
        int acc = 0;
        for (int b0 = 0; b0 < B; b0 += 64) {
            const int b = b0 + lane, k = b < B ? (tiles_of(b) + T - 1) / T : 0;
            int sum = k;
            for (int o = 1; o < min(B - b0, 64); o <<= 1) {
                const int up = __shfl_up(sum, o, 64);
                if (lane >= o) sum += up;
            }
            if (b < B) {
                slot0[b] = acc + sum - k, nch[b] = k;
                if (b < kPlanCached) s_slot[b] = acc + sum - k;
            }
            acc += __builtin_amdgcn_readlane(sum, min(B - b0, 64) - 1);
        }
        acc = acc < max_items ? acc : max_items;
        if (lane == 0) work->n_items = s_items = acc;   // cannot exceed the bound when seq_len respects the host's
    }
    __syncthreads();
    // counting sort by tile count, longest first, a thread per item: the sequence is the last one whose slots start at or
    // before it (one without chunks starts where the next one does)
    struct Chunk { int b, kb, tiles; };
    auto chunk_of = [&](int i) {
        int lo = 0, hi = B;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (slot_of(mid) <= i) lo = mid; else hi = mid;
        }
        const int tiles = tiles_of(lo), k = (tiles + T - 1) / T, per = (tiles + k - 1) / k, first = (i - slot_of(lo)) * per;
        return Chunk{lo, first * kKT, max(min(per, tiles - first), 0)};
    };
    const int n_items = s_items;
    for (int i = tid; i < n_items; i += 256) atomicAdd(&s_hist[chunk_of(i).tiles], 1);
    __syncthreads();
    if (wave == 0) {   // s_pos[t] = items longer than t
        const int h = s_hist[64 - lane];
        int sum = h;
        for (int o = 1; o < T; o <<= 1) {   // (no chunk is longer than T: the lanes before T's hold zeros)
            const int up = __shfl_up(sum, o, 64);
            if (lane >= o) sum += up;
        }
        s_pos[64 - lane] = sum - h;
        if (lane == 63) s_pos[0] = sum;
    }
    __syncthreads();
    for (int i = tid; i < n_items; i += 256) {
        const Chunk c = chunk_of(i);
        AttnItem it;
        it.b = c.b, it.k_begin = c.kb, it.k_end = min(total_of(c.b), c.kb + c.tiles * kKT), it.slot = i;
#pragma unroll
        for (int q = 0; q < kAhead * kKT / 16; ++q) {
            const int lp = c.kb / 16 + q;
            const int pg = lp < max_pages && lp * 16 < it.k_end ? block_table[(int64_t)c.b * max_pages + lp] : -1;
            it.page[q] = pg >= 0 && pg < n_pages ? pg : -1;
        }
        items[atomicAdd(&s_pos[c.tiles], 1)] = it;
    }
}

// (non-temporal: a key or value row is read by one workgroup, or by the row groups of one work item at the same
// time, and not again before the next step; marked so, the stream leaves more of the caches to the activations and
// partial results around it: drafter attention 0.59 -> 0.48 ms per step, the step 0.3-0.5 % shorter, same box,
// alternating libraries)
__device__ __forceinline__ void dma_buf_16(u32x4_t rsrc, uint32_t voff_bytes, uint32_t soff_bytes,
                                           uint32_t lds_bytes) {
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen nt lds"
                 :
                 : "v"(voff_bytes), "s"(rsrc), "s"(soff_bytes), "s"(lds_bytes)
                 : "memory", "m0");
}
// The workgroup's program, for a wave that owns NT row tiles (tiles wave, wave + 8, ...).  Waves of one
// workgroup may run different instances (a wave whose share of the row tiles is smaller skips the
// matrix and softmax work it has no rows for; NT = 0: it only fetches its part of the K/V tiles and
// keeps the barriers): every instance passes the same barriers in the same order.
// Workgroup id -> (work item, kv head, row group).  Ids are dealt round-robin over the 8 XCDs, and the row groups of
// one (item, kv head) read the same keys and values: they get ids 8 apart, so that they run on one XCD at the same
// time and the second finds the rows in that XCD's L2.  (With one row group this is item = id / n_kv, head = id % n_kv.)
__device__ __forceinline__ void attn_decode(int id, int heads, int n_kv, int& rank, int& kh, int& rg) {
    const int per = 8 * (heads / n_kv);
    const int g = id / per, within = id - g * per;
    rg = within >> 3;
    const int q = g * 8 + (within & 7);
    rank = q / n_kv;
    kh = q - rank * n_kv;
}

template <int NT>
__device__ __forceinline__ void attn_body(const Rows& rows, const KVLayer& kv, const uint16_t* __restrict__ qkv,
                                          float* __restrict__ part_o, float* __restrict__ part_ml,
                                          const AttnWork* __restrict__ work, int n_seq, int heads, int n_kv, int n_q_heads, int row_tiles,
                                          int tiles_per_group, int r_pad, float scale_log2, float lazy_raw, int max_items) {
    constexpr int TPW = NT > 0 ? NT : 1;   // array extents (nothing is computed in them when NT = 0)
    extern __shared__ __align__(16) uint16_t lds[];
    int rank, kh, rg;
    attn_decode(blockIdx.x, heads, n_kv, rank, kh, rg);   // (n_kv = kv.n_kv, n_seq = rows.B: in registers from the start)
    // (the item is requested together with the count, not after it: where the grid reaches past the list, entry 0 stands in)
    const int n_items = work->n_items;
    const AttnItem* item_p = (const AttnItem*)((const int*)(work + 1) + 2 * n_seq) + (rank < max_items ? rank : 0);
    const AttnItem item = *item_p;
    if (rank >= n_items) return;  // uniform
    const int b = item.b;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, g4 = lane >> 4;
    const int G = n_q_heads / kv.n_kv;
    const int n = rows.n;
    const int R = n * G;
    const int k_begin = item.k_begin, k_end = item.k_end;
    if (k_begin >= k_end) return;  // uniform (an empty sequence)
    const int ctx = kv.seq_len[b];
    const int qkv_dim = (n_q_heads + 2 * kv.n_kv) * kD;
    const int nv = rows.n_valid ? min(rows.n_valid[b], n) : n;

    // ---- this wave's row tiles: Q fragments, masks, accumulators
    u32x4_t qf[TPW][4];
    int row_i[TPW];
    bool tile_on[TPW];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tile = rg * tiles_per_group + wave + 8 * t;
        tile_on[t] = (wave + 8 * t) < tiles_per_group && tile < row_tiles;
        const int r = tile * 16 + l16;
        const int i = r / G, gq = r - i * G;
        const bool valid = tile_on[t] && r < R && i < nv;
        row_i[t] = valid ? i : -1;
        const uint16_t* qp = qkv + (int64_t)(b * n + (valid ? i : 0)) * qkv_dim + (kh * G + gq) * kD + g4 * 8;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            u32x4_t z = {0u, 0u, 0u, 0u};
            qf[t][ks] = valid ? *(const u32x4_t*)(qp + ks * 32) : z;
        }
    }
    f32x4_t acc[TPW][8];
    float m_run[TPW];
    f32x4_t acc_l[TPW];   // running softmax denominator, accumulated by the matrix pipe (PV product against a row of ones)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        m_run[t] = kNegBig;
        acc_l[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) acc[t][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    // ---- K/V tiles: a ring of kStages LDS stages, each [64 keys][128] for K then the same for V,
    // filled by direct global->LDS loads.  One DMA instruction moves 4 keys (1 KB): lane -> key
    // lane/16 of the block, 16-byte slot lane%16, and it fetches logical chunk slot ^ swizzle(key), so a
    // row's chunks are XOR-swizzled by its key index: by key & 15 for K (the 16-byte fragment reads of 16
    // consecutive keys hit 16 distinct chunks) and by 2*key & 15 for V (a transposing read touches two
    // neighbouring chunks of each of 8 keys; with key & 15 those collided pairwise: a third of the LDS
    // cycles were bank conflicts).
    const uint16_t* kpool = (const uint16_t*)kv.k;
    const uint16_t* vpool = (const uint16_t*)kv.v;
    int32_t* page_ids = (int32_t*)(lds + kStages * kStageElems);
    uint64_t* mask_lds = (uint64_t*)(page_ids + kMaxChunk / 16 + 2);  // [n][2] visibility bits of this sequence's rows
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int n_tiles = (k_end - k_begin + kKT - 1) / kKT;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)lds;
    // Every DMA instruction of a wave covers 4 consecutive keys of one page, so the page, the source
    // address and the range check are wave-uniform: they live in scalar registers (a raw buffer
    // descriptor per instruction: base = the block's first key, size = the block, or 0 for a page the
    // block table does not back, which makes every lane out of range: nothing is fetched), and a lane
    // contributes only its constant offset inside the block.
    uint32_t ck[2], cv[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int key_t = (wave_u + 8 * e) * 4 + (lane >> 4);   // key slot inside the tile
        // logical 16-byte chunk this lane fetches: K rows are swizzled by the key slot (the 16 keys of
        // a QK^T fragment read then hit 16 distinct chunks), V rows by twice the key slot (a
        // transposing V read takes two neighbouring chunks of each of 8 keys: they stay distinct)
        ck[e] = (uint32_t)(((lane & 15) ^ (key_t & 15)) * 16);
        cv[e] = (uint32_t)(((lane & 15) ^ ((2 * key_t) & 15)) * 16);
    }
    const uint32_t kq = (uint32_t)lane >> 4;
    auto desc = [&](const uint16_t* base, uint32_t bytes) {
        const uint64_t p = (uint64_t)(uintptr_t)base;
        u32x4_t d;
        d[0] = __builtin_amdgcn_readfirstlane((uint32_t)p);
        d[1] = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32) & 0xffffu);
        d[2] = __builtin_amdgcn_readfirstlane(bytes);
        d[3] = 0x00020000u;
        return d;
    };
    // page_of: page of the 16 keys that start at index 16 * i of the chunk
    auto issue_dma = [&](int tile, int stage, auto page_of) {
        const int t0 = k_begin + tile * kKT;
        const int last = k_end - 1;
        int kb[2], pgv[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            int k0 = t0 + (wave_u + 8 * e) * 4;             // first key of the 4-key block
            k0 = k0 <= last ? k0 : (last & ~3);             // blocks past the end re-read the last key's block
            kb[e] = k0;
            pgv[e] = page_of((k0 - k_begin) >> 4);          // page_size is 16 for this kernel
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int blk = wave_u + 8 * e;
            const int pg = __builtin_amdgcn_readfirstlane(pgv[e]);
            const int lim = min(3, last - kb[e]);           // keys past the end re-read the last key (masked later)
            const int64_t off = (((int64_t)(pg < 0 ? 0 : pg) * kv.n_kv + kh) * 16 + (kb[e] & 15)) * kD;
            const uint32_t size = pg >= 0 ? 1024u : 0u;
            const uint32_t row = min(kq, (uint32_t)lim) << 8;
            const uint32_t dst = lds_base + (uint32_t)(stage * kStageElems + blk * 512) * 2u;
            dma_buf_16(desc(kpool + off, size), row | ck[e], 0u, dst);
            dma_buf_16(desc(vpool + off, size), row | cv[e], 0u, dst + kKT * kD * 2u);
        }
    };
    // the first tiles' pages come with the work item: the fetches start before the masks and the block table are read (with
    // the item asked for together with the count: 8.5 -> 8.1 us at one sequence of 8192, 53.7 -> 53.0 at 16, 16 nodes each)
    auto first_tiles = [&]() {
#pragma unroll
        for (int st = 0; st < kAhead; ++st)
            issue_dma(st < n_tiles ? st : n_tiles - 1, st, [&](int i) { return item_p->page[__builtin_amdgcn_readfirstlane(i)]; });
    };
    first_tiles();
    {
        for (int i = tid; i < n; i += 512) {
            uint64_t m0 = 0, m1 = 0;
            if (i < nv) {
                if (rows.mask) {
                    const uint64_t* mp = rows.mask + (int64_t)(b * n + i) * rows.mask_words;
                    m0 = mp[0];
                    m1 = rows.mask_words > 1 ? mp[1] : 0ull;
                } else {  // causal within the new rows
                    m0 = i >= 63 ? ~0ull : ((2ull << i) - 1ull);
                    m1 = i < 64 ? 0ull : (i >= 127 ? ~0ull : ((2ull << (i - 64)) - 1ull));
                }
            }
            mask_lds[2 * i] = m0;
            mask_lds[2 * i + 1] = m1;
        }
        // page ids of this chunk, range-checked once (-1 = not backed by the block table)
        const int first_page = k_begin / kv.page_size;
        const int n_pg = (k_end - 1) / kv.page_size - first_page + 1;
        int unbacked = 0;
        for (int pi = tid; pi < n_pg; pi += 512) {
            const int lp = first_page + pi;
            int pg = lp < kv.max_pages ? kv.block_table[(int64_t)b * kv.max_pages + lp] : -1;
            pg = (pg >= 0 && pg < kv.n_pages) ? pg : -1;
            page_ids[pi] = pg;
            unbacked |= pg < 0;
        }
        // slots whose DMA is skipped (unbacked pages: a caller error) must still hold finite values:
        // only then is the ring zeroed, and the first tiles are fetched again
        if (__syncthreads_or(unbacked)) {
            __builtin_amdgcn_s_waitcnt(0x0F70u);
            __syncthreads();
            u32x4_t z = {0u, 0u, 0u, 0u};
            for (int e = tid; e < kStages * kStageElems / 8; e += 512) *(u32x4_t*)(lds + e * 8) = z;
            __syncthreads();
            first_tiles();
        }
    }

    // Drain every load issued so far (Q fragments, table reads, the first DMAs) once, here, so that the
    // compiler's own wait bookkeeping enters the loop clean and adds no vmcnt(0) of its own inside it,
    // which would also drain the DMA queue on every tile.
    __builtin_amdgcn_s_waitcnt(0x0F70u);
    // P of the tile whose PV product is still owed (packed bf16, the second product's B operand)
    u32x4_t pb[TPW][2];
#pragma unroll
    for (int t = 0; t < NT; ++t) pb[t][0] = pb[t][1] = u32x4_t{0u, 0u, 0u, 0u};
    auto pv_step = [&](const uint16_t* vt) {
        if constexpr (NT == 0) return;
        // ---- O^T += V^T P^T.  V stays row-major in LDS; ds_read_b64_tr_b16 hands lane (l16, g4) the
        // four keys 4*g4 .. 4*g4+3 of a 16-key sub-tile for head dimension 16*dt + l16: the 16 lanes of
        // a group address a 4-key x 16-dim block (lane s -> key s/4, dims 4*(s%4) ..) and the
        // instruction transposes it.  Two such reads (sub-tiles 2*half, 2*half+1) form the 8 k-slots.
        // Four batches (key half, dimension half) of 8 reads + 4*TPW MFMAs; a batch's reads are issued
        // before the MFMAs of the batch in front of it.
        typedef __attribute__((ext_vector_type(4))) short s16x4_t;
        typedef __attribute__((ext_vector_type(8))) short s16x8_t;
        s16x4_t vv[2][4][2];
        auto read_v = [&](int half, int dq, s16x4_t (*v)[2]) {
#pragma unroll
            for (int d4 = 0; d4 < 4; ++d4)
#pragma unroll
                for (int sub = 0; sub < 2; ++sub) {
                    const int dt = dq * 4 + d4;
                    const int key_t = half * 32 + sub * 16 + 4 * g4 + (l16 >> 2);
                    const int lcv = 2 * dt + ((l16 & 3) >> 1);
                    const uint16_t* vp = vt + key_t * kD + ((lcv ^ ((2 * key_t) & 15)) * 8) + (l16 & 1) * 4;
                    v[d4][sub] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)vp);
                }
        };
        auto mul_v = [&](int half, int dq, s16x4_t (*v)[2]) {
            if (dq == 0) {   // denominator: the same product against a V^T row of ones (bf16 1.0 = 0x3f80)
                const s16x8_t one8 = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc_l[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, one8),
                                                                      __builtin_bit_cast(bf16x8_t, pb[t][half]),
                                                                      acc_l[t], 0, 0, 0);
            }
#pragma unroll
            for (int d4 = 0; d4 < 4; ++d4) {
                const int dt = dq * 4 + d4;
                s16x8_t v8 = {v[d4][0][0], v[d4][0][1], v[d4][0][2], v[d4][0][3],
                              v[d4][1][0], v[d4][1][1], v[d4][1][2], v[d4][1][3]};
                bf16x8_t a = __builtin_bit_cast(bf16x8_t, v8);
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8_t, pb[t][half]),
                                                                        acc[t][dt], 0, 0, 0);
            }
        };
        read_v(0, 0, vv[0]);
        read_v(0, 1, vv[1]);
        mul_v(0, 0, vv[0]);
        read_v(1, 0, vv[0]);
        mul_v(0, 1, vv[1]);
        read_v(1, 1, vv[1]);
        mul_v(1, 0, vv[0]);
        mul_v(1, 1, vv[1]);
        __builtin_amdgcn_sched_group_barrier(0x100, 16, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 5 * NT, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * NT, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 9 * NT, 0);
    };
    // The two waves that share a SIMD (w and w + 4) run the loop half a period apart, so that one's
    // softmax (VALU) runs under the other's two matrix products instead of both doing the same thing
    // at the same time.  Per tile a wave does [PV of the previous tile, S = QK^T] (matrix pipe) and then
    // [softmax] (VALU), two halves of about equal length.  The early waves 0..3 meet the tile barrier at
    // the top of the iteration, before the matrix half; the late waves 4..7 meet the same barrier
    // between their two halves, after QK^T of the tile before.  After each release the early wave of a
    // SIMD therefore multiplies while the late one exponentiates, and the other way round in the second
    // half of the period (measured with cycle stamps: with the late waves' barrier at the top as well,
    // one phase apart only, both multiplied at once and the late wave's softmax ran while the early
    // one sat at the barrier, 5700 against 5200 clocks per tile).  A wave raises its issue priority for
    // its matrix half: a late MFMA costs the pipe, a late exp only the wave that waits for it.
    // Barrier number it guarantees tile it has landed (every wave waited for its own DMAs first) and
    // that nobody reads stage (it - 2) % kStages any more, which is where the fetch issued after it
    // (tile it + 2) lands: the early waves read V of tile it-2 before barrier it, the late ones in the
    // iteration that ended with it.  Both kinds pass exactly n_tiles barriers.
    const bool late = wave_u >= 4;
    auto tile_wait = [&](int it) {
        __builtin_amdgcn_s_waitcnt(0x0F70u | (4 * (kAhead - 1)));  // vmcnt: this tile's 4 DMAs per wave have landed
        __builtin_amdgcn_s_barrier();
    };
    auto tile_fetch = [&](int it) {
        const int nxt = it + kAhead;
        issue_dma(nxt < n_tiles ? nxt : n_tiles - 1, nxt % kStages, [&](int i) { return page_ids[i]; });
    };
    if (late) tile_wait(0);
    for (int it = 0; it < n_tiles; ++it) {
        if (!late) tile_wait(it);
        tile_fetch(it);
        __builtin_amdgcn_s_setprio(2);
        if (it > 0) pv_step(lds + ((it - 1) % kStages) * kStageElems + kKT * kD);
        const int t0 = k_begin + it * kKT;
        const uint16_t* kt = lds + (it % kStages) * kStageElems;
        // 1 for the tile(s) touching the tree region or the chunk's tail, else 0.  Used as the trip count
        // of the masking loop below: a loop with a uniform run-time bound stays a real branch, whereas an
        // `if` around this much select-able code gets flattened and would run on every tile.
        const int mask_reps = t0 + kKT > ctx ? 1 : 0;

        // ---- S^T = K Q^T: each K fragment is read once and feeds the TPW independent row tiles.  The
        // LDS reads are issued in batches of 4 fragments ahead of the 4*TPW MFMAs that consume them, so
        // one LDS latency is exposed per batch instead of one per fragment.
        f32x4_t scs[TPW][4];
        bf16x8_t kf[2][4];
        auto read_k = [&](int st, bf16x8_t* f) {
            const uint16_t* kp = kt + (st * 16 + l16) * kD;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                f[ks] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)(kp + (((4 * ks + g4) ^ l16) * 8)));
        };
        auto mul_k = [&](int st, const bf16x8_t* f) {
#pragma unroll
            for (int t = 0; t < NT; ++t) scs[t][st] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    scs[t][st] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[ks], __builtin_bit_cast(bf16x8_t, qf[t][ks]),
                                                                         scs[t][st], 0, 0, 0);
        };
        // the next 16 keys' fragments fly under each batch's MFMAs: order = 8 reads, then
        // (12 MFMAs, 4 reads) twice, then the last two batches of MFMAs
        if constexpr (NT > 0) {
            read_k(0, kf[0]);
            read_k(1, kf[1]);
            mul_k(0, kf[0]);
            read_k(2, kf[0]);
            mul_k(1, kf[1]);
            read_k(3, kf[1]);
            mul_k(2, kf[0]);
            mul_k(3, kf[1]);
            __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 4 * NT, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 4 * NT, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 8 * NT, 0);
        }
        __builtin_amdgcn_s_setprio(0);
        if (late && it + 1 < n_tiles) tile_wait(it + 1);
        // ---- per row tile: online softmax, P packed straight into the second product's B operand
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            f32x4_t sc[4];
#pragma unroll
            for (int st = 0; st < 4; ++st) sc[st] = scs[t][st];
            float tmax = kNegBig;
            for (int rep = 0; rep < mask_reps; ++rep) {  // region / tail tile only (see mask_reps)
                uint64_t m0 = 0, m1 = 0;
                const int i = row_i[t];
                if (i >= 0) {  // from the LDS copy: no global load (and so no vmcnt wait) inside the loop
                    m0 = mask_lds[2 * i];
                    m1 = mask_lds[2 * i + 1];
                }
#pragma unroll
                for (int st = 0; st < 4; ++st)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int key = t0 + st * 16 + g4 * 4 + v;
                        const int jj = key - ctx;  // index into the masked region when >= 0
                        const uint64_t w = jj < 64 ? m0 : m1;
                        const bool bit = (w >> (jj & 63)) & 1ull;
                        const bool vis = (i >= 0) & (key < k_end) & ((jj < 0) | (bit & (jj < 128)));
                        sc[st][v] = vis ? sc[st][v] : kNegBig;
                    }
            }
#pragma unroll
            for (int st = 0; st < 4; ++st)
#pragma unroll
                for (int v = 0; v < 4; ++v) tmax = fmaxf(tmax, sc[st][v]);
            // Lazy running maximum: softmax is invariant to the reference value, which only has to keep
            // exp2 in range.  As long as no score of this tile exceeds the reference in use by more than
            // 2^8 in the exponent (P <= 256: harmless in bf16 and in the fp32 sums), it stays, and the
            // rescaling of the accumulators (33 multiplies per row tile), the exp of the correction and the
            // cross-lane maximum are all skipped; the decision is taken per wave.
            if (__builtin_amdgcn_ballot_w64(tmax > m_run[t] + lazy_raw) != 0) {
                tmax = group_max4(tmax);
                const float m_new = fmaxf(m_run[t], tmax);
                const float alpha = __builtin_amdgcn_exp2f((m_run[t] - m_new) * scale_log2);
                m_run[t] = m_new;
                acc_l[t] *= alpha;
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) acc[t][dt] *= alpha;
            }
            // the clamp keeps exp2(x*c - mc) = 0 for masked scores (-1e30) while no key has been visible yet
            const float mc = fmaxf(m_run[t], -1e29f) * scale_log2;
            uint32_t pk[4][2];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                float pv[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float x = sc[st][v];
                    float e = __builtin_amdgcn_exp2f(fmaf(x, scale_log2, -mc));
                    pv[v] = e;
                }
                pk[st][0] = pack_bf16x2(pv[0], pv[1]);
                pk[st][1] = pack_bf16x2(pv[2], pv[3]);
            }
            pb[t][0] = u32x4_t{pk[0][0], pk[0][1], pk[1][0], pk[1][1]};
            pb[t][1] = u32x4_t{pk[2][0], pk[2][1], pk[3][0], pk[3][1]};
        }
    }
    pv_step(lds + ((n_tiles - 1) % kStages) * kStageElems + kKT * kD);
    __builtin_amdgcn_s_waitcnt(0x0F70u);  // drain the redundant tail DMAs before the LDS is released

    // ---- partial results: part_o [slot][n_kv][r_pad][128], part_ml [..][r_pad][2]
    const int64_t pbase = ((int64_t)item.slot * kv.n_kv + kh) * r_pad;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (!tile_on[t]) continue;
        const int tile = rg * tiles_per_group + wave + 8 * t;
        const int r = tile * 16 + l16;
        const float l = acc_l[t][0];   // every lane of the row holds the full sum
        float* po = part_o + (pbase + r) * kD;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) *(f32x4_t*)(po + dt * 16 + g4 * 4) = acc[t][dt];
        if (g4 == 0) {
            part_ml[(pbase + r) * 2] = m_run[t];
            part_ml[(pbase + r) * 2 + 1] = l;
        }
    }
}

template <int TPW>
__global__ __launch_bounds__(512) void attn_mfma_k(const AttnWork* __restrict__ work, int n_seq, int heads, int n_kv, int max_items,
                                                   int row_tiles, int tiles_per_group, const uint16_t* __restrict__ qkv,
                                                   float* __restrict__ part_o, float* __restrict__ part_ml, int n_q_heads, int r_pad,
                                                   float scale_log2, float lazy_raw, Rows rows, KVLayer kv) {
    // row tiles of this wave that exist (tile indices rise with t, so they are the first n_on)
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int rank_, kh_, rg;
    attn_decode(blockIdx.x, heads, n_kv, rank_, kh_, rg);
    int n_on = 0;
#pragma unroll
    for (int t = 0; t < TPW; ++t)
        n_on += ((wave + 8 * t) < tiles_per_group && rg * tiles_per_group + wave + 8 * t < row_tiles) ? 1 : 0;
#define TLT_BODY(N) attn_body<N>(rows, kv, qkv, part_o, part_ml, work, n_seq, heads, n_kv, n_q_heads, row_tiles, tiles_per_group, r_pad, scale_log2, lazy_raw, max_items)
    if (n_on >= TPW) TLT_BODY(TPW);
    else if (TPW >= 2 && n_on == TPW - 1) TLT_BODY((TPW >= 2 ? TPW - 1 : 0));
    else if (TPW >= 3 && n_on == TPW - 2) TLT_BODY((TPW >= 3 ? TPW - 2 : 0));
    else TLT_BODY(0);
#undef TLT_BODY
}

// The chunks' partial outputs merged (running max in raw score units), added up in chunk order, by one of two kernels.
// With few rows in all (plain decoding, small batches) a wave's chunks, one load latency each, are the whole kernel: one wave per (b, kv head,
// row), four rows per workgroup; the lanes read a chunk's maximum and sum each, and the outputs of 16 chunks are requested together (on the 17
// chunks that one sequence of 8192 had at 8 tiles each: 12 us one after the other, 6.3 four at a time, 4.8 this way; on its 33 at 4 tiles
// 6.1; 3 sequences x 23 nodes 7.3).
// WPR: waves per row.  With four, the waves of a workgroup fetch and weigh 16 chunks of a row each, so that 64 of them are one trip to memory instead of
// four (attn_merge_wide); the first wave adds all of them up from LDS, in the same order as by itself: the same bits either way.  (Each wave adding up its own
// and the four sums added instead: other bits, and 2 % longer or shorter for the whole call, 1 node of 8192 15.4 us, 8 nodes of 30000 25.3.)
template <int WPR>
__global__ __launch_bounds__(256) void attn_combine_few_k(const AttnWork* __restrict__ work, const float* __restrict__ part_o,
                                                     const float* __restrict__ part_ml, uint16_t* __restrict__ out, int n_seq, int n,
                                                     int n_q_heads, int n_kv, int max_items, int r_pad, float scale_log2,
                                                     const int32_t* __restrict__ n_valid) {
    static_assert(WPR == 1 || WPR == 4, "a wave or a workgroup per row");
    constexpr int U = 16;
    __shared__ float2 s_v[WPR > 1 ? U * (WPR - 1) : 1][64];   // the other waves' weighted outputs
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), part = WPR == 1 ? 0 : wave, lane = threadIdx.x & 63;
    const int r = WPR == 1 ? blockIdx.x * 4 + wave : blockIdx.x, kh = blockIdx.y, b = blockIdx.z;
    const int G = n_q_heads / n_kv;
    if (r >= n * G) return;  // wave-uniform (with four waves per row there are as many workgroups as rows)
    const int i = r / G, gq = r - i * G;
    const int nv = n_valid ? min(n_valid[b], n) : n;
    uint32_t* o = (uint32_t*)(out + ((int64_t)(b * n + i) * n_q_heads + kh * G + gq) * kD);
    const int* slot0 = (const int*)(work + 1);
    const int first = slot0[b];
    int used = slot0[n_seq + b];
    if (first + used > max_items) used = max(max_items - first, 0);
    if (i >= nv || used <= 0) {   // (uniform over a row's waves)
        if (part == 0) o[lane] = 0u;
        return;
    }
    if (part > 0 && used <= U) return;   // (the first wave alone: it meets no barrier below either)
    const int64_t pbase = ((int64_t)first * n_kv + kh) * r_pad + r;
    const int64_t pstride = (int64_t)n_kv * r_pad;
    float2 ml = make_float2(kNegBig, 0.f), v[U];   // lane c: chunk c's (maximum, sum)
    auto fetch = [&](int c) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            v[u] = c + u < used ? *(const float2*)(part_o + (pbase + (c + u) * pstride) * kD + lane * 2) : make_float2(0.f, 0.f);
    };
    if (lane < used) ml = *(const float2*)(part_ml + (pbase + lane * pstride) * 2);
    fetch(U * part);
    float M = ml.x;
    for (int c = lane + 64; c < used; c += 64) M = fmaxf(M, part_ml[(pbase + c * pstride) * 2]);
    M = wave_max(M);
    float w_lane = exp2f((ml.x - M) * scale_log2), l_lane = ml.y * w_lane;
    float a0 = 0.f, a1 = 0.f, L = 0.f;
    auto add = [&](int c, float2 x) {
        L += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l_lane), c & 63));
        a0 += x.x;
        a1 += x.y;
    };
    for (int c0 = 0; c0 < used; c0 += U * WPR) {   // (uniform over a row's waves)
        const int c = c0 + U * part;
        if (c0 > 0) {
            if (WPR > 1) __syncthreads();   // (s_v has been read)
            fetch(c);
            if ((c0 & 63) == 0) {
                ml = c0 + lane < used ? *(const float2*)(part_ml + (pbase + (c0 + lane) * pstride) * 2) : make_float2(kNegBig, 0.f);
                w_lane = exp2f((ml.x - M) * scale_log2), l_lane = ml.y * w_lane;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c + u < used) {   // wave-uniform
                const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_lane), (c + u) & 63));
                v[u] = make_float2(v[u].x * w, v[u].y * w);
                if (part == 0) add(c + u, v[u]);
            }
        if (WPR > 1 && used > U) {
            if (part > 0) {
#pragma unroll
                for (int u = 0; u < U; ++u) s_v[U * (part - 1) + u][lane] = v[u];
            }
            __syncthreads();
            if (part == 0)
                for (int g = U; g < min(U * WPR, used - c0); g += U) {
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = s_v[g - U + u][lane];
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (c0 + g + u < used) add(c0 + g + u, v[u]);
                }
        }
    }
    if (part > 0) return;
    const float inv = L > 0.f ? 1.0f / L : 0.f;
    o[lane] = pack_bf16x2(a0 * inv, a1 * inv);
}
// Four waves per row where a sequence can have 17 chunks (a second batch of 16), as long as the rows' workgroups are at most two per CU: behind that the waves
// that wait at the barrier are missed elsewhere.  It is the longest sequence that counts: its rows end last, and those of shorter ones are left to their first
// wave.  Whole attention call, us, one wave and four, 28 query and 4 kv heads: one sequence of 8192, 1 node 16.7/15.3, 8 nodes 19.5/17.9, 16 nodes 23.6/22.4, 24 nodes
// (672 rows) 27.7/27.1, 48 nodes 37.6/38.3; of 30000, 8 nodes 27.6/25.8; 2 sequences, 8 nodes 22.1/21.1; 3 of 5000, 4 nodes 19.5/18.6, 23 nodes (1932 rows) 31.9/33.0;
// one of 30000 beside three of 1500, 1 node 25.7/23.5, beside fifteen of 600 28.3/26.1; where no sequence has 17, 4 of 8192, 1 node 21.1/21.2, 16 of 8192 52.3/51.8.
constexpr int kMergeChunks = 17, kMergeRows = 512;
static bool attn_merge_wide(const AttnPlan& p, int B, int rows, int bound_total) {
    // chunks that the longest sequence has at most in one round of items: all of them, fewer where they would be shorter than kMinTiles
    const int per_round = (256 + p.heads - 1) / p.heads, tiles = (bound_total + kKT - 1) / kKT;
    return rows <= kMergeRows && std::min(per_round, (tiles + kMinTiles - 1) / kMinTiles) >= kMergeChunks;
}

// With the chip full of waves, several rounds of them, a wave's load latency counts once per round: half a wave per row, 16 bytes per lane and
// four chunks' outputs requested together make the rounds half as many (us, against a wave per row with one chunk after the other: 32 sequences x
// 48 nodes 17.2 -> 11.5, the 32B shape's 16 x 32 16.1 -> 11.0, 4 x 64 9.4 -> 7.7, 1200 prompt rows 12.2 -> 7.0; a wave per row with four
// chunks requested together 17.2).
__global__ __launch_bounds__(256) void attn_combine_k(const AttnWork* __restrict__ work, const float* __restrict__ part_o,
                                                     const float* __restrict__ part_ml, uint16_t* __restrict__ out, int n_seq, int n,
                                                     int n_q_heads, int n_kv, int max_items, int r_pad, float scale_log2,
                                                     const int32_t* __restrict__ n_valid) {
    constexpr int U = 4;
    const int r = blockIdx.x * 8 + (threadIdx.x >> 5), kh = blockIdx.y, b = blockIdx.z, l32 = threadIdx.x & 31;
    const int G = n_q_heads / n_kv;
    if (r >= n * G) return;
    const int* slot0 = (const int*)(work + 1);
    const int first = slot0[b];
    int used = slot0[n_seq + b];
    if (first + used > max_items) used = max(max_items - first, 0);
    const int i = r / G, gq = r - i * G;
    const int nv = n_valid ? min(n_valid[b], n) : n;
    uint2* o = (uint2*)(out + ((int64_t)(b * n + i) * n_q_heads + kh * G + gq) * kD) + l32;
    if (i >= nv || used <= 0) {
        *o = make_uint2(0u, 0u);
        return;
    }
    const int64_t pbase = ((int64_t)first * n_kv + kh) * r_pad + r;
    const int64_t pstride = (int64_t)n_kv * r_pad;
    f32x4_t v[U];
    float2 ml[U];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c0 + u < used) {   // (uniform)
                ml[u] = *(const float2*)(part_ml + (pbase + (c0 + u) * pstride) * 2);
                v[u] = *(const f32x4_t*)(part_o + (pbase + (c0 + u) * pstride) * kD + l32 * 4);
            }
    };
    fetch(0);
    float M = kNegBig, L = 0.f;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < used) M = fmaxf(M, ml[u].x);
    for (int c = U; c < used; ++c) M = fmaxf(M, part_ml[(pbase + c * pstride) * 2]);
    for (int c0 = 0; c0 < used; c0 += U) {
        if (c0 > 0) fetch(c0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c0 + u < used) {
                const float w = exp2f((ml[u].x - M) * scale_log2);
                L += ml[u].y * w;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += v[u][e] * w;
            }
    }
    const float inv = L > 0.f ? 1.0f / L : 0.f;
    *o = make_uint2(pack_bf16x2(acc[0] * inv, acc[1] * inv), pack_bf16x2(acc[2] * inv, acc[3] * inv));
}

static size_t attn_need_bytes(int B, const AttnPlan& p, int n_kv) {
    return attn_work_bytes(B, p.max_items) + (size_t)p.max_items * n_kv * p.r_pad * (kD + 2) * sizeof(float);
}

size_t attention_workspace_bytes(int B, int n, int n_q_heads, int n_kv_heads, int d, int max_ctx) {
    if (d != kD) return 256;
    const int G = n_q_heads / n_kv_heads;
    size_t need = 0;   // any row count up to n may be asked for later
    for (int m = 1; m <= n; ++m) {
        const AttnPlan p = plan_attention(B, m, G, n_kv_heads, max_ctx + 128);
        const size_t x = attn_need_bytes(B, p, n_kv_heads);
        need = x > need ? x : need;
    }
    return need + 256;
}

template <int TPW>
static hipError_t launch_attn_mfma(hipStream_t s, const Rows& rows, const KVLayer& kv, const void* qkv, void* out,
                                   int n_q_heads, const AttnPlan& p, AttnWork* work, float* part_o, float* part_ml,
                                   bool reuse_plan, unsigned int* status) {
    const size_t lds = (size_t)kStages * kStageElems * sizeof(uint16_t) + (kMaxChunk / 16 + 2) * sizeof(int32_t) +
                       (size_t)kMaxRows * 2 * sizeof(uint64_t);
    if (rows.n > kMaxRows) return hipErrorInvalidValue;
    auto kern = attn_mfma_k<TPW>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int tiles_per_group = (p.row_tiles + p.row_groups - 1) / p.row_groups;
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)kD);
    if (!reuse_plan)
        hipLaunchKernelGGL(attn_plan_k, dim3(1), dim3(256), 2 * sizeof(int) * (rows.B < kPlanCached ? rows.B : kPlanCached), s, kv.seq_len,
                           rows.B, rows.n_region, p.heads, p.max_items, work, kv.seq_len_bound, status, kv.block_table, kv.max_pages,
                           kv.n_pages, rows.mask ? nullptr : rows.n_valid);
    // (ids come in groups of 8 (item, kv head) pairs x row groups: see attn_decode)
    const int id_groups = (p.max_items * kv.n_kv + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(id_groups * 8 * p.row_groups), dim3(512), lds, s, (const AttnWork*)work, rows.B, p.heads, kv.n_kv,
                       p.max_items, p.row_tiles, tiles_per_group, (const uint16_t*)qkv, part_o, part_ml, n_q_heads, p.r_pad, scale_log2,
                       8.0f / scale_log2, rows, kv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int R = rows.n * (n_q_heads / kv.n_kv);
    if ((int64_t)R * kv.n_kv * rows.B <= 4096) {   // (waves: half of what the chip holds at once)
        auto few = [&](auto merge, int blocks) {
            hipLaunchKernelGGL(merge, dim3(blocks, kv.n_kv, rows.B), dim3(256), 0, s, (const AttnWork*)work, (const float*)part_o, (const float*)part_ml,
                               (uint16_t*)out, rows.B, rows.n, n_q_heads, kv.n_kv, p.max_items, p.r_pad, scale_log2, rows.n_valid);
        };
        if (attn_merge_wide(p, rows.B, R * kv.n_kv * rows.B, kv.seq_len_bound + rows.n_region)) few(attn_combine_few_k<4>, R);
        else few(attn_combine_few_k<1>, (R + 3) / 4);
    } else {
        hipLaunchKernelGGL(attn_combine_k, dim3((R + 7) / 8, kv.n_kv, rows.B), dim3(256), 0, s, (const AttnWork*)work,
                           (const float*)part_o, (const float*)part_ml, (uint16_t*)out, rows.B, rows.n, n_q_heads, kv.n_kv, p.max_items, p.r_pad,
                           scale_log2, rows.n_valid);
    }
    return hipGetLastError();
}

hipError_t attention(hipStream_t s, int dtype, const Rows& rows, const KVLayer& kv, const void* qkv, void* out,
                     int n_q_heads, void* ws, size_t ws_bytes, int impl, bool reuse_plan, unsigned int* status) {
    if (rows.B * rows.n <= 0) return hipSuccess;
    if (kv.d % 64 != 0 || kv.d > 256) return hipErrorInvalidValue;
    const int G = n_q_heads / kv.n_kv;
    const bool mfma_ok = dtype == BF16 && kv.d == kD && rows.n_region <= 128 && kv.page_size == 16;
    if (mfma_ok && impl != 0) {
        const AttnPlan p = plan_attention(rows.B, rows.n, G, kv.n_kv, kv.seq_len_bound + rows.n_region);
        if (attn_need_bytes(rows.B, p, kv.n_kv) <= ws_bytes) {
            AttnWork* work = (AttnWork*)ws;
            float* part_o = (float*)((char*)ws + attn_work_bytes(rows.B, p.max_items));
            float* part_ml = part_o + (size_t)p.max_items * kv.n_kv * p.r_pad * kD;
            switch (p.tpw) {
                case 1: return launch_attn_mfma<1>(s, rows, kv, qkv, out, n_q_heads, p, work, part_o, part_ml, reuse_plan, status);
                case 2: return launch_attn_mfma<2>(s, rows, kv, qkv, out, n_q_heads, p, work, part_o, part_ml, reuse_plan, status);
                default: return launch_attn_mfma<3>(s, rows, kv, qkv, out, n_q_heads, p, work, part_o, part_ml, reuse_plan, status);
            }
        }
        if (impl == 1) return hipErrorInvalidValue;  // explicitly requested but the workspace cannot hold it
    }
    float scale = 1.0f / sqrtf((float)kv.d);
    dim3 grid(rows.n, n_q_heads, rows.B), block(64 * kRowWaves);
    if (dtype == F32)
        hipLaunchKernelGGL(attn_wave_per_row_k<float>, grid, block, 0, s, rows, kv, (const float*)qkv, (float*)out,
                           n_q_heads, scale);
    else
        hipLaunchKernelGGL(attn_wave_per_row_k<bf16>, grid, block, 0, s, rows, kv, (const bf16*)qkv, (bf16*)out,
                           n_q_heads, scale);
    return hipGetLastError();
}

}  // namespace tlt

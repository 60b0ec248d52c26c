// Row-wise kernels of the decoder block: embedding gather, RMSNorm, rotary embedding fused with the
// write of new keys/values into the paged cache, SiLU gating, the drafter's input rows.
// All are HBM-bound streaming kernels: one workgroup per row, 16-byte accesses where the layout allows.
#include "dev_common.h"
#include "kernels.h"

namespace tlt {

// Four consecutive elements at a 4-element boundary (8 or 16 bytes) as floats, and back.
__device__ __forceinline__ float4 load_four(const float* p) { return *(const float4*)p; }
__device__ __forceinline__ float4 load_four(const bf16* p) {
    const uint2 v = *(const uint2*)p;
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
}
__device__ __forceinline__ void store_four(float* p, const float4& v) { *(float4*)p = v; }
__device__ __forceinline__ void store_four(bf16* p, const float4& v) { *(uint2*)p = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w)); }

// VEC: h % 4 == 0 and every base on a boundary of four elements (the rows are then, too): a row's loads are a few per thread and all
// in flight at once; element by element it was a chain of them (256 rows of 3584: 10.6 -> 5.3 us; the drafter's input below, 8 rows: 7.7 -> 5.2).
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void embed_rows_k(int M, int h, int V, const int32_t* __restrict__ tokens, const T* __restrict__ embed,
                                                    float* __restrict__ x) {
    const int r = blockIdx.x, t = tokens[r];
    const bool ok = t >= 0 && t < V;
    const T* e = embed + (int64_t)(ok ? t : 0) * h;
    float* o = x + (int64_t)r * h;
    if constexpr (VEC) {
#pragma unroll 4
        for (int c = 4 * threadIdx.x; c < h; c += 4 * 256) store_four(o + c, ok ? load_four(e + c) : make_float4(0.f, 0.f, 0.f, 0.f));
    } else {
        for (int c = threadIdx.x; c < h; c += 256) o[c] = ok ? to_float(e[c]) : 0.f;
    }
}

// Row r of a norm launch: where it is read, and where it goes with its addends absorbed (see NormIO).
struct NormRow {
    const float* in;
    float* keep;      // null: it stays where it is
    int64_t src;      // row of x, and of the addends
    bool absorb;
};
template <bool PLAIN>   // row r of x, kept there (io is the default one, and its words need not be waited for)
__device__ __forceinline__ NormRow norm_row(const NormIO& io, int h, float* x, bool add) {
    const int r = blockIdx.x;
    NormRow o;
    if constexpr (PLAIN) {
        o.src = r;
        o.in = x + (int64_t)r * h;
        o.absorb = add;
        o.keep = add ? x + (int64_t)r * h : nullptr;
        return o;
    }
    o.src = (int64_t)r * io.src_stride;
    float* copy = io.copy ? io.copy + ((int64_t)(r / io.copy_n) * io.copy_stride + io.copy_base + r % io.copy_n) * h : nullptr;
    bool have = true;
    if (io.n > 0) {
        const int raw = io.n_valid[r], nv = raw < io.n ? raw : io.n;
        have = nv > 0;
        o.src = (int64_t)r * io.n + (have ? nv - 1 : 0);
        if (io.len && threadIdx.x == 0) io.len[r] += raw;
    }
    o.in = have ? x + o.src * h : copy;   // (no new row: the one that was kept last time)
    o.absorb = have && add;
    o.keep = !have ? nullptr : (copy ? copy : (add ? x + o.src * h : nullptr));
    return o;
}

// `add` (optional, [n_add][rows of x][h] in TA = T or float): the residual stream takes x[r] += add[r]
// first -- the output projection leaves its product there instead of read-modify-writing x itself.
template <typename T, typename TA>
__global__ __launch_bounds__(256) void rmsnorm_k(int h, float* __restrict__ x, const T* __restrict__ gamma,
                                                 float eps, T* __restrict__ out, const TA* __restrict__ add, int n_add,
                                                 int64_t add_stride, int assign, NormIO io) {
    __shared__ float red[4];
    const NormRow row = norm_row<false>(io, h, x, add != nullptr);
    T* o = out + (int64_t)blockIdx.x * h;
    auto value = [&](int c) {
        float v = (row.absorb && assign) ? 0.f : row.in[c];
        if (row.absorb)
            for (int k = 0; k < n_add; ++k) v += to_float(add[k * add_stride + row.src * h + c]);
        return v;
    };
    float ss = 0.f;
    for (int c = threadIdx.x; c < h; c += 256) {
        const float v = value(c);
        if (row.keep) row.keep[c] = v;   // (each element is read, kept and read again by the same thread)
        ss += v * v;
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = red[0] + red[1] + red[2] + red[3];
    float inv = 1.0f / sqrtf(tot / (float)h + eps);
    const float* again = row.keep ? row.keep : row.in;
    for (int c = threadIdx.x; c < h; c += 256) o[c] = from_float<T>(again[c] * inv * to_float(gamma[c]));
}

// Same, for h % 4 == 0 and h <= 1024 * NK: the row is read once with 16-byte loads and stays in
// registers (NK float4 per thread) between the reduction and the scaling.
template <typename T, int NK, typename TA, bool PLAIN, int NB = 4, int NTHR = 256>   // NB: slices of `add` whose loads are issued together
__global__ __launch_bounds__(NTHR) void rmsnorm_vec_k(int h, float* __restrict__ x, const T* __restrict__ gamma,
                                                     float eps, T* __restrict__ out, const TA* __restrict__ add,
                                                     int n_add, int64_t add_stride, int assign, NormIO io) {
    __shared__ float red[NTHR / 64];
    const int h4 = h >> 2;
    const NormRow row = norm_row<PLAIN>(io, h, x, add != nullptr);
    T* o = out + (int64_t)blockIdx.x * h;
    float4 v[NK];
    // (the gains are requested with the row, not after the reduction: one memory latency instead of two)
    typedef __attribute__((ext_vector_type(sizeof(T)))) uint32_t gain_t;   // four T
    gain_t gv[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int c = threadIdx.x + k * NTHR;
        gv[k] = c < h4 ? ((const gain_t*)gamma)[c] : gain_t{};
    }
    float ss = 0.f;
    {
#pragma unroll
        for (int k = 0; k < NK; ++k) {
            const int c = threadIdx.x + k * NTHR;
            v[k] = (c < h4 && !(row.absorb && assign)) ? ((const float4*)row.in)[c] : make_float4(0.f, 0.f, 0.f, 0.f);
            if (row.absorb && c < h4) {
                const TA* a = add + row.src * h + 4 * c;
                if constexpr (sizeof(TA) == 2) {
                    const uint2 pk = *(const uint2*)a;
                    v[k].x += __uint_as_float(pk.x << 16);
                    v[k].y += __uint_as_float(pk.x & 0xffff0000u);
                    v[k].z += __uint_as_float(pk.y << 16);
                    v[k].w += __uint_as_float(pk.y & 0xffff0000u);
                } else {
                    // partial products, summed in their fixed order; the loads of up to four slices are issued
                    // together (one after the other they would each expose a memory latency)
                    for (int j0 = 0; j0 < n_add; j0 += NB) {
                        float4 av[NB];
#pragma unroll
                        for (int u = 0; u < NB; ++u)
                            av[u] = j0 + u < n_add ? *(const float4*)(a + (j0 + u) * add_stride) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                        for (int u = 0; u < NB; ++u) {
                            v[k].x += av[u].x; v[k].y += av[u].y; v[k].z += av[u].z; v[k].w += av[u].w;
                        }
                    }
                }
            }
            if (row.keep && c < h4) ((float4*)row.keep)[c] = v[k];
            ss += v[k].x * v[k].x + v[k].y * v[k].y + v[k].z * v[k].z + v[k].w * v[k].w;
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < NTHR / 64; ++w) tot += red[w];
    const float inv = 1.0f / sqrtf(tot / (float)h + eps);
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const int c = threadIdx.x + k * NTHR;
        if (c >= h4) continue;
        float g[4];
        if constexpr (sizeof(T) == 2) {
            g[0] = __uint_as_float(gv[k][0] << 16), g[1] = __uint_as_float(gv[k][0] & 0xffff0000u);
            g[2] = __uint_as_float(gv[k][1] << 16), g[3] = __uint_as_float(gv[k][1] & 0xffff0000u);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) g[q] = __uint_as_float(gv[k][q]);
        }
        float y[4] = {v[k].x * inv * g[0], v[k].y * inv * g[1], v[k].z * inv * g[2], v[k].w * inv * g[3]};
        if constexpr (sizeof(T) == 2) {
            *(uint2*)(o + 4 * c) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
        } else {
            *(float4*)(o + 4 * c) = make_float4(y[0], y[1], y[2], y[3]);
        }
    }
}

constexpr int kRopeThreads = 512;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
template <typename T>
union Piece {   // 16 bytes of T
    u32x4_t v;
    T e[16 / sizeof(T)];
    __device__ Piece() {}
};

// One workgroup per row.  Angles are formed in double (positions reach 32K, where an fp32 product
// pos * inv_freq already carries ~1e-3 rad of rounding), once per (row, pair index), then reused by
// every head.  q is rotated in place; k is rotated and stored with v at the row's cache slot.  An
// optional projection bias is added first (to q, k and v).
// Every layer of a forward rotates the same rows by the same angles into the same slots: the first one (TBL = false)
// leaves both in `tab`, the others (TBL = true) read them there.  The kernel is a chain of latencies (length, block
// table, double-precision power and sine, the rotation, v after q and k); with the table, and a thread for every piece, it has
// one load to wait for.  7B shape, us per layer before and after: 1 row 8.3 -> 4.7, 64 rows 9.3 -> 6.3, 256 rows 9.9 ->
// 7.2, 1536 rows 13.0 -> 9.8 (kernel traces).
template <typename T, bool SRC32, bool TBL>   // SRC32: the projection arrives as fp32 partial products (its own instance: it needs many more registers)
__global__ __launch_bounds__(kRopeThreads) void rope_kv_write_k(const float* __restrict__ src32, T* __restrict__ qkv, const int64_t* __restrict__ tab_at,
                                                       const float* __restrict__ tab_cs, int64_t src_stride, int n_src, int n_q_heads, int n_kv,
                                                       int d, const T* __restrict__ bias, float theta, Rows rows, KVLayer kv, RopeTable tab) {
    extern __shared__ __align__(16) float cs[];  // [d/2] cos, [d/2] sin
    const int half = d >> 1;   // (the first words, which a wave has from the start, are all that its loads need: n_kv = kv.n_kv, d = kv.d)
    const int r = blockIdx.x;
    const int qkv_dim = (n_q_heads + 2 * n_kv) * d;
    T* row = qkv + (int64_t)r * qkv_dim;
    // src32 (optional): the projection's product still in fp32 (a split-K GEMM accumulated it there);
    // q then goes to `qkv` in T for the attention kernel, exactly as when it is rotated in place
    const float* row32 = SRC32 ? src32 + (int64_t)r * qkv_dim : nullptr;
    auto load_piece = [&](int elem, Piece<T>& out) {   // VEC consecutive elements of the row, as T
        if constexpr (SRC32) {
#pragma unroll
            for (int k = 0; k < 16 / (int)sizeof(T); k += 4) {
                float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
                for (int j0 = 0; j0 < n_src; j0 += 8) {   // partial products of a split projection, in their fixed order
                    float4 g[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        g[u] = j0 + u < n_src ? *(const float4*)(row32 + (j0 + u) * src_stride + elem + k) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        f.x += g[u].x; f.y += g[u].y; f.z += g[u].z; f.w += g[u].w;
                    }
                }
                out.e[k] = from_float<T>(f.x);
                out.e[k + 1] = from_float<T>(f.y);
                out.e[k + 2] = from_float<T>(f.z);
                out.e[k + 3] = from_float<T>(f.w);
            }
        } else {
            out.v = *(const u32x4_t*)(row + elem);
        }
    };
    // both halves of a rotation pair at once: with partial products every slice's loads for the two
    // pieces are issued together (one memory latency instead of one per piece and slice batch)
    auto load_pair = [&](int elem_lo, int elem_hi, Piece<T>& lo, Piece<T>& hi) {
        if constexpr (!SRC32) {
            lo.v = *(const u32x4_t*)(row + elem_lo);
            hi.v = *(const u32x4_t*)(row + elem_hi);
            return;
        }
        constexpr int NQ = 16 / (int)sizeof(T) / 4;   // float4 per piece
        float4 f[2][NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) f[0][q] = f[1][q] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int j0 = 0; j0 < n_src; j0 += 8) {   // partial products of a split projection, in their fixed order
            float4 g[2][NQ][8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const bool on = j0 + u < n_src;
                    g[0][q][u] = on ? *(const float4*)(row32 + (j0 + u) * src_stride + elem_lo + 4 * q) : make_float4(0.f, 0.f, 0.f, 0.f);
                    g[1][q][u] = on ? *(const float4*)(row32 + (j0 + u) * src_stride + elem_hi + 4 * q) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh) {
                        f[hh][q].x += g[hh][q][u].x; f[hh][q].y += g[hh][q][u].y;
                        f[hh][q].z += g[hh][q][u].z; f[hh][q].w += g[hh][q][u].w;
                    }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            lo.e[4 * q] = from_float<T>(f[0][q].x); lo.e[4 * q + 1] = from_float<T>(f[0][q].y);
            lo.e[4 * q + 2] = from_float<T>(f[0][q].z); lo.e[4 * q + 3] = from_float<T>(f[0][q].w);
            hi.e[4 * q] = from_float<T>(f[1][q].x); hi.e[4 * q + 1] = from_float<T>(f[1][q].y);
            hi.e[4 * q + 2] = from_float<T>(f[1][q].z); hi.e[4 * q + 3] = from_float<T>(f[1][q].w);
        }
    };
    T* kc = (T*)kv.k;
    T* vc = (T*)kv.v;
    // 16-byte pieces, one per thread (and more where the heads need it): VEC consecutive pair indices j of one q or k
    // head, both halves of each pair, or VEC consecutive elements of v
    constexpr int VEC = 16 / sizeof(T);
    const int cph = half / VEC;   // pieces per half head
    const int n_piece = (n_q_heads + n_kv) * cph, n_all = n_piece + n_kv * d / VEC;
    const int v0 = (n_q_heads + n_kv) * d;
    auto load = [&](int e, u32x4_t& lo, u32x4_t& hi) {   // (plain vectors: unions merged over the two branches end in scratch)
        if (e < n_piece) {
            const int hd = e / cph, j0 = (e - hd * cph) * VEC;
            Piece<T> a, b;
            load_pair(hd * d + j0, hd * d + half + j0, a, b);
            lo = a.v;
            hi = b.v;
        } else {
            Piece<T> a;
            load_piece(v0 + (e - n_piece) * VEC, a);
            lo = a.v;
        }
    };
    // the first piece's loads fly while the angles and the slot are found
    u32x4_t lo0 = {0u, 0u, 0u, 0u}, hi0 = lo0;
    if ((int)threadIdx.x < n_all) load(threadIdx.x, lo0, hi0);
    int64_t at;   // element offset of the row's slot in the cache (head 0); -1: no page, -2: the row is not active
    const float* c_row = cs;
    if constexpr (TBL) {
        at = tab_at[r];
        c_row = tab_cs + (int64_t)r * d;
    } else {
        const int b = r / rows.n, i = r - b * rows.n;
        at = -2;
        if (!rows.n_valid || i < rows.n_valid[b]) {
            const int ctx = kv.seq_len[b];
            const int pos = ctx + rows.pos_base + (rows.pos_off ? rows.pos_off[r] : rows.pos_stride * i);
            PageRef pr;
            const bool have = locate(kv.block_table, kv.max_pages, kv.n_pages, kv.page_size, b, ctx + rows.slot_base + i, pr);
            at = have ? (pr.page * kv.n_kv * kv.page_size + pr.row) * d : -1;
            for (int j = threadIdx.x; j < half; j += blockDim.x) {
                double inv_freq = pow((double)theta, -2.0 * (double)j / (double)d);
                double sn, c;
                sincos((double)pos * inv_freq, &sn, &c);
                cs[j] = (float)c;
                cs[half + j] = (float)sn;
                if (tab.cs) {
                    tab.cs[(int64_t)r * d + j] = (float)c;
                    tab.cs[(int64_t)r * d + half + j] = (float)sn;
                }
            }
        }
        if (tab.cs && threadIdx.x == 0) tab.at[r] = at;
        __syncthreads();
    }
    if (at == -2) return;
    const int64_t head_stride = (int64_t)kv.page_size * d;
    for (int e = threadIdx.x; e < n_all; e += blockDim.x) {
        if (e != (int)threadIdx.x) load(e, lo0, hi0);
        Piece<T> lo, hi, blo, bhi;
        lo.v = lo0;
        hi.v = hi0;
        if (e >= n_piece) {
            if (at < 0) continue;
            const int v = (e - n_piece) * VEC, kh = v / d;
            if (bias) {
                blo.v = *(const u32x4_t*)(bias + v0 + v);
#pragma unroll
                for (int k = 0; k < VEC; ++k) lo.e[k] = from_float<T>(to_float(lo.e[k]) + to_float(blo.e[k]));
            }
            *(u32x4_t*)(vc + at + kh * head_stride + (v - kh * d)) = lo.v;
            continue;
        }
        const int hd = e / cph, j0 = (e - hd * cph) * VEC;
        if (bias) {
            blo.v = *(const u32x4_t*)(bias + hd * d + j0);
            bhi.v = *(const u32x4_t*)(bias + hd * d + half + j0);
        }
        f32x4_t cv[VEC / 4], sv[VEC / 4];
#pragma unroll
        for (int k = 0; k < VEC / 4; ++k) {
            cv[k] = *(const f32x4_t*)(c_row + j0 + 4 * k);
            sv[k] = *(const f32x4_t*)(c_row + half + j0 + 4 * k);
        }
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
            float x1 = to_float(lo.e[k]), x2 = to_float(hi.e[k]);
            if (bias) {
                x1 += to_float(blo.e[k]);
                x2 += to_float(bhi.e[k]);
            }
            const float c = cv[k / 4][k % 4], sn = sv[k / 4][k % 4];
            lo.e[k] = from_float<T>(x1 * c - x2 * sn);
            hi.e[k] = from_float<T>(x2 * c + x1 * sn);
        }
        if (hd < n_q_heads) {
            T* p = row + (int64_t)hd * d;
            *(u32x4_t*)(p + j0) = lo.v;
            *(u32x4_t*)(p + half + j0) = hi.v;
        } else if (at >= 0) {
            T* p = kc + at + (hd - n_q_heads) * head_stride;
            *(u32x4_t*)(p + j0) = lo.v;
            *(u32x4_t*)(p + half + j0) = hi.v;
        }
    }
}

template <typename T>
__global__ void swiglu_k(int64_t count, const T* __restrict__ g, const T* __restrict__ u, T* __restrict__ out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) {
        float a = to_float(g[i]);
        out[i] = from_float<T>(a / (1.0f + expf(-a)) * to_float(u[i]));
    }
}

template <typename T, bool VEC>   // (VEC: as embed_rows_k)
__global__ __launch_bounds__(256) void draft_input_k(int n, int h, int V, const int32_t* __restrict__ tok, const int32_t* __restrict__ src,
                              const int32_t* __restrict__ n_valid, int src_seq_stride, int64_t hidden_rows,
                              const float* __restrict__ hidden, const T* __restrict__ embed, T* __restrict__ xin) {
    int r = blockIdx.x;
    int b = r / n, i = r - b * n;
    int t = tok[r];
    int64_t sr = src[r];
    bool ok = t >= 0 && t < V && sr >= 0 && (!n_valid || i < n_valid[b]);
    if (ok && src_seq_stride > 0) {
        ok = sr < src_seq_stride;
        sr += (int64_t)b * src_seq_stride;
    }
    ok = ok && sr < hidden_rows;
    T* o = xin + (int64_t)r * 2 * h;
    if constexpr (VEC) {
        const T* e = embed + (int64_t)(ok ? t : 0) * h;
        const float* hid = hidden + (ok ? sr : 0) * h;
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
        for (int c = 4 * threadIdx.x; c < h; c += 4 * 256) {
            const float4 a = ok ? load_four(e + c) : z, b4 = ok ? load_four(hid + c) : z;
            store_four(o + c, a);
            store_four(o + h + c, b4);
        }
        return;
    }
    for (int c = threadIdx.x; c < h; c += 256) {
        o[c] = ok ? embed[(int64_t)t * h + c] : from_float<T>(0.f);
        o[h + c] = ok ? from_float<T>(hidden[sr * h + c]) : from_float<T>(0.f);
    }
}

__global__ void add_i32_k(int n, int32_t* dst, const int32_t* a, int add_const) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] += (a ? a[i] : 0) + add_const;
}

__global__ void report_words_k(int n, const int32_t* __restrict__ src, const unsigned int* __restrict__ status, int32_t* __restrict__ dst) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
    else if (i == n) dst[n] = status ? (int32_t)*status : 0;
}

__global__ void zero_f32_k(int64_t count, float4* __restrict__ dst) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) dst[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__global__ void copy_f32_k(int64_t count, const float4* __restrict__ src, float4* __restrict__ dst) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) dst[i] = src[i];
}

// Last row of every n rows of x -> dst row b * dst_seq_stride.
__global__ void gather_last_rows_k(int n, int h4, const float4* __restrict__ src, float4* __restrict__ dst, int dst_seq_stride) {
    const int b = blockIdx.x;
    const int64_t sr = (int64_t)b * n + n - 1, d = (int64_t)b * dst_seq_stride;
    for (int c = threadIdx.x; c < h4; c += blockDim.x) dst[d * h4 + c] = src[sr * h4 + c];
}

// One workgroup per virtual sequence b * C + j = chunk j of sequence b in this pass (see PrefillPass).
__global__ void prefill_rows_k(PrefillPass p) {
    const int v = blockIdx.x, b = v / p.C, j = v - b * p.C;
    const int start = p.done + j * p.m, cnt = min(p.m, p.n_tokens - start);
    if (threadIdx.x == 0) {
        p.n_valid[v] = cnt;
        p.len_t[v] = p.seq_len_t[b] + j * p.m;
        p.len_d[v] = p.seq_len_d[b] + j * p.m;
    }
    const int32_t* t = p.tokens + (int64_t)b * p.token_stride + start;
    for (int i = threadIdx.x; i < p.m; i += blockDim.x) {
        p.tok[(int64_t)v * p.m + i] = i < cnt ? t[i] : -1;
        p.nxt[(int64_t)v * p.m + i] = i < cnt ? t[i + 1] : -1;
        p.src[(int64_t)v * p.m + i] = i;
    }
    for (int i = threadIdx.x; i < p.pages_t; i += blockDim.x) p.vtab_t[(int64_t)v * p.pages_t + i] = p.table_t[(int64_t)b * p.pages_t + i];
    for (int i = threadIdx.x; i < p.pages_d; i += blockDim.x) p.vtab_d[(int64_t)v * p.pages_d + i] = p.table_d[(int64_t)b * p.pages_d + i];
}

hipError_t prefill_rows(hipStream_t s, int B, const PrefillPass& p) {
    hipLaunchKernelGGL(prefill_rows_k, dim3(B * p.C), dim3(256), 0, s, p);
    return hipGetLastError();
}

#define DISPATCH_T(dtype, ...)              \
    if ((dtype) == F32) {                   \
        using T = float;                    \
        __VA_ARGS__;                        \
    } else {                                \
        using T = bf16;                     \
        __VA_ARGS__;                        \
    }

hipError_t embed_rows(hipStream_t s, int dtype, int M, int h, int V, const int32_t* tokens, const void* embed, float* x) {
    if (M <= 0) return hipSuccess;
    const uintptr_t four = dtype == F32 ? 15 : 7;
    if (h % 4 == 0 && ((uintptr_t)embed & four) == 0 && ((uintptr_t)x & 15) == 0) {
        DISPATCH_T(dtype, hipLaunchKernelGGL((embed_rows_k<T, true>), dim3(M), dim3(256), 0, s, M, h, V, tokens, (const T*)embed, x));
    } else {
        DISPATCH_T(dtype, hipLaunchKernelGGL((embed_rows_k<T, false>), dim3(M), dim3(256), 0, s, M, h, V, tokens, (const T*)embed, x));
    }
    return hipGetLastError();
}

template <typename T, typename TA>
static void rmsnorm_launch_t(hipStream_t s, int M, int h, float* x, const void* gamma, float eps, void* out, const NormIO& io,
                             const void* add, int n_add, int64_t add_rows, bool assign) {
    const int64_t add_stride = add_rows * h;
    const bool vec_ok = h % 4 == 0 && (((uintptr_t)x | (uintptr_t)add | (uintptr_t)io.copy) & 15) == 0 &&
                        ((uintptr_t)gamma & (4 * sizeof(T) - 1)) == 0;
    const bool plain = io.src_stride == 1 && io.n == 0 && !io.copy;
    auto launch = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3(M), dim3(threads), 0, s, h, x, (const T*)gamma, eps, (T*)out, (const TA*)add, n_add, add_stride,
                           (int)assign, io);
    };
    if (vec_ok && h <= 4096 && add && (n_add > 4 || M <= 64) && sizeof(TA) == 4)
        // many slices or few rows (so few workgroups): one 16-byte position per thread and all its slices' loads in
        // flight at once.  (Few rows and up to four slices, against 256 threads, us per norm inside a forward of 1-32 rows: widths
        // 3584 and 4096 1.4 less, 1536 0.4 less, 256 to 1024 and 2048 the same within 0.3, though most waves are idle at 256.)
        plain ? launch(rmsnorm_vec_k<T, 1, TA, true, 12, 1024>, 1024) : launch(rmsnorm_vec_k<T, 1, TA, false, 12, 1024>, 1024);
    else if (vec_ok && h > 4096 && h <= 8192 && M <= 512 && add && sizeof(TA) == 4)
        // (wider rows: two positions per thread and up to eight slices of each in flight; with 256 threads eight positions waited for their slices one
        // after the other.  Width 5120, us per norm inside a step, 256 threads and 1024: 25 rows 5.8 and 4.4, 112 rows 8.3 and 5.3, 150 rows 7.3 and 5.8, 512 rows
        // 12.9 and 12.4.  With more rows the chip is full of either and the bytes count: medians over widths 4608 to 8192, 512 rows 10.0 and 10.0, 1024 16.8 and 18.5,
        // 2048 30.1 and 33.1, 4096 54.4 and 62.3.)
        plain ? launch(rmsnorm_vec_k<T, 2, TA, true, 8, 1024>, 1024) : launch(rmsnorm_vec_k<T, 2, TA, false, 8, 1024>, 1024);
    else if (vec_ok && h <= 4096)
        plain ? launch(rmsnorm_vec_k<T, 4, TA, true>, 256) : launch(rmsnorm_vec_k<T, 4, TA, false>, 256);
    else if (vec_ok && h <= 8192)   // (the 32B and 70B widths)
        plain ? launch(rmsnorm_vec_k<T, 8, TA, true>, 256) : launch(rmsnorm_vec_k<T, 8, TA, false>, 256);
    else
        launch(rmsnorm_k<T, TA>, 256);
}

hipError_t rmsnorm(hipStream_t s, int dtype, int M, int h, float* x, const void* gamma, float eps, void* out, const NormIO& io,
                   const void* add, bool add_f32, int n_add, int64_t add_rows, bool assign) {
    if (M <= 0) return hipSuccess;
    if (add && !add_f32 && dtype != F32 && n_add != 1) return hipErrorInvalidValue;   // several addends: fp32 partial products only
    if (dtype == F32) rmsnorm_launch_t<float, float>(s, M, h, x, gamma, eps, out, io, add, n_add, add_rows, assign);
    else if (!add || add_f32) rmsnorm_launch_t<bf16, float>(s, M, h, x, gamma, eps, out, io, add, n_add, add_rows, assign);
    else rmsnorm_launch_t<bf16, bf16>(s, M, h, x, gamma, eps, out, io, add, n_add, add_rows, assign);
    return hipGetLastError();
}

__global__ void add_parts_k(int64_t count4, float4* __restrict__ x, const float4* __restrict__ parts, int n_parts, int assign) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count4; i += stride) {
        float4 v = assign ? make_float4(0.f, 0.f, 0.f, 0.f) : x[i];
        for (int k0 = 0; k0 < n_parts; k0 += 4) {
            float4 p[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = k0 + u < n_parts ? parts[(k0 + u) * count4 + i] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                v.x += p[u].x; v.y += p[u].y; v.z += p[u].z; v.w += p[u].w;
            }
        }
        x[i] = v;
    }
}

hipError_t add_parts(hipStream_t s, int64_t count, float* x, const float* parts, int n_parts, bool assign) {
    if (count <= 0 || n_parts <= 0) return hipSuccess;
    const int64_t c4 = count / 4;
    int blocks = (int)((c4 + 255) / 256);
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(add_parts_k, dim3(blocks), dim3(256), 0, s, c4, (float4*)x, (const float4*)parts, n_parts, (int)assign);
    return hipGetLastError();
}

hipError_t rope_kv_write(hipStream_t s, int dtype, const Rows& rows, const KVLayer& kv, void* qkv, int n_q_heads,
                         float theta, const void* bias, const RopeTable& tab, bool from_table, const float* src32, int n_src) {
    int M = rows.B * rows.n;
    if (M <= 0) return hipSuccess;
    // the kernel moves 16-byte pieces: rows of qkv and of the cache are multiples of 16 bytes by the
    // configuration check, the bases must be aligned as well
    if ((((uintptr_t)qkv | (uintptr_t)bias | (uintptr_t)kv.k | (uintptr_t)kv.v | (uintptr_t)src32 | (uintptr_t)tab.cs) & 15) != 0)
        return hipErrorInvalidValue;
    const int qkv_dim = (n_q_heads + 2 * kv.n_kv) * kv.d, vec = dtype == F32 ? 4 : 8;
    const int pieces = (n_q_heads + kv.n_kv) * (kv.d / 2 / vec) + kv.n_kv * kv.d / vec;
    const int threads = pieces >= kRopeThreads ? kRopeThreads : (pieces + 63) / 64 * 64;
    const size_t lds = from_table ? 0 : sizeof(float) * kv.d;
    const int64_t src_stride = (int64_t)M * qkv_dim;
#define TLT_ROPE(SRC, TBL)                                                                                                  \
    DISPATCH_T(dtype, hipLaunchKernelGGL((rope_kv_write_k<T, SRC, TBL>), dim3(M), dim3(threads), lds, s, src32, (T*)qkv, \
                                         (const int64_t*)tab.at, (const float*)tab.cs, src_stride, n_src, n_q_heads, kv.n_kv, kv.d,    \
                                         (const T*)bias, theta, rows, kv, tab))
    if (src32 && from_table) { TLT_ROPE(true, true); }
    else if (src32) { TLT_ROPE(true, false); }
    else if (from_table) { TLT_ROPE(false, true); }
    else { TLT_ROPE(false, false); }
#undef TLT_ROPE
    return hipGetLastError();
}

hipError_t swiglu(hipStream_t s, int dtype, int64_t count, const void* g, const void* u, void* out) {
    if (count <= 0) return hipSuccess;
    int blocks = (int)((count + 255) / 256);
    if (blocks > 16384) blocks = 16384;
    DISPATCH_T(dtype, hipLaunchKernelGGL(swiglu_k<T>, dim3(blocks), dim3(256), 0, s, count, (const T*)g, (const T*)u, (T*)out));
    return hipGetLastError();
}

hipError_t draft_input(hipStream_t s, int dtype, int B, int n, int h, int V, const int32_t* tok, const int32_t* src,
                       const int32_t* n_valid, int src_seq_stride, int64_t hidden_rows, const float* hidden,
                       const void* embed, void* xin) {
    if (B * n <= 0) return hipSuccess;
    const uintptr_t four = dtype == F32 ? 15 : 7;
    const bool vec = h % 4 == 0 && (((uintptr_t)embed | (uintptr_t)xin) & four) == 0 && ((uintptr_t)hidden & 15) == 0;
#define TLT_DRAFT_INPUT(VEC)                                                                                                     \
    DISPATCH_T(dtype, hipLaunchKernelGGL((draft_input_k<T, VEC>), dim3(B * n), dim3(256), 0, s, n, h, V, tok, src, n_valid,      \
                                         src_seq_stride, hidden_rows, hidden, (const T*)embed, (T*)xin))
    if (vec) { TLT_DRAFT_INPUT(true); }
    else { TLT_DRAFT_INPUT(false); }
#undef TLT_DRAFT_INPUT
    return hipGetLastError();
}

hipError_t add_i32(hipStream_t s, int n, int32_t* dst, const int32_t* a, int add_const) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(add_i32_k, dim3((n + 255) / 256), dim3(256), 0, s, n, dst, a, add_const);
    return hipGetLastError();
}

hipError_t report_words(hipStream_t s, int n, const int32_t* src, const unsigned int* status, int32_t* dst) {
    hipLaunchKernelGGL(report_words_k, dim3(n / 256 + 1), dim3(256), 0, s, n, src, status, dst);
    return hipGetLastError();
}

hipError_t copy_f32(hipStream_t s, int64_t count, const float* src, float* dst) {
    if (count <= 0) return hipSuccess;
    int64_t c4 = count / 4;  // callers pass multiples of 4 floats (hidden sizes are)
    int blocks = (int)((c4 + 255) / 256);
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(copy_f32_k, dim3(blocks), dim3(256), 0, s, c4, (const float4*)src, (float4*)dst);
    return hipGetLastError();
}

hipError_t zero_f32(hipStream_t s, int64_t count, float* dst) {
    if (count <= 0) return hipSuccess;
    int64_t c4 = count / 4;  // callers pass multiples of 4 floats
    int blocks = (int)((c4 + 255) / 256);
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(zero_f32_k, dim3(blocks), dim3(256), 0, s, c4, (float4*)dst);
    return hipGetLastError();
}

hipError_t gather_last_rows(hipStream_t s, int B, int n, int h, const float* src, float* dst, int dst_seq_stride) {
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_last_rows_k, dim3(B), dim3(256), 0, s, n, h / 4, (const float4*)src, (float4*)dst, dst_seq_stride);
    return hipGetLastError();
}

}  // namespace tlt

// C[M][N] (op)= A[M][K] . W[N][K]^T  -- every projection of the decoder block, the LM head and the
// drafter's input projection.  Both operands are K-contiguous, which is what the MFMA operand
// layout wants: a lane feeds 8 consecutive k values of one row.
//
// bf16 path (gfx950): v_mfma_f32_32x32x16_bf16, fp32 accumulation.  A workgroup of 4 waves (2x2)
// owns a (64*WTM) x (64*WTN) tile; each wave owns WTM x WTN MFMA tiles of 32x32.  K is walked in
// steps of 64 through rings of LDS slots (SA for the activation rows, SB for the weight rows) filled
// by direct global->LDS loads (no staging registers, no ds_write).  Workgroups are persistent: as
// many as the chip holds at once, each walking several tiles with the load pipeline running across
// tile boundaries; ids are remapped so that each XCD (ids are dealt round-robin over the 8 XCDs) walks
// a contiguous range of tiles, M fastest: neighbours on one XCD share the same weight tile in that
// XCD's L2.
// Measured on MI355X, and what shapes the kernel: a register-only MFMA loop with one wave per SIMD
// reaches ~2.0 PFLOP/s; the chip clocks down to ~1.6-1.8 GHz under sustained MFMA load; a CU's
// vector-memory front end moves ~50 B/clk of global->LDS traffic when rows are fetched as whole
// 128-byte lines (~110 GB/s per CU, half that for 64-byte pieces), so the 64 KB a 256x256 tile
// needs per K step occupy it for ~1300 of the step's 2048 MFMA clocks.  With the output stores
// switched off the 256x256 kernel runs at 1.34-1.42 PFLOP/s on the M = 1536 shapes; the stores of a
// tile are not overlapped with compute (all workgroups finish their tiles together and the burst
// runs at the HBM write rate, ~5-6 TB/s whatever the store shape), which costs 8-15 %.
//
// Generic path (fp32 mode, odd shapes): 64x64 LDS-tiled FMA kernel with full bounds checks.
#include "dev_common.h"
#include <cmath>
#include "kernels.h"

namespace tlt {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;  // 16-byte register vector (HIP's uint4 struct defeats SROA)

constexpr int kBK = 64;

template <int OUT>
__device__ __forceinline__ void store_out(void* C, int64_t idx, float v) {
    if (OUT == OUT_T)
        ((bf16*)C)[idx] = from_float<bf16>(v);
    else if (OUT == OUT_F32 || OUT == OUT_SPLIT_F32)
        ((float*)C)[idx] = v;
    else if (OUT == OUT_ADD_F32)
        ((float*)C)[idx] += v;
    else if (OUT == OUT_ATOMIC_ADD_F32)
        unsafeAtomicAdd((float*)C + idx, v);   // split-K partial sums: hardware fp32 add at the L2
}

constexpr uint32_t vmcnt_imm(int n) { return 0x0F70u | (uint32_t)(n & 15) | ((uint32_t)(n >> 4) << 14); }

// ------------------------------------------------------------------------------------------------
// The main loop is software-pipelined by hand.  What the schedule has to respect on this chip:
//  * one wave per SIMD issues in order, so anything that blocks the wave blocks its matrix pipe;
//  * the vector-memory front end accepts one 1 KB global->LDS wave instruction every ~20 clocks and
//    a wave that issues one while it is busy waits for its turn, so the loads are never issued as a
//    burst: every MFMA row (WTN MFMAs) is followed by exactly one load, all step long;
//  * a slot can only be refilled after the barrier that frees it and must have landed before the
//    barrier that publishes it.  The activation rows get one slot more than the weight rows (3 + 2
//    slots of 32 KB = the whole 160 KB LDS for a 256x256 tile): weight loads are issued in the first
//    half of that window and have the second half to land, activation loads are issued in the
//    second half and have a whole further step.
// Per K step t (four 16-wide slices, fragment register sets F0/F1):
//    slice 0 on F0 | LDS reads of slice 1 -> F1 | W tile t-1+SB, second half
//    slice 1 on F1 | LDS reads of slice 2 -> F0 | A tile t-1+SA, first half
//    slice 2 on F0 | LDS reads of slice 3 -> F1 | A tile t-1+SA, second half
//    wait for the reads and for tile t+1, barrier                 (tile t's slots are free from here)
//    slice 3 on F1 | LDS reads of (t+1, slice 0) -> F0 | W tile t+SB, first half
// so the last slice's MFMAs cover the barrier skew and the first reads of the next tile.  The loads
// are issued from inline assembly (buffer descriptor + 32-bit per-lane byte offset + scalar K offset) and waited for
// explicitly: the compiler does not see them and so cannot order them against the LDS reads with a
// full vmcnt(0).
// LDS layout: tile rows unpadded (128 B = 8 chunks of 16 B), chunk c of row r at c ^ ((r >> 1) & 7).
// The LDS has 64 banks (256 B per clock): a 16-byte fragment read is served 16 lanes at a time, and
// with this swizzle 16 consecutive rows hit 16 distinct 16-byte columns (SQ_LDS_BANK_CONFLICT = 0;
// swizzling with r & 7 instead costs a two-way conflict on every read).
__device__ __forceinline__ void dma_buf_16(u32x4_t rsrc, uint32_t voff_bytes, uint32_t soff_bytes,
                                           uint32_t lds_bytes) {
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :
                 : "v"(voff_bytes), "s"(rsrc), "s"(soff_bytes), "s"(lds_bytes)
                 : "memory", "m0");
}
// the same load marked non-temporal: for weight rows that no other workgroup reads, see NTW below
__device__ __forceinline__ void dma_buf_16_nt(u32x4_t rsrc, uint32_t voff_bytes, uint32_t soff_bytes,
                                              uint32_t lds_bytes) {
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen nt lds"
                 :
                 : "v"(voff_bytes), "s"(rsrc), "s"(soff_bytes), "s"(lds_bytes)
                 : "memory", "m0");
}

// GLU = true: the fused gate/up projection.  A workgroup's BN weight rows are BN/2 rows of W (gate)
// followed by the same BN/2 rows of W2 (up); each wave multiplies both halves for its columns and
// the epilogue stores silu(gate) * up, so C is [M][N] with N counting gate columns and the two
// intermediate matrices never exist.
// (The kernel's N is only the row stride of C: which column tiles exist is decided by total_tiles, and ncols,
// a multiple of 32, is where the launch's output columns end: the last column tile may reach past it.)
// NTW = true: the weight rows are fetched with the non-temporal hint.  For a single row of tiles that is not cut
// along K every weight row is read by one workgroup, once, and the hint keeps the stream from displacing what the
// caches hold of the activations and of the neighbouring kernels' data: the LM head at 40-256 rows 5-8 % faster
// (233 -> 221 us, 207 -> 193), gate/up at 256 rows 2-3 %, the small kernels around them 1-4 %.  With several row
// tiles per weight tile, or with K cuts, the same hint costs 1-5 % (o projection at 1536 rows 46.7 -> 48.1 us, the
// down projection's 8 cuts at 256 rows 45.2 -> 47.6): those launches do not take it, except the K cuts of 128x128
// tiles at up to 128 rows (one row of tiles: 14.8 -> 14.1 us at 40 rows, plain decoding at batch 32 5.60 -> 5.56 ms).
// (Kernel traces of both builds on one box.)
template <int WGM, int WGN, int WTM, int WTN, int SA, int SB, int OUT, bool GLU = false, bool NTW = false>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_pipe_k(int M, int N, int K, const uint16_t* __restrict__ A,
                                                        const uint16_t* __restrict__ W, const uint16_t* __restrict__ W2,
                                                        void* __restrict__ C, int nbm, int total_tiles, int per_xcd,
                                                        int ksplit, int wg_per_xcd, int32_t* __restrict__ C2, int kskew,
                                                        int64_t split_stride, int ncols) {
    constexpr int NW = WGM * WGN;
    constexpr int BKS = 64;
    constexpr int BM = 32 * WTM * WGM, BN = 32 * WTN * WGN;
    constexpr int ASZ = BM * BKS, BSZ = BN * BKS;      // elements per A slot / W slot
    constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW;  // 1 KB DMA instructions per wave per tile: A part, W part
    constexpr int NR = WTM + WTN;                     // fragment reads per slice
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile rows must split evenly over the waves");
    static_assert(LA % 2 == 0 && WTM >= 2, "schedule: each operand's loads are split over two slices");
    static_assert(SA >= 2 && SB >= 2, "at least double buffering");
    constexpr int RQ = (NR + WTM / 2 - 1) / (WTM / 2);   // fragment reads issued by each of the first WTM/2 MFMA rows
    // loads that may still be in flight when tile t+1 must be complete: those issued after its A part (each step issues W, then A) and
    // after its W part, fewest for W tile 1, which the prologue issues after the A tiles (later ones have (SB - 1) * LA + (SB - 2) * LB behind
    // them).  Loads retire in order, so slots of one operand beyond what the other's ring allows keep nothing more in flight.
    constexpr int kInFlightA = (SA - 2) * (LA + LB), kInFlightB = LA + (SB - 2) * LB;
    constexpr int kInFlight = kInFlightA < kInFlightB ? kInFlightA : kInFlightB;
    constexpr int BNO = GLU ? BN / 2 : BN;            // output columns per workgroup
    // widths that do not divide the 128 columns every launch is a multiple of: the last column tile may be partial
    constexpr bool kPartialN = BNO % 64 != 0;
    static_assert(!GLU || NW % 2 == 0, "gate and up halves split over waves");
    // GLU with an odd number of column tiles: each is 16 gate rows and the 16 up rows that belong to them (else a wave's
    // first column tiles are gate rows, as many up rows follow)
    constexpr bool kMixed = GLU && WTN % 2 != 0;
    static_assert(!kMixed || (WGN == 1 && BNO % 16 == 0), "one wave across the columns, swizzle of the up half as the gate half's");
    extern __shared__ __align__(16) uint16_t lds[];   // SA A slots, then SB W slots

    // Persistent workgroups: XCD x (ids are dealt round-robin over the XCDs) owns the logical tiles
    // x*per_xcd .. (x+1)*per_xcd-1 and its wg_per_xcd workgroups walk them with that stride, so at any
    // time an XCD works on a contiguous run of tiles (M fastest: neighbours share a weight tile in L2).
    // The K steps of all of a workgroup's tiles form one sequence that the slot rings run through
    // without draining: while the last steps of a tile compute, the first K tiles of the next one load.
    const int pid = blockIdx.x;
    const int xcd = pid & 7, wslot = pid >> 3;
    const int first = xcd * per_xcd + wslot;
    int range_end = total_tiles - xcd * per_xcd;
    range_end = range_end < per_xcd ? range_end : per_xcd;
    if (wslot >= range_end) return;
    const int n_my = (range_end - wslot + wg_per_xcd - 1) / wg_per_xcd;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    const int l32 = lane & 31, lhi = lane >> 5;
    const int nk_all = K / BKS;
    const bool up_wave = GLU && wave >= NW / 2;

    // tile j of this workgroup: M fastest, then N, then the K split.  An XCD's run of tiles then lies in one K split
    // (or two): its workgroups walk the same K range together and share the activation K tiles in its L2, where
    // with the split inside N every XCD would fetch the activation rows of every K range.
    struct TileInfo { int m0, n0, kt0, nt, split; };
    const int nbn_all = total_tiles / (nbm * ksplit);
    auto tile_info = [&](int j) {
        const int logical = first + j * wg_per_xcd;
        const int tile_m = logical % nbm, tile_n = (logical / nbm) % nbn_all, split = logical / (nbm * nbn_all);
        TileInfo ti;
        // (integer division runs on the vector ALU: pin the uniform results back into scalar registers)
        ti.m0 = __builtin_amdgcn_readfirstlane(tile_m * BM);
        ti.n0 = __builtin_amdgcn_readfirstlane(tile_n * BNO);
        // K tiles of split i: an even cut, or (kskew > 0) lengths that rise linearly from the mean - kskew
        // to the mean + kskew, so that the splits of a one-round launch end at different times and the
        // partial tiles of the early ones are added while the others still multiply
        auto kbound = [&](int i) {   // (nk_all * ksplit < 2^31 by the shape check)
            int k = nk_all * i / ksplit;
            if (kskew > 0) k += kskew * (i * (i - 1) - i * (ksplit - 1)) / (ksplit - 1);
            return k;
        };
        ti.kt0 = __builtin_amdgcn_readfirstlane(kbound(split));
        ti.nt = __builtin_amdgcn_readfirstlane(kbound(split + 1)) - ti.kt0;
        ti.split = __builtin_amdgcn_readfirstlane(split);
        return ti;
    };
    // raw buffer descriptors (four scalar words: base, base high bits, size in bytes, format) over a
    // tile's two row panels.  The activation panel's size is its valid rows: lanes that would fetch rows
    // past M are out of range and fetch nothing (their accumulator rows are never stored).  Every
    // in-range offset is below 2^31 by the launcher's shape check.
    auto desc = [&](const uint16_t* base, uint32_t bytes) {
        const uint64_t p = (uint64_t)(uintptr_t)base;
        u32x4_t d;
        d[0] = __builtin_amdgcn_readfirstlane((uint32_t)p);
        d[1] = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32) & 0xffffu);
        d[2] = bytes;
        d[3] = 0x00020000u;
        return d;
    };
    auto desc_a = [&](const TileInfo& ti) {
        int rows = M - ti.m0;
        rows = rows < BM ? rows : BM;
        return desc(A + (int64_t)ti.m0 * K, (uint32_t)(rows * K * 2));
    };
    // (GLU: the first half of the waves fetch the gate rows, the second half the up rows; a wave's
    // LB blocks are BN / NW consecutive tile rows, so they never straddle the two halves)
    // Where the last column tile of a launch may be partial (kPartialN), the weight panel's size is its valid rows
    // as well: rows past ncols fetch nothing, and the columns they would make are never stored.
    auto desc_b = [&](const TileInfo& ti) {
        const uint16_t* base = up_wave ? W2 + ((int64_t)ti.n0 - BN / 2) * K : W + (int64_t)ti.n0 * K;
        if constexpr (!kPartialN) return desc(base, 0x7fffffffu);
        int cols = ncols - ti.n0;
        cols = cols < BNO ? cols : BNO;
        return desc(base, (uint32_t)(((up_wave ? BN / 2 : 0) + cols) * K * 2));
    };

    // DMA addressing: wave w fills 1 KB blocks w*LA .. of an A slot (8 tile rows each) and w*LB .. of
    // a W slot; lane -> (row r of the block, stored chunk c) fetches the logical chunk that the
    // swizzle places there
    const int r = lane >> 3, c = lane & 7;
    uint32_t offA[LA], offB[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int trow = (wave * LA + i) * 8 + r;
        offA[i] = ((uint32_t)trow * (uint32_t)K + (c ^ ((trow >> 1) & 7)) * 8) * 2u;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int trow = (wave * LB + i) * 8 + r;
        offB[i] = ((uint32_t)trow * (uint32_t)K + (c ^ ((trow >> 1) & 7)) * 8) * 2u;
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)lds;
    const uint32_t lds_waveA = lds_base + (uint32_t)(wave * LA) * 1024u;
    const uint32_t lds_waveB = lds_base + (uint32_t)(SA * ASZ * 2) + (uint32_t)(wave * LB) * 1024u;

    // load cursors: the next K tile each operand fetches, in the order the compute side consumes them
    // (descriptor, absolute K tile index, end of the tile's K range).  When a cursor reaches the end of
    // its tile it jumps to the `next` triple, which the compute loop points at its following tile, or,
    // after the last one, at an empty descriptor (loads that fetch nothing keep the schedule uniform, see gemm_bf16_few_k).  All
    // of it is scalar selects: the K loop stays one basic block.  A cursor runs at most SA-1 (SB-1) K
    // tiles ahead, so with at least max(SA, SB) K tiles per tile (the launcher's condition for giving a workgroup
    // more than one) it never needs more than the one following tile.
    const TileInfo ti0 = tile_info(0);
    u32x4_t rsA = desc_a(ti0), rsB = desc_b(ti0), rsA_nx = rsA, rsB_nx = rsB;
    int a_kt = ti0.kt0, a_end = ti0.kt0 + ti0.nt, b_kt = a_kt, b_end = a_end;
    int nx_kt0 = a_end - 1, nx_end = a_end;
    uint32_t kA2 = (uint32_t)a_kt * (BKS * 2), kB2 = kA2;   // byte offset of the cursor's K tile in a row
    auto advance_a = [&]() {
        ++a_kt;
        const bool wrap = a_kt == a_end;
#pragma unroll
        for (int w = 0; w < 3; ++w) rsA[w] = wrap ? rsA_nx[w] : rsA[w];
        a_kt = wrap ? nx_kt0 : a_kt;
        a_end = wrap ? nx_end : a_end;
        kA2 = (uint32_t)a_kt * (BKS * 2);
    };
    auto advance_b = [&]() {
        ++b_kt;
        const bool wrap = b_kt == b_end;
#pragma unroll
        for (int w = 0; w < 3; ++w) rsB[w] = wrap ? rsB_nx[w] : rsB[w];
        b_kt = wrap ? nx_kt0 : b_kt;
        b_end = wrap ? nx_end : b_end;
        kB2 = (uint32_t)b_kt * (BKS * 2);
    };
    // point `next` at tile j+1 (call while both cursors are inside tile j)
    auto set_next = [&](int j, const TileInfo& tj) {
        if (j + 1 < n_my) {
            const TileInfo tn = tile_info(j + 1);
            rsA_nx = desc_a(tn);
            rsB_nx = desc_b(tn);
            nx_kt0 = tn.kt0;
            nx_end = tn.kt0 + tn.nt;
        } else {
            rsA_nx[2] = rsB_nx[2] = 0u;
            nx_kt0 = tj.kt0 + tj.nt - 1;
            nx_end = tj.kt0 + tj.nt;
        }
    };
    set_next(0, ti0);

#define TLT_DMA_A(slot, d) dma_buf_16(rsA, offA[d], kA2, lds_waveA + (uint32_t)((slot) * ASZ * 2 + (d) * 1024));
#define TLT_DMA_B(slot, d)                                                                                        \
    {                                                                                                             \
        if constexpr (NTW) dma_buf_16_nt(rsB, offB[d], kB2, lds_waveB + (uint32_t)((slot) * BSZ * 2 + (d) * 1024)); \
        else dma_buf_16(rsB, offB[d], kB2, lds_waveB + (uint32_t)((slot) * BSZ * 2 + (d) * 1024));                \
    }

    f32x16_t acc[WTM][WTN];
#pragma unroll
    for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int j = 0; j < WTN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // prologue: K tile 0 first, then A tiles 1 .. SA-2, W tiles 1 .. SB-2 and the first half of W tile SB-1
#pragma unroll
    for (int d = 0; d < LA; ++d) TLT_DMA_A(0, d)
    advance_a();
#pragma unroll
    for (int d = 0; d < LB; ++d) TLT_DMA_B(0, d)
    advance_b();
#pragma unroll
    for (int st = 1; st < SA - 1; ++st) {
#pragma unroll
        for (int d = 0; d < LA; ++d) TLT_DMA_A(st, d)
        advance_a();
    }
#pragma unroll
    for (int st = 1; st < SB - 1; ++st) {
#pragma unroll
        for (int d = 0; d < LB; ++d) TLT_DMA_B(st, d)
        advance_b();
    }
#pragma unroll
    for (int d = 0; d < LB / 2; ++d) TLT_DMA_B(SB - 1, d)

    const int fragA = (wm * (WTM * 32) + l32) * BKS;
    // tile row of column tile j of this wave (GLU: j < WTN/2 are gate rows, the rest the matching up rows)
    auto colrow = [&](int j) {
        return kMixed ? j * 16 : GLU ? (j / (WTN / 2)) * (BN / 2) + (j % (WTN / 2)) * 32 : j * 32;
    };
    const int fragB = (kMixed ? (l32 & 15) + (l32 >> 4) * (BN / 2) : (GLU ? wn * (WTN / 2 * 32) : wn * (WTN * 32)) + l32) * BKS;
    const int sw = (l32 >> 1) & 7;   // (rows 16 apart, and the two halves, share their swizzle)

    bf16x8_t fa[2][WTM], fb[2][WTN];
    // read q of a slice's NR fragment reads: the W fragments first (every MFMA row needs them all)
#define TLT_READ1(buf, pa, pb, kk, q)                                                                             \
    {                                                                                                             \
        const int ch = ((2 * (kk) + lhi) ^ sw) * 8;                                                               \
        if ((q) < WTN) fb[buf][q] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)((pb) + fragB + colrow(q) * BKS + ch)); \
        else fa[buf][(q) - WTN] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)((pa) + fragA + ((q) - WTN) * 32 * BKS + ch)); \
    }
#define TLT_MFMA(buf, i, j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[buf][i], fb[buf][j], acc[i][j], 0, 0, 0);
    // one slice: the MFMA rows on fragment set `buf`; the reads of the next slice into the other set
    // in its first rows; the H loads base .. base+H-1 of operand OP (0 = A, 1 = W) spread evenly
    // over the rows, each issued after its row's MFMAs.  Odd rows run their columns backwards, so that
    // consecutive MFMAs always share one operand (the launches run against the power limit: 0.4 % of
    // the verification GEMMs' time, measured)
#define TLT_SLICE(buf, pa, pb, rkk, OP, slot, base, H)                                                            \
    _Pragma("unroll") for (int i = 0; i < WTM; ++i) {                                                              \
        if (i < WTM / 2) {                                                                                        \
            _Pragma("unroll") for (int q = i * RQ; q < (i + 1) * RQ && q < NR; ++q) TLT_READ1((buf) ^ 1, pa, pb, rkk, q) \
        }                                                                                                         \
        _Pragma("unroll") for (int j = 0; j < WTN; ++j) TLT_MFMA(buf, i, ((i & 1) ? WTN - 1 - j : j))              \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
        _Pragma("unroll") for (int d = (i * (H)) / WTM; d < ((i + 1) * (H)) / WTM; ++d) {                          \
            if ((OP) == 0) TLT_DMA_A(slot, (base) + d) else TLT_DMA_B(slot, (base) + d)                            \
        }                                                                                                         \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
    }

    __builtin_amdgcn_s_waitcnt(vmcnt_imm((SA - 2) * LA + (SB - 2) * LB + LB / 2));   // K tile 0 has landed
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int q = 0; q < NR; ++q) TLT_READ1(0, lds, lds + SA * ASZ, 0, q)

    // slot of the current K tile in each ring; pa_/pb_ = slot of the one before (refilled during this step)
    int sa = 0, sb = 0, pa_ = SA - 1, pb_ = SB - 1;
    for (int j = 0; j < n_my; ++j) {
        const TileInfo ti = tile_info(j);
        if (j > 0) set_next(j, ti);
        for (int t = 0; t < ti.nt; ++t) {
            const uint16_t* pa = lds + sa * ASZ;
            const uint16_t* pb = lds + SA * ASZ + sb * BSZ;
            const int na = sa + 1 == SA ? 0 : sa + 1, nb = sb + 1 == SB ? 0 : sb + 1;
            // the first slice's fragments were requested a whole slice ago; waiting here, before the next
            // reads are issued, keeps the compiler from waiting for those as well
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            TLT_SLICE(0, pa, pb, 1, 1, pb_, LB / 2, LB - LB / 2)      // W cursor, second half
            advance_b();
            TLT_SLICE(1, pa, pb, 2, 0, pa_, 0, LA / 2)                // A cursor, first half
            TLT_SLICE(0, pa, pb, 3, 0, pa_, LA / 2, LA / 2)           //           second half
            advance_a();
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(kInFlight));        // the next K tile has landed
            __builtin_amdgcn_s_barrier();                            // ... for every wave; this one's slots are free
            __builtin_amdgcn_sched_barrier(0);
            TLT_SLICE(1, lds + na * ASZ, lds + SA * ASZ + nb * BSZ, 0, 1, sb, 0, LB / 2)   // W cursor, first half
            pa_ = sa; pb_ = sb; sa = na; sb = nb;
        }
        // the tile is complete: store it and clear the accumulators while the next tile's loads land
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (OUT == OUT_ROWMAX) {
            // best (value, column) of each of this wave's WTM*32 rows over its WTN*32 columns: first over a
            // lane's own WTN columns of the row, then across the 32 lanes that hold the row's other
            // columns.  That second reduction is a reduce-scatter: every exchange halves the rows a lane
            // still carries, so it costs 2*NV exchanges instead of 5*NV; a lane ends with rows
            // k = lane32*NV/32 .. of the wave's NV = WTM*16 (row index k = i*16 + v within its half).
            constexpr int NV = WTM * 16;
            const int col0 = (int)split_stride + ti.n0;   // (this launch's first column in the whole product, no cuts here)
            float bv[NV];
            int bi[NV];
#pragma unroll
            for (int i = 0; i < WTM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float m = acc[i][0][v];
                    int mi = col0 + wn * (WTN * 32) + l32;
#pragma unroll
                    for (int jj = 1; jj < WTN; ++jj)
                        if (acc[i][jj][v] > m) {   // strictly greater: the lower column wins a tie
                            m = acc[i][jj][v];
                            mi = col0 + wn * (WTN * 32) + jj * 32 + l32;
                        }
                    bv[i * 16 + v] = m;
                    bi[i * 16 + v] = mi;
                }
#pragma unroll
            for (int H = NV / 2, mask = 16; mask >= 1; H >>= 1, mask >>= 1) {
                const bool upper = (l32 & mask) != 0;   // this lane keeps the upper half of what it carries
#pragma unroll
                for (int k = 0; k < (H > 0 ? H : 1); ++k) {
                    if (H > 0) {
                        const float send_v = upper ? bv[k] : bv[k + H];
                        const int send_i = upper ? bi[k] : bi[k + H];
                        const float keep_v = upper ? bv[k + H] : bv[k];
                        const int keep_i = upper ? bi[k + H] : bi[k];
                        const float ov = __shfl_xor(send_v, mask, 64);
                        const int oi = __shfl_xor(send_i, mask, 64);
                        const bool take = ov > keep_v || (ov == keep_v && oi < keep_i);
                        bv[k] = take ? ov : keep_v;
                        bi[k] = take ? oi : keep_i;
                    }
                }
            }
            constexpr int PER = NV / 32;   // rows a lane ends with
            const int P = N;               // partial blocks per row of the whole product
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                const int k = l32 * PER + e, i = k >> 4, v = k & 15;
                const int row = ti.m0 + wm * (WTM * 32) + i * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3);
                if (row < M) {
                    const int64_t o = (int64_t)row * P + ti.n0 / (WTN * 32) + wn;
                    ((float*)C)[o] = bv[e];
                    C2[o] = bi[e];
                }
            }
        } else if constexpr (kMixed && OUT == OUT_T) {
            // Lanes l and l + 16 of a half-wave hold gate and up of one column.  Swapping the odd 16-lane rows of one
            // accumulator with the even ones of the next gives both to one lane: the lower lane row v, the upper one
            // row v + 1.  Neighbouring lanes then trade a value, so that each stores two adjacent columns.
            const int odd16 = (l32 >> 4) & 1, odd = lane & 1;
#pragma unroll
            for (int i = 0; i < WTM; ++i)
#pragma unroll
                for (int jj = 0; jj < WTN; ++jj)
#pragma unroll
                    for (int vq = 0; vq < 4; ++vq) {
                        float r[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            float x0, x1;   // (see below: out of their registers here, not all at once)
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x0) : "a"(acc[i][jj][4 * vq + 2 * e]));
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x1) : "a"(acc[i][jj][4 * vq + 2 * e + 1]));
                            const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
                            const float g = __uint_as_float(p[0]), u = __uint_as_float(p[1]);
                            r[e] = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
                        }
                        // r[0]: row 4 vq + odd16, r[1]: two rows on; even lanes keep the first, odd ones the second
                        const float other = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(odd ? r[0] : r[1]), 0xB1, 0xF, 0xF, false));
                        const uint32_t out = odd ? pack_bf16x2(other, r[1]) : pack_bf16x2(r[0], other);
                        const int row = ti.m0 + wm * (WTM * 32) + i * 32 + 8 * vq + 4 * lhi + 2 * odd + odd16;
                        const int col0 = ti.n0 + jj * 16;   // (ncols is a multiple of 16: a block is valid or not as a whole)
                        if (row < M && (!kPartialN || col0 < ncols)) *(uint32_t*)((bf16*)C + (int64_t)row * N + col0 + (l32 & 14)) = out;
                        __builtin_amdgcn_sched_barrier(0);
                    }
        } else if constexpr (GLU && OUT == OUT_T) {
            // A lane holds one column of four consecutive rows (v = 4 vq .. 4 vq + 3) of each 32x32 block: stored
            // as they lie, that is 2 bytes per lane and store instruction, and the tile's 512 of those cost
            // more than its arithmetic.  The four lanes of a quad trade values instead (two exchanges of fp32 with
            // the neighbour, one of a packed pair with the lane two over) until each holds four adjacent
            // columns of one row, and stores them as 8 bytes (gate/up at M = 1536: 408 -> 394 us, at M = 128: 95 -> 88;
            // the same trade for fp32 output, or for a plain bf16 product, gains nothing: measured).
            const int q4 = lane & 3;
            const bool odd = (q4 & 1) != 0, hi2 = (q4 & 2) != 0;
            auto swap1 = [](float x) {   // value of the neighbouring lane (quad permutation 1, 0, 3, 2)
                return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));
            };
            auto swap2 = [](uint32_t x) {   // value of the lane two over (quad permutation 2, 3, 0, 1)
                return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false);
            };
#pragma unroll
            for (int i = 0; i < WTM; ++i) {
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    const int row = ti.m0 + wm * (WTM * 32) + i * 32 + 8 * vq + 4 * lhi + q4;   // the row this lane stores
#pragma unroll
                    for (int jj = 0; jj < WTN / 2; ++jj) {
                        float r[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            // (the accumulators leave their registers here and nowhere earlier: left to itself the
                            // compiler copies most of the tile out first and spills)
                            float g, u;
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(g) : "a"(acc[i][jj][4 * vq + e]));
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(u) : "a"(acc[i][jj + WTN / 2][4 * vq + e]));
                            // (hardware reciprocal, 1 ulp: the result is rounded to bf16 anyway, and an IEEE division
                            // per element costs the tile epilogue several microseconds)
                            r[e] = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
                        }
                        // rows 0/1 and 2/3: an even lane keeps the lower row and gets the neighbour's column of it
                        const float n01 = swap1(odd ? r[0] : r[1]), n23 = swap1(odd ? r[2] : r[3]);
                        const uint32_t w01 = odd ? pack_bf16x2(n01, r[1]) : pack_bf16x2(r[0], n01);
                        const uint32_t w23 = odd ? pack_bf16x2(n23, r[3]) : pack_bf16x2(r[2], n23);
                        // lanes 0/1 of the quad keep rows 0/1, lanes 2/3 rows 2/3; the other pair of columns comes over
                        const uint32_t other = swap2(hi2 ? w01 : w23);
                        uint2 out;
                        out.x = hi2 ? other : w01;
                        out.y = hi2 ? w23 : other;
                        const int col0 = ti.n0 + wn * (WTN / 2 * 32) + jj * 32;   // (a 32-column block is valid or not as a whole)
                        if (row < M && (!kPartialN || col0 < ncols)) *(uint2*)((bf16*)C + (int64_t)row * N + col0 + (l32 & ~3)) = out;
                        // (keeps the compiler from fetching all accumulators first: that spills, and a reload from
                        // scratch waits for every load in flight, the next tile's first K tiles included)
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        } else {
#pragma unroll
        for (int i = 0; i < WTM; ++i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int row = ti.m0 + wm * (WTM * 32) + i * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3);
                if (row < M) {
                    if (GLU) {
#pragma unroll
                        for (int jj = 0; jj < WTN / 2; ++jj) {
                            const int col0 = ti.n0 + wn * (WTN / 2 * 32) + jj * 32;
                            if (kPartialN && col0 >= ncols) continue;
                            int col = col0 + l32;
                            const float g = acc[i][jj][v], u = acc[i][jj + WTN / 2][v];
                            // (hardware reciprocal, 1 ulp: the result is rounded to bf16 anyway, and an IEEE division
                            // per element costs the tile epilogue several microseconds)
                            store_out<OUT>(C, (int64_t)row * N + col, g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u);
                        }
                    } else {
#pragma unroll
                        for (int jj = 0; jj < WTN; ++jj) {
                            const int col0 = ti.n0 + wn * (WTN * 32) + jj * 32;
                            if (kPartialN && col0 >= ncols) continue;
                            int col = col0 + l32;
                            store_out<OUT>(C, (OUT == OUT_SPLIT_F32 ? (int64_t)ti.split * split_stride : (int64_t)0) + (int64_t)row * N + col,
                                           acc[i][jj][v]);
                        }
                    }
                }
            }
        }
        }
#pragma unroll
        for (int i = 0; i < WTM; ++i)
#pragma unroll
            for (int jj = 0; jj < WTN; ++jj)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][jj][v] = 0.f;
    }
#undef TLT_READ1
#undef TLT_MFMA
#undef TLT_SLICE
#undef TLT_DMA_A
#undef TLT_DMA_B
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // drain the redundant tail fetches before the LDS is released
}

template <typename T, int OUT>
__device__ __forceinline__ void store_out_t(void* C, int64_t idx, float v) {
    if (OUT == OUT_T)
        ((T*)C)[idx] = from_float<T>(v);
    else if (OUT == OUT_F32)
        ((float*)C)[idx] = v;
    else
        ((float*)C)[idx] += v;
}

template <typename T, int OUT>
__global__ __launch_bounds__(256) void gemm_generic_k(int M, int N, int K, const T* __restrict__ A,
                                                      const T* __restrict__ W, void* __restrict__ C) {
    __shared__ float As[16][65], Ws[16][65];
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int idx = tid + i * 256, row = idx >> 4, k = idx & 15;
            int gm = m0 + row, gn = n0 + row, gk = k0 + k;
            As[k][row] = (gm < M && gk < K) ? to_float(A[(int64_t)gm * K + gk]) : 0.f;
            Ws[k][row] = (gn < N && gk < K) ? to_float(W[(int64_t)gn * K + gk]) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            float a[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = As[k][ty * 4 + i];
                w[i] = Ws[k][tx * 4 + i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int row = m0 + ty * 4 + i;
        if (row >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int col = n0 + tx * 4 + j;
            if (col < N) store_out_t<T, OUT>(C, (int64_t)row * N + col, acc[i][j]);
        }
    }
}

// fp32 products of few rows (fp32 mode up to kF32FewRows rows).  What bounds them is latency: a tiny decoder's
// products are a few hundred kilobytes, and a 64x64 tile walks K in steps of 16 with a barrier each while a handful of
// workgroups run.  Here a workgroup owns 16 weight rows x 16 T activation rows, its four waves take every fourth piece of 16
// k, each straight from memory into the operands of v_mfma_f32_16x16x4_f32 (fp32 in, fp32 accumulation; a lane holds
// 4 consecutive k of its row, and which k an instruction's four slots mean is the same for both operands), and add
// their sums through LDS: as many workgroups as the width allows, no barrier in the K loop and all its loads in flight.
// Measured against the 64x64 tiles below (us per call): M 2, N 1024, K 256: 28.0 -> 4.6; M 16, N 256, K 768: 81 -> 5.1; M 64,
// N 512, K 1280: 151 -> 6.9; M 16, N = K = 3584: 474 -> 16; M 256, N = K = 3584: 565 -> 163 (linear in the rows from there).
// GLU: W2 is the up matrix, C = silu(A W^T) * (A W2^T).
// NORM: the rows of A are made here: every workgroup normalises its (at most 16) rows into LDS, and the first one of a row block leaves the
// rows it read, the addend absorbed, for the next reader of the stream.  A tiny decoder's step is as long as its launches are many: a norm of
// its own costs a launch of 2.9 us on the host and 2.5-3 us of the chip, here it is 8 KB per workgroup from the caches.
typedef __attribute__((ext_vector_type(4))) float f32x4v_t;
template <int T, int OUT, bool GLU, bool NORM = false>
__global__ __launch_bounds__(256) void gemm_f32_few_k(int M, int N, int K, const float* __restrict__ A, const float* __restrict__ W,
                                                      const float* __restrict__ W2, float* __restrict__ C, NormIn ni) {
    constexpr int NG = GLU ? 2 : 1, U = 4;   // U: pieces whose loads are issued together
    static_assert(!NORM || T == 1, "the normalised rows of one 16-row block fit the LDS");
    __shared__ __align__(16) float red[4][NG][T][256];
    extern __shared__ __align__(16) float xn_s[];   // NORM: [16][K + 4]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16 * T;
    // rows past the edges read the last row: their results are not stored
    const int wrow = n0 + l16 < N ? n0 + l16 : N - 1;
    const float* wp[NG];
    wp[0] = W + (int64_t)wrow * K + 4 * g;
    if constexpr (GLU) wp[1] = W2 + (int64_t)wrow * K + 4 * g;
    const float* ap[T];   // (NORM: A is null and nothing is read through it)
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int row = m0 + 16 * t + l16;
        ap[t] = A + (int64_t)(row < M ? row : M - 1) * K + 4 * g;
    }
    if constexpr (NORM) {
        // a wave per row, four rows each; K <= 1024: at most four 16-byte pieces per lane (the launcher checks).  All rows are requested before the
        // first is summed: one after the other, every four rows cost a trip to the caches per product (a forward of 8 blocks of 1024 elements,
        // us: 8 rows 328 -> 296, 12 rows 365 -> 311, 16 rows 396 -> 326)
        f32x4v_t v[4][4], add[4][4], gam[4];
        const f32x4v_t zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = m0 + wave + 4 * q;   // (wave-uniform; rows past the end are never stored, what their LDS holds does not matter)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = 4 * lane + 256 * u;
                const bool on = r < M && c < K;
                v[q][u] = on && !(ni.add && ni.assign) ? *(const f32x4v_t*)(ni.x + (int64_t)r * K + c) : zero;
                add[q][u] = on && ni.add ? *(const f32x4v_t*)(ni.add + (int64_t)r * K + c) : zero;
                if (q == 0) gam[u] = c < K ? *(const f32x4v_t*)(ni.gamma + c) : zero;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = m0 + wave + 4 * q;
            if (r >= M) break;
            float ss = 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (ni.add) v[q][u] += add[q][u];
                ss += v[q][u][0] * v[q][u][0] + v[q][u][1] * v[q][u][1] + v[q][u][2] * v[q][u][2] + v[q][u][3] * v[q][u][3];
            }
            const float inv = 1.0f / sqrtf(wave_sum(ss) / (float)K + ni.eps);
            float* keep = blockIdx.x == 0 && ni.x_out ? ni.x_out + ((int64_t)(r / ni.out_n) * ni.out_stride + ni.out_base + r % ni.out_n) * K : nullptr;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = 4 * lane + 256 * u;
                if (c >= K) continue;
                *(f32x4v_t*)(xn_s + (wave + 4 * q) * (K + 4) + c) = v[q][u] * inv * gam[u];
                if (keep) *(f32x4v_t*)(keep + c) = v[q][u];
            }
        }
        __syncthreads();
    }
    f32x4v_t acc[NG][T];
#pragma unroll
    for (int i = 0; i < NG; ++i)
#pragma unroll
        for (int t = 0; t < T; ++t) acc[i][t] = f32x4v_t{0.f, 0.f, 0.f, 0.f};
    for (int k0 = wave * 16; k0 < K; k0 += 64 * U) {
        f32x4v_t w[U][NG], a[U][T];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 64 * u;
            const bool on = k + 4 * g < K;   // (K % 4 == 0: a lane's four values are in range or not as a whole)
#pragma unroll
            for (int i = 0; i < NG; ++i) w[u][i] = on ? *(const f32x4v_t*)(wp[i] + k) : f32x4v_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if constexpr (NORM) a[u][t] = on ? *(const f32x4v_t*)(xn_s + l16 * (K + 4) + 4 * g + k) : f32x4v_t{0.f, 0.f, 0.f, 0.f};
                else a[u][t] = on ? *(const f32x4v_t*)(ap[t] + k) : f32x4v_t{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < NG; ++i)
#pragma unroll
                    for (int t = 0; t < T; ++t)
                        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][i][e], a[u][t][e], acc[i][t], 0, 0, 0);
    }
    // a lane holds weight rows 4g .. 4g+3 of activation row l16: [activation row][weight row] in LDS
#pragma unroll
    for (int i = 0; i < NG; ++i)
#pragma unroll
        for (int t = 0; t < T; ++t) *(f32x4v_t*)&red[wave][i][t][l16 * 16 + 4 * g] = acc[i][t];
    __syncthreads();
    const int row16 = threadIdx.x >> 4, col = n0 + (threadIdx.x & 15);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int row = m0 + 16 * t + row16;
        if (row >= M || col >= N) continue;
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) v += red[q][0][t][threadIdx.x];
        if constexpr (GLU) {
            float u = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) u += red[q][NG - 1][t][threadIdx.x];
            v = v / (1.0f + expf(-v)) * u;
        }
        store_out_t<float, OUT>(C, (int64_t)row * N + col, v);
    }
}

constexpr int kF32FewRows = 256;
static bool f32_few_ok(int M, int K, const void* A, const void* W, const void* W2 = nullptr) {
    return M <= kF32FewRows && K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W | (uintptr_t)W2) & 15) == 0;
}
// Where the 64x64 tiles are many, no workgroup waits for the others any more and they share their rows through LDS: from
// 1500 of them above 96 rows, and from 512 above 32 rows where K is one step of a wave (us, few-row and tiled kernel on the same
// buffers: M 256, N 152064, K 896: 1875 and 1506; M 256, N 32000, K 2048: 803 and 724; M 160, N 152064, K 64: 159 and 92; on the
// other side M 256, N 16000, K 896: 184 and 203; M 65, N 64000, K 256: 79 and 95).  The fused gate/up
// product saves an activation kernel besides and stays (M 256, N 32768, K 896: 582 against two products of 341).
static bool f32_tiles_pay(int M, int N, int K) {
    const int64_t tiles = (int64_t)((N + 63) / 64) * ((M + 63) / 64);
    return M > 32 && (K <= 64 ? tiles >= 512 : M > 96 && tiles >= 1500);
}
template <int T>
static hipError_t launch_f32_few_t(hipStream_t s, int out_mode, int M, int N, int K, const void* A, const void* W, const void* W2, void* C) {
    const dim3 grid((N + 15) / 16, (M + 16 * T - 1) / (16 * T)), block(256);
    const float *a = (const float*)A, *w = (const float*)W, *w2 = (const float*)W2;
    if (W2) hipLaunchKernelGGL((gemm_f32_few_k<T, OUT_F32, true>), grid, block, 0, s, M, N, K, a, w, w2, (float*)C, NormIn());
    else if (out_mode == OUT_ADD_F32) hipLaunchKernelGGL((gemm_f32_few_k<T, OUT_ADD_F32, false>), grid, block, 0, s, M, N, K, a, w, w2, (float*)C, NormIn());
    else hipLaunchKernelGGL((gemm_f32_few_k<T, OUT_F32, false>), grid, block, 0, s, M, N, K, a, w, w2, (float*)C, NormIn());
    return hipGetLastError();
}
static hipError_t launch_f32_few(hipStream_t s, int out_mode, int M, int N, int K, const void* A, const void* W, const void* W2, void* C) {
    // (more rows per workgroup re-read the weights less, fewer keep more of the chip busy: M 33, N 512, K 1280 14.8 us with
    // 64 rows per workgroup, 6.9 with 16; M 64, N = K = 3584: 38 and 46)
    const int64_t wgs = (int64_t)((N + 15) / 16) * ((M + 15) / 16);
    if (M <= 16 || wgs <= 512) return launch_f32_few_t<1>(s, out_mode, M, N, K, A, W, W2, C);
    if (M <= 32 || wgs <= 1024) return launch_f32_few_t<2>(s, out_mode, M, N, K, A, W, W2, C);
    return launch_f32_few_t<4>(s, out_mode, M, N, K, A, W, W2, C);
}

// One row block of at most 1024 elements a row: every workgroup then reads all rows, at most 64 KB and the addend's as many, which the saved
// launch pays for while the rows are few: up to 12, and up to 16 of at most 256 elements, where launches count most.  A forward of 8 blocks,
// us, this way and with norms of their own (replayed from a graph; enqueued one by one where that differs by more than 2 %):
//   width 64:   8 rows 186 / 194 (201 / 250)   12 rows 199 / 201 (207 / 257)   16 rows 209 / 202 (217 / 250)
//   width 256:  8 rows 220 / 232 (226 / 261)   12 rows 232 / 239 (235 / 268)   16 rows 241 / 243 (244 / 274)
//   width 1024: 8 rows 296 / 318               12 rows 311 / 325               16 rows 326 / 328, with 4096 to 8192 columns 483 / 477
bool gemm_f32_norm_supported(int dtype, int M, int N, int K, const NormIn& n, const void* W, const void* W2) {
    return dtype == F32 && M <= (K <= 256 ? 16 : 12) && K <= 1024 && N <= 16 * 512 && f32_few_ok(M, K, n.x, W, W2) &&
           (((uintptr_t)n.add | (uintptr_t)n.gamma | (uintptr_t)n.x_out) & 15) == 0;
}
template <bool GLU>
static hipError_t launch_f32_norm(hipStream_t s, int M, int N, int K, const NormIn& n, const void* W, const void* W2, void* C) {
    if (M <= 0 || N <= 0) return hipSuccess;
    const size_t lds = (size_t)16 * (K + 4) * sizeof(float);
    auto kern = gemm_f32_few_k<1, OUT_F32, GLU, true>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 16 * (1024 + 4) * (int)sizeof(float));
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((N + 15) / 16), dim3(256), lds, s, M, N, K, (const float*)nullptr, (const float*)W, (const float*)W2, (float*)C, n);
    return hipGetLastError();
}
hipError_t gemm_f32_norm(hipStream_t s, int M, int N, int K, const NormIn& n, const void* W, void* C) {
    return launch_f32_norm<false>(s, M, N, K, n, W, nullptr, C);
}
hipError_t gemm_f32_norm_glu(hipStream_t s, int M, int N, int K, const NormIn& n, const void* Wg, const void* Wu, void* act) {
    return launch_f32_norm<true>(s, M, N, K, n, Wg, Wu, act);
}

// Few activation rows (M <= 32, one row of tiles): the weights stream through once and nothing else counts.  A
// workgroup owns 32 * WTN weight rows (GLU: half of them gate rows, half the matching up rows), WTN being free so
// that the tiles come out at just under one per CU.  The K steps of 64 go through a ring of S slots (activation rows and
// weight rows, both by global->LDS loads, S - 1 steps in flight); of a step's four 16-wide slices each of the four waves multiplies
// one, so that a fragment is read from the LDS once, and the four waves' sums meet in LDS at the end.
// A step's loads are whole 128-byte lines; fetched straight into MFMA operands (64 bytes per row and instruction)
// the vector-memory front end is the limit instead: 68 us at M = 16 on the gate/up shape below.
template <int WTN, int S, int OUT, bool GLU>
__global__ __launch_bounds__(256) void gemm_bf16_few_k(int M, int N, int K, const uint16_t* __restrict__ A, const uint16_t* __restrict__ W,
                                                       const uint16_t* __restrict__ W2, void* __restrict__ C, int nbn, int ksplit) {
    constexpr int NW = 4, BM = 32, BN = 32 * WTN, BNO = GLU ? BN / 2 : BN;
    constexpr int SLOT = (BM + BN) * 64;           // elements per slot: activation rows, then weight rows
    constexpr int LB = (BN / 8 + NW - 1) / NW;     // 1 KB loads per wave and step: weights (a wave's last one may be idle)
    constexpr int L = 1 + LB;                      // ... and activations
    constexpr bool kIdle = (BN / 8) % NW != 0;
    static_assert(S >= 3 && (S - 2) * L < 64, "the wait below counts the loads of S - 2 steps");
    static_assert(S * SLOT * 2 >= 4 * 32 * BN * 4, "the ring also holds the four slices' sums of 32 rows");
    extern __shared__ __align__(16) uint16_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lhi = lane >> 5, slice = wave;
    const int tile = blockIdx.x % nbn, cut = blockIdx.x / nbn, n0 = tile * BNO;
    // (integer division runs on the vector ALU: the uniform results go back into scalar registers)
    const int nk = K / 64, kt0 = __builtin_amdgcn_readfirstlane((int)((int64_t)nk * cut / ksplit));
    const int nt = __builtin_amdgcn_readfirstlane((int)((int64_t)nk * (cut + 1) / ksplit)) - kt0;
    auto desc = [&](const uint16_t* base, uint32_t bytes) {   // raw buffer descriptor; rows past its size fetch nothing
        const uint64_t p = (uint64_t)(uintptr_t)base;
        u32x4_t d;
        d[0] = __builtin_amdgcn_readfirstlane((uint32_t)p);
        d[1] = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32) & 0xffffu);
        d[2] = __builtin_amdgcn_readfirstlane(bytes);
        d[3] = 0x00020000u;
        return d;
    };
    const int cols = N - n0 < BNO ? N - n0 : BNO;
    u32x4_t rs_a = desc(A, (uint32_t)M * (uint32_t)K * 2u);
    // load i of a wave covers 8 consecutive tile rows (BNO is a multiple of 8: they are gate rows or up rows as a whole)
    const int r = lane >> 3, c = lane & 7;
    u32x4_t rs_b[LB];
    uint32_t off_b[LB], dst_b[LB];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)lds;
    const uint32_t lds_a = lds_base + (uint32_t)wave * 1024u;
    const int row_a = wave * 8 + r;
    const uint32_t off_a = ((uint32_t)row_a * (uint32_t)K + (c ^ ((row_a >> 1) & 7)) * 8) * 2u;
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        // (an idle load has an empty descriptor, fetches nothing and aims at a kilobyte behind the ring)
        const int row0 = (i * NW + wave) * 8, row = row0 + r;
        const bool on = !kIdle || row0 < BN, up = GLU && row0 >= BNO;
        rs_b[i] = desc((up ? W2 : W) + (int64_t)n0 * K, on ? (uint32_t)cols * (uint32_t)K * 2u : 0u);
        off_b[i] = ((uint32_t)(up ? row - BNO : row) * (uint32_t)K + (c ^ ((row >> 1) & 7)) * 8) * 2u;
        dst_b[i] = lds_base + (on ? (uint32_t)(BM * 128 + row0 * 128) : (uint32_t)(S * SLOT * 2));
    }
    // step t.  Past the end the loads stay, so that the wait counts hold, but have empty descriptors: the last step fetched again was S - 1 steps of
    // traffic (a third of a cut's 18) in front of the sums (one sequence decoded plainly 12.45 -> 12.40 ms, 16 sequences 17.41 -> 17.27).
    auto fetch = [&](int t, int slot) {
        const uint32_t k2 = (uint32_t)(kt0 + (t < nt ? t : nt - 1)) * 128u, so = (uint32_t)slot * (SLOT * 2);
        rs_a[2] = t < nt ? rs_a[2] : 0u;
#pragma unroll
        for (int i = 0; i < LB; ++i) rs_b[i][2] = t < nt ? rs_b[i][2] : 0u;
#pragma unroll
        for (int i = 0; i < LB; ++i)
            dma_buf_16_nt(rs_b[i], off_b[i], k2, kIdle && i == LB - 1 && wave + i * NW >= BN / 8 ? dst_b[i] : dst_b[i] + so);
        dma_buf_16(rs_a, off_a, k2, lds_a + so);
    };
    f32x16_t acc[WTN];
#pragma unroll
    for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll
    for (int t = 0; t < S - 1; ++t) fetch(t, t);
    const int frag = l32 * 64 + ((2 * slice + lhi) ^ ((l32 >> 1) & 7)) * 8;   // row l32 of a block, this wave's slice
    int slot = 0;
    for (int t = 0; t < nt; ++t) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // the last step's fragments have left their slot
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((S - 2) * L));           // step t has landed
        __builtin_amdgcn_s_barrier();                                 // ... for every wave
        __builtin_amdgcn_sched_barrier(0);
        fetch(t + S - 1, slot == 0 ? S - 1 : slot - 1);
        __builtin_amdgcn_sched_barrier(0);
        const uint16_t* p = lds + slot * SLOT + frag;
        bf16x8_t fb[WTN];
        const bf16x8_t fa = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)p);
#pragma unroll
        for (int j = 0; j < WTN; ++j) fb[j] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)(p + (BM + j * 32) * 64));
#pragma unroll
        for (int j = 0; j < WTN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, fb[j], acc[j], 0, 0, 0);
        slot = slot + 1 == S ? 0 : slot + 1;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));      // the empty fetches at the end as well: the ring is reused below
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // the four slices' sums: [slice][32][BN], then four columns per thread
    float* red = (float*)lds;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int row = 8 * (v >> 2) + 4 * lhi + (v & 3);
        if (row < M) {
#pragma unroll
            for (int j = 0; j < WTN; ++j) red[(slice * 32 + row) * BN + j * 32 + l32] = acc[j][v];
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < M * (BNO / 4); e += 64 * NW) {
        const int row = e / (BNO / 4), col = (e - row * (BNO / 4)) * 4;
        if (col >= cols) continue;
        auto sum4 = [&](int c0) {
            const float* p = red + row * BN + c0;
            float4 s = *(const float4*)p;
#pragma unroll
            for (int q = 1; q < 4; ++q) {
                const float4 o = *(const float4*)(p + q * 32 * BN);
                s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
            }
            return s;
        };
        const float4 g = sum4(col);
        const int64_t at = (int64_t)row * N + n0 + col;
        if constexpr (GLU) {
            const float4 u = sum4(BNO + col);
            auto act = [](float x, float y) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)) * y; };
            *(uint2*)((bf16*)C + at) = make_uint2(pack_bf16x2(act(g.x, u.x), act(g.y, u.y)), pack_bf16x2(act(g.z, u.z), act(g.w, u.w)));
        } else {
            *(float4*)((float*)C + (int64_t)cut * M * N + at) = g;
        }
    }
}

template <int WTN, bool GLU>
static hipError_t launch_few(hipStream_t s, int M, int N, int K, const void* A, const void* W, const void* W2, void* C, int ksplit = 1) {
    constexpr int BM = 32, BN = 32 * WTN, BNO = GLU ? BN / 2 : BN;
    constexpr int kFit = 159 * 1024 / ((BM + BN) * 128), S = kFit < 8 ? kFit : 8;
    constexpr size_t lds = (size_t)S * (BM + BN) * 128 + 1024;
    auto kern = gemm_bf16_few_k<WTN, S, GLU ? OUT_T : OUT_SPLIT_F32, GLU>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int nbn = (N + BNO - 1) / BNO;
    hipLaunchKernelGGL(kern, dim3(nbn * ksplit), dim3(256), lds, s, M, N, K, (const uint16_t*)A, (const uint16_t*)W, (const uint16_t*)W2, C, nbn,
                       ksplit);
    return hipGetLastError();
}

// Gate/up at up to 32 rows: the tile's weight rows in blocks of 32, the fewest that leave at most one workgroup per CU (in
// two rounds the second one's CUs are idle half of the time).  0: the tiled launches below take the product.
// Against those (us, best of three alternating runs on cold weights): N 18944, K 3584 (237 tiles of 80 columns): M = 1 59.0 ->
// 42.9 (6.3 TB/s); N 27648, K 5120 (247 of 112): M = 1 90.7 -> 84.0; N 11008, K 4096: M = 1 40.0 -> 35.0; N 4864, K 896: M = 1 10.6 -> 7.3.
// Four blocks are the width of the 64x128 tiles, which then run one per CU and are the better ones (N 14336, K 4096: 45.5 against 46.5); eight
// leave too few slots (N 32768, K 8192: 169 against 197), and seven need a K that pays for the sums of the four slices.
static int few_glu_width(int M, int N, int K) {
    int wtn = 2;
    while ((N + 16 * wtn - 1) / (16 * wtn) > 256) ++wtn;
    return M > 32 || wtn > 7 || wtn == 4 || (wtn == 7 && K < 512) ? 0 : wtn;
}
static hipError_t launch_few_glu(hipStream_t s, int wtn, int M, int N, int K, const void* A, const void* W, const void* W2, void* C) {
#define TLT_FEW(n) if (wtn == n) return launch_few<n, true>(s, M, N, K, A, W, W2, C);
    TLT_FEW(2) TLT_FEW(3) TLT_FEW(5) TLT_FEW(6) TLT_FEW(7)
#undef TLT_FEW
    return hipErrorInvalidValue;
}

// Products kept as partial sums at up to 32 rows: tiles of 64 columns, cut along K so that the workgroups come out at
// just under one per CU; wider tiles where their cuts fill more of the chip.  Returns the tile width in blocks of 32 columns, 0
// where the general plan of the cuts is the better one:
// - the cuts' first columns an odd multiple of 2048 apart (wider tiles: any multiple), in more than 2048 rows.  Whatever it is that
//   these streams collide in, they do so at every row count, and the general plan's more and shorter cuts do not (us, this kernel
//   and the general plan, slices read back at 4 TB/s included, same buffers, M = 16): N 8192: K 4096 17.1 and 14.9, K 12288 41.3 and
//   35.8, K 28672 up to 92 and 78; N 10240, K 8192 34.1 and 31.3; N 4096, K 8192 18.1 and 15.7; N 14336, K 6144 37.4 and 33.1.  At other K
//   this kernel wins by 2 to 30 % (N 8192: K 5120 by 7, K 8192 by 6; N 4096, K 4096 by 12; N 14336, K 12288 by 16).
// - the general plan has more than four times the cuts: a wave here adds up a quarter of its cut, and the sums would run longer
//   than before (N 18432, K 16384: 7 cuts against 1, error to float64 2.9e-7 and 3.9e-7).
static int few_split_plan(int N, int K, int general_cuts, int max_cuts, int* cuts) {
    int best = 0, best_wgs = 0;
    for (int wtn = 2; wtn <= 4; ++wtn) {
        const int nbn = (N + 32 * wtn - 1) / (32 * wtn);
        int ks = 256 / nbn;
        if (ks > K / 64 / 6) ks = K / 64 / 6;
        if (ks > max_cuts) ks = max_cuts;
        if (ks < 1 || nbn > 256) continue;
        if (best == 0 || (best_wgs < 200 && nbn * ks > best_wgs)) best = wtn, best_wgs = nbn * ks, *cuts = ks;
    }
    if (best == 0 || general_cuts > 4 * *cuts) return 0;
    const int apart = *cuts * 2048;
    if (N > 2048 && K % apart == 0 && (best > 2 || (K / apart) % 2 != 0)) return 0;
    return best;
}

// Gate/up at 33 to 256 rows.  A wave owns 32 activation rows and the whole width of the tile, so a workgroup has as many waves (2 to 8) as the rows
// fill and no matrix product is spent on padding beyond the last 32; the tile is as wide as leaves at most one workgroup per CU (32 * WTN
// weight rows: 16 gate and the matching 16 up rows in turns, as the mixed tiles of gemm_bf16_pipe_k).  A K step's four 16-wide slices run as there:
// the fragments of the next slice are read under a slice's products, the last slice's products run behind the barrier that publishes the next step,
// and the step's loads (weights first) are dealt out behind the products, S - 1 steps ahead.
// What bounds it: every byte, cold weights and the activation rows that each workgroup takes from L2 alike, comes through the CU's load path at
// about 57 GB/s at 2.4 GHz (a load-only kernel with these loads: 40.7 us at 32 rows, 44.8 at 96, 49.6 at 192, 52.2 at 256 for N 18944, K 3584), and the
// chip holds 1.6 to 2 GHz here under its power limit: what is saved is padding (128- and 256-row tiles) and the sums of four slices in
// LDS (gemm_bf16_few_k).  Dispatch and measurements: mid_glu_width.
// Products kept as partial sums (GLU off) have whole tiles of 32 * WTN columns and one of ksplit cuts of K per workgroup.  CH: how many chains of
// products a cut is summed in (its 16-wide slices in turns, added pairwise at the end), in registers that are idle otherwise, so that
// few long cuts round no worse than many short ones (mid_split_plan).  SEG: in how many pieces of K one after the other, where chains side by side do not fit
// the registers (mid_glu_four).
template <int NW, int WTN, int S, bool GLU, int CH, int SEG>
__global__ __launch_bounds__(64 * NW) void gemm_bf16_mid_k(int M, int N, int K, const uint16_t* __restrict__ A, const uint16_t* __restrict__ W,
                                                           const uint16_t* __restrict__ W2, void* __restrict__ C, int per_xcd, int nbn, int ksplit, int ldc) {
    constexpr int BM = 32 * NW, BN = 32 * WTN, BNO = GLU ? BN / 2 : BN;
    constexpr int SLOT = (BM + BN) * 64;           // elements per slot: activation rows, then weight rows
    constexpr int LA = 4, LB = (BN / 8 + NW - 1) / NW, L = LA + LB;   // 1 KB loads per wave and step (a wave's last weight load may be idle)
    constexpr bool kIdle = (BN / 8) % NW != 0;
    static_assert(SEG == 1 || CH == 1, "one or the other");
    extern __shared__ __align__(16) uint16_t lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    // (an XCD's workgroups own neighbouring columns: the lines that two tiles share are completed in its L2; of a product cut along K they
    // own the same cut, whose activations each XCD then fetches once)
    const int at = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const int cut = GLU ? 0 : __builtin_amdgcn_readfirstlane(at / nbn), n0 = (GLU ? at : at - cut * nbn) * BNO;
    if (GLU ? n0 >= N : cut >= ksplit) return;
    const int kt0 = GLU ? 0 : __builtin_amdgcn_readfirstlane((int)((int64_t)(K / 64) * cut / ksplit));
    const int nt = GLU ? K / 64 : __builtin_amdgcn_readfirstlane((int)((int64_t)(K / 64) * (cut + 1) / ksplit)) - kt0;
    auto desc = [&](const uint16_t* base, uint32_t bytes) {   // raw buffer descriptor; rows past its size fetch nothing
        const uint64_t p = (uint64_t)(uintptr_t)base;
        u32x4_t d;
        d[0] = __builtin_amdgcn_readfirstlane((uint32_t)p);
        d[1] = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32) & 0xffffu);
        d[2] = __builtin_amdgcn_readfirstlane(bytes);
        d[3] = 0x00020000u;
        return d;
    };
    const int cols = N - n0 < BNO ? N - n0 : BNO;
    u32x4_t rs_a = desc(A, (uint32_t)M * (uint32_t)K * 2u);
    const int r = lane >> 3, c = lane & 7;
    u32x4_t rs_b[LB];
    uint32_t off_a[LA], off_b[LB], dst_b[LB];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)lds;
    const uint32_t lds_a = lds_base + (uint32_t)(wave * LA) * 1024u;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int row = (wave * LA + i) * 8 + r;
        off_a[i] = ((uint32_t)row * (uint32_t)K + (c ^ ((row >> 1) & 7)) * 8) * 2u;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        // (an idle load has an empty descriptor, fetches nothing and aims at a kilobyte behind the ring)
        const int row0 = (i * NW + wave) * 8, row = row0 + r;
        const bool on = !kIdle || row0 < BN, up = GLU && row0 >= BNO;
        rs_b[i] = desc((up ? W2 : W) + (int64_t)n0 * K, on ? (uint32_t)cols * (uint32_t)K * 2u : 0u);
        off_b[i] = ((uint32_t)(up ? row - BNO : row) * (uint32_t)K + (c ^ ((row >> 1) & 7)) * 8) * 2u;
        dst_b[i] = lds_base + (on ? (uint32_t)(BM * 128 + row0 * 128) : (uint32_t)(S * SLOT * 2));
    }
    // load i of a step, weights first; past the last step, which `upto` is told, loads fetch nothing, so that the wait counts hold
    auto upto = [&](int t) {
        rs_a[2] = t < nt ? rs_a[2] : 0u;
#pragma unroll
        for (int i = 0; i < LB; ++i) rs_b[i][2] = t < nt ? rs_b[i][2] : 0u;
    };
    auto load = [&](int i, uint32_t k2, uint32_t so) {
        if (i < LB) {
            const uint32_t dst = kIdle && i == LB - 1 && wave + i * NW >= BN / 8 ? dst_b[i] : dst_b[i] + so;
            dma_buf_16_nt(rs_b[i], off_b[i], k2, dst);
        } else {
            dma_buf_16(rs_a, off_a[i - LB], k2, lds_a + so + (i - LB) * 1024u);
        }
    };
    auto koff = [&](int t) { return (uint32_t)(kt0 + (t < nt ? t : nt - 1)) * 128u; };
    f32x16_t acc[CH][WTN], done[SEG > 1 ? WTN : 1];   // (done: the finished pieces of K)
#pragma unroll
    for (int h = 0; h < CH; ++h)
#pragma unroll
        for (int j = 0; j < WTN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[h][j][v] = 0.f;
    if constexpr (SEG > 1)
#pragma unroll
        for (int j = 0; j < WTN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) done[j][v] = 0.f;
    int seg = 1;
    constexpr int Q3 = (L + 3) / 4;                // loads issued under slice 3; the rest under slices 0 .. 2 of the next step
    static_assert(S >= 3 && (S - 2) * L + Q3 < 64, "what the waits below count");
#pragma unroll
    for (int t = 0; t < S - 1; ++t) {
        upto(t);
#pragma unroll
        for (int i = 0; i < L; ++i) load(i, koff(t), (uint32_t)t * (SLOT * 2));
    }
    upto(S - 1);
#pragma unroll
    for (int i = 0; i < Q3; ++i) load(i, koff(S - 1), (uint32_t)(S - 1) * (SLOT * 2));
    const int sw = (l32 >> 1) & 7;
    const int fragA = (wave * 32 + l32) * 64;
    const int fragB = (GLU ? (l32 & 15) + (l32 >> 4) * BNO : l32) * 64;   // 16 gate rows and the 16 up rows that belong to them
    bf16x8_t fa[2], fb[2][WTN];
    auto read = [&](int buf, const uint16_t* p, int kk) {
        const int ch = ((2 * kk + lhi) ^ sw) * 8;
        fa[buf] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)(p + fragA + ch));
#pragma unroll
        for (int j = 0; j < WTN; ++j)
            fb[buf][j] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)(p + BM * 64 + fragB + j * (GLU ? 16 : 32) * 64 + ch));
    };
    auto mul = [&](int kk) {
#pragma unroll
        for (int j = 0; j < WTN; ++j)
            acc[kk % CH][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk & 1], fb[kk & 1][j], acc[kk % CH][j], 0, 0, 0);
    };
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((S - 2) * L + Q3));   // step 0 has landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read(0, lds, 0);
    int slot = 0, before = S - 1;                  // this step's slot; the one whose refill is under way
    for (int t = 0; t < nt; ++t) {
        const uint16_t* p = lds + slot * SLOT;
        const int next = slot + 1 == S ? 0 : slot + 1;
        const uint32_t k2 = koff(t + S - 1), so = (uint32_t)before * (SLOT * 2);
#pragma unroll
        for (int kk = 0; kk < 3; ++kk) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            read((kk + 1) & 1, p, kk + 1);
            __builtin_amdgcn_sched_barrier(0);
            mul(kk);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = Q3 + kk * (L - Q3) / 3; i < Q3 + (kk + 1) * (L - Q3) / 3; ++i) load(i, k2, so);
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((S - 2) * L));   // step t + 1 has landed
        __builtin_amdgcn_s_barrier();                         // ... for every wave; this step's slot is free
        __builtin_amdgcn_sched_barrier(0);
        read(0, lds + next * SLOT, 0);
        __builtin_amdgcn_sched_barrier(0);
        mul(3);
        __builtin_amdgcn_sched_barrier(0);
        upto(t + S);
#pragma unroll
        for (int i = 0; i < Q3; ++i) load(i, koff(t + S), (uint32_t)slot * (SLOT * 2));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (SEG > 1) {
            if (seg < SEG && (t + 1) * SEG >= nt * seg) {   // (the end of a piece of K)
                ++seg;
#pragma unroll
                for (int j = 0; j < WTN; ++j) {
                    done[j] += acc[0][j];
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[0][j][v] = 0.f;
                }
            }
        }
        before = slot;
        slot = next;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));      // the empty fetches at the end as well, before the LDS is released
    if constexpr (SEG > 1) {
#pragma unroll
        for (int j = 0; j < WTN; ++j) acc[0][j] += done[j];
    }
    if constexpr (GLU) {                           // chain after chain, as gemm_bf16_few_k adds its four waves' sums
#pragma unroll
        for (int h = 1; h < CH; ++h)
#pragma unroll
            for (int j = 0; j < WTN; ++j) acc[0][j] += acc[h][j];
    } else {                                       // a lane's column of every block, 128 bytes of a row per half-wave
        float* out = (float*)C + (int64_t)cut * M * ldc + n0 + l32;
#pragma unroll
        for (int h = CH / 2; h > 0; h /= 2)
#pragma unroll
            for (int i = 0; i < h; ++i)
#pragma unroll
                for (int j = 0; j < WTN; ++j) acc[i][j] += acc[i + h][j];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = wave * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3);
#pragma unroll
            for (int j = 0; j < WTN; ++j)
                if (row < M && j * 32 < cols) out[(int64_t)row * ldc + j * 32] = acc[0][j][v];
        }
        return;
    }
    // (as the mixed tiles of gemm_bf16_pipe_k: gate and up of a column lie in lanes l and l + 16 of a half-wave)
    const int row0 = wave * 32 + 4 * lhi, odd16 = (l32 >> 4) & 1, odd = lane & 1;
#pragma unroll
    for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            float x[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[0][j][4 * vq + 2 * e]), __float_as_uint(acc[0][j][4 * vq + 2 * e + 1]), false, false);
                const float g = __uint_as_float(q[0]), u = __uint_as_float(q[1]);
                x[e] = g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
            }
            const float other = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(odd ? x[0] : x[1]), 0xB1, 0xF, 0xF, false));
            const uint32_t out = odd ? pack_bf16x2(other, x[1]) : pack_bf16x2(x[0], other);
            const int row = row0 + 8 * vq + 2 * odd + odd16, col0 = j * 16;
            if (row < M && col0 < cols) *(uint32_t*)((bf16*)C + (int64_t)row * N + n0 + col0 + (l32 & 14)) = out;
        }
}

template <int NW, int WTN, bool GLU, int CH, int SEG = 1>
static hipError_t launch_mid(hipStream_t s, int M, int N, int K, const void* A, const void* W, const void* W2, void* C, int ksplit = 1, int ldc = 0) {
    constexpr bool kIdle = (4 * WTN) % NW != 0;
    constexpr int kSlot = (32 * NW + 32 * WTN) * 128, kFit = (GLU ? 159 * 1024 : 160 * 1024 - (kIdle ? 1024 : 0)) / kSlot, S = kFit < 6 ? kFit : 6;
    constexpr size_t lds = (size_t)S * kSlot + (kIdle ? 1024 : 0);
    constexpr int BNO = GLU ? 16 * WTN : 32 * WTN;
    auto kern = gemm_bf16_mid_k<NW, WTN, S, GLU, CH, SEG>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int nbn = (N + BNO - 1) / BNO, per_xcd = (nbn * ksplit + 7) / 8;
    hipLaunchKernelGGL(kern, dim3(8 * per_xcd), dim3(64 * NW), lds, s, M, N, K, (const uint16_t*)A, (const uint16_t*)W, (const uint16_t*)W2, C, per_xcd,
                       nbn, ksplit, ldc ? ldc : N);
    return hipGetLastError();
}

// Width of gemm_bf16_mid_k's tiles in blocks of 16 gate and 16 up rows: the fewest that leave at most one workgroup per CU; 0: another kernel.
// From 65 rows on, measured against the tiled kernels and a few-row kernel with two groups of waves (us per call, p10 of 40 calls, cold weights, activations
// rewritten before every call, about 4 us of event overhead in both figures, sums in one chain; *: rings of two slots, which lose and are not built):
//   rows            72         128        160        192        224        256
//   18944 x 3584    52.7/49.4  59.6/54.8  66.4/59.4  69.3/65.0  72.3/68.4  74.0/73.3    (5 blocks)
//   27648 x 5120    96.0/91.7  104/101    127/110    128/124    133/154*   138/157*     (7)
//   24576 x 6144    101/98     108/105    141/111    142/119    145/126    145/165*     (6)
//   13824 x 5120    61.8/58.2  72.2/66.4  84.0/74.2  84.2/74.5  86.7/79.5  87.4/81.6    (4)
//   11008 x 4096    42.0/36.9  47.9/43.3  64.9/50.0  68.2/53.2  73.6/55.8  79.0/59.3    (3)
//   8192 x 4096     41.6/29.1  45.8/35.4  41.3/40.7  42.6/45.3  44.1/48.0  46.5/49.0    (2)
// Two blocks leave half of the chip idle.  At five blocks 256 rows are even alone and 2 % slower in a step (eight waves draw more power than four of 64 rows).
// With K below 1024 the wide ones still gain (18944 x 512, 128 rows: 16.8 -> 15.3), and the narrow ones above 128 rows (11008 x 512: 160 rows 16.0 -> 13.6).
// At 33 to 64 rows against the 64-row tiles (short K, four blocks) and the few-row kernel with 64 rows (the others), a graph of calls on cold weights, no
// event between them, four sums where there are four:
//   rows            33         48         64
//   4864 x 768      7.8/7.6    8.4/7.8    9.0/8.3      (2 blocks)
//   8192 x 3584     22.2/21.8  23.3/22.6  24.9/23.9
//   11008 x 1024    11.8/11.9  12.2/12.1  12.9/12.4    (3)
//   11008 x 3584    28.9/28.4  30.2/29.3  32.1/30.6
//   18944 x 512     13.2/11.0  13.3/11.1  13.7/11.3    (5)
//   18944 x 1536    24.6/24.5  25.4/24.7  26.8/25.2
//   18944 x 3584    45.6/45.3  47.0/46.1  48.4/46.8
//   24576 x 512     13.7/12.7  13.8/12.8  14.3/12.9    (6)
//   22016 x 1024    19.0/19.9  19.8/20.1  20.6/20.2
//   24576 x 3584    56.5/56.6  57.3/57.0  58.5/57.4
//   27648 x 5120    90.2/90.1  92.2/91.2  92.1/91.9    (7)
// (K 1024 at 33 to 40 rows is where the adds between quarters show, 0.1 to 0.9 us; a K from 1536 on hides them.)
// Not at four blocks, where the tiles come out at one per CU too and the ring is shorter (14336 x 1024 12.9/13.5 at 33 rows, x 2560 29.4/31.4 at 64, x 5120
// 53.1/55.9; x 3584 38.0/37.8), nor at seven with K below 2560 (28672 x 128 7.7/8.6 at 33 rows, x 512 14.2/14.6, x 2048 51.1/52.3; x 1536 33.9/33.4).
static int mid_glu_width(int M, int N, int K) {
    int wtn = 2;
    while ((N + 16 * wtn - 1) / (16 * wtn) > 256) ++wtn;
    if (M <= 32 || wtn > 7 || (wtn == 4 && M <= 64)) return 0;
    const int rows = wtn == 2 ? 128 : wtn <= 4 ? 256 : wtn <= 6 ? 224 : 192;
    const int k_min = wtn == 7 && M <= 64 ? 2560 : wtn >= 5 || (wtn == 2 && M <= 64) ? 64 : wtn == 4 || M > 128 ? 512 : 1024;
    return M <= rows && K >= k_min ? wtn : 0;
}
// Whether the tile's sums over K are four (long K up to 128 rows; gemm_bf16_few_k has four at up to 32): one chain errs twice as far.  Rms error of an up sum
// to float64, four and one: K 1024 1.0e-7 and 1.8e-7, 3584 1.8e-7 and 3.7e-7.  Two blocks of columns hold four chains side by side, with the few-row
// kernel's bits; wider ones add up K in quarters (four chains of 5 blocks are 320 registers that the compiler copies between its two files: 18944 x 3584, 64
// rows 61.5 us; of 6 and 7 they do not fit).  The adds between quarters cost 0.3 to 1 us: us per call on cold weights, one chain and four sums,
//   rows            48           64           72           128
//   4864 x 896      8.9/9.4      9.0/9.7      -            -           (2 blocks)
//   11008 x 4096    38.5/39.0    38.8/39.3    -            -           (3)
//   14336 x 4096    -            -            49.5/50.1    51.5/52.1   (4)
//   18944 x 3584    45.5/46.0    45.8/46.5    46.5/47.0    51.1/51.9   (5)
//   24576 x 6144    112/113      113/114      115/115      120/121     (6)
//   27648 x 5120    89.6/90.5    90.4/91.4    -            -           (7)
// Shorter K and the other widths stay in one chain, with the bits of all tiles; above 128 rows the registers are taken.
static bool mid_glu_four(int M, int wtn, int K) {
    if (M <= 64) return wtn == 2 || K >= 1024;
    return M <= 128 && (wtn == 4 || ((wtn == 5 || wtn == 6) && K >= 2560));
}
static hipError_t launch_mid_glu(hipStream_t s, int wtn, int M, int N, int K, const void* A, const void* Wg, const void* Wu, void* act) {
    if (mid_glu_four(M, wtn, K)) {
#define TLT_MID(nw, n) if ((M + 31) / 32 == nw && wtn == n) return launch_mid<nw, n, true, n == 2 ? 4 : 1, n == 2 ? 1 : 4>(s, M, N, K, A, Wg, Wu, act);
        TLT_MID(2, 2) TLT_MID(2, 3) TLT_MID(2, 5) TLT_MID(2, 6) TLT_MID(2, 7)
        TLT_MID(3, 4) TLT_MID(3, 5) TLT_MID(3, 6)
        TLT_MID(4, 4) TLT_MID(4, 5) TLT_MID(4, 6)
#undef TLT_MID
        return hipErrorInvalidValue;
    }
#define TLT_MID(nw, n) if ((M + 31) / 32 == nw && wtn == n) return launch_mid<nw, n, true, 1>(s, M, N, K, A, Wg, Wu, act);
    TLT_MID(2, 5) TLT_MID(2, 6)
    TLT_MID(3, 2) TLT_MID(3, 3) TLT_MID(3, 5) TLT_MID(3, 6) TLT_MID(3, 7)
    TLT_MID(4, 2) TLT_MID(4, 3) TLT_MID(4, 5) TLT_MID(4, 6) TLT_MID(4, 7)
    TLT_MID(5, 3) TLT_MID(5, 4) TLT_MID(5, 5) TLT_MID(5, 6) TLT_MID(5, 7)
    TLT_MID(6, 3) TLT_MID(6, 4) TLT_MID(6, 5) TLT_MID(6, 6) TLT_MID(6, 7)
    TLT_MID(7, 3) TLT_MID(7, 4) TLT_MID(7, 5) TLT_MID(7, 6)
    TLT_MID(8, 3) TLT_MID(8, 4)
#undef TLT_MID
    return hipErrorInvalidValue;
}

// Products kept as partial sums at 33 to 256 rows: gemm_bf16_mid_k with a workgroup per (64 columns up to 128 rows, 128 above; cut), the cuts as many as
// leave at most one workgroup per CU.  Returns whether it takes the product; elsewhere the general plan is the better one.
// - Up to 128 rows, K up to 4096: the general plan's 128x128 tiles come out even only with twice the cuts (and slices to write and read back).  Longer cuts
//   pay for narrow tiles, which re-read the activation rows more often (K 7168: -2 to +2 %, K 8192 -4 to -9 %).  Us per call on cold weights, a graph of 40
//   calls, slices read back at 4 TB/s included, the general plan and this kernel:
//     rows           40           72           96           128
//     3584 x 3584    9.8/9.1      12.0/10.8    13.2/11.8    14.5/13.2   (9 and 4 cuts)
//     4608 x 3584    10.6/10.3    13.0/12.4    14.2/13.5    15.9/15.1   (7 and 3)
//     4096 x 4096    10.6/10.0    13.1/11.5    14.3/13.0    16.0/14.1   (8 and 4)
//     8192 x 2048    10.6/10.3    13.0/11.6    14.2/12.7    16.1/14.1   (4 and 2)
//   Not with the cuts' first columns an odd multiple of 2048 apart (see few_split_plan; 8192 x 4096: 15.3/18.0, 21.4/22.3), nor uncut (14336 x 3584: 28.9/31.9).
// - From 129 rows on, where the general plan too fills the chip by cutting (its 256-row tiles pad 130 rows to 256, two rows of 128-row tiles
//   read the weights twice):
//     rows           136          160          192          224          256
//     3584 x 18944   39.3/37.5    41.2/39.2    43.3/40.7    45.8/44.2    47.8/49.4   (9 cuts)
//     5120 x 27648   77.9/64.7    80.8/68.8    79.2/70.9    82.9/76      86.9/82.6   (12 or 6, and 6)
//     7168 x 5120    27.8/26.7    29.4/27.8    31.2/28.6    32.6/31.1    34.5/33.9   (4)
//     8192 x 8192    42.4/39.2    43.8/40.7    45.7/42.1    48.1/45.4    50.5/49.6   (4)
//     14336 x 5120   44.4/41.1    47.1/43.8    48.9/45.0    51.6/48.0    53.9/50.7   (2)
//   (above 224 rows nothing is padding, and in less than 5120 columns the gain is -4 to +2 %; with long K it is -3 % at 4608 x 18944 and 3584 x 18944, +6 and +7 % at
//   4608 x 14336 and 4096 x 28672, which stay where they were.)  Where the general plan prefers fewer, longer cuts of wide tiles (3584 x 3584: 4) it is ahead by 1
//   to 6 %.  The gain is the card's too: from 193 rows on two cards showed 0 to +13 % over this range, two others -4 to +6 %.
// The kernel's two or four chains per cut keep the serial sums no longer than the general plan's in either case; error to float64 (slices added in fp32) 1.24e-7 ->
// 0.98e-7 at 3584 x 3584, 2.8e-7 -> 2.0e-7 at 3584 x 18944, even where this kernel has half of the cuts (14336 x 8192 at 136 rows: 2.73e-7 either way).
static bool mid_split_plan(int M, int N, int K, int general_cuts, int max_cuts, int* cuts) {
    if (M <= 32 || M > 256) return false;
    const int cols = M <= 128 ? 64 : 128, nbn = N / cols;
    int ks = 256 / nbn;
    if (ks > K / 64 / 6) ks = K / 64 / 6;
    if (ks > max_cuts) ks = max_cuts;
    if (ks < 2 || nbn * ks < 200) return false;
    *cuts = ks;
    if (M <= 128) return K <= 4096 && general_cuts <= 4 * ks && !(N > 2048 && K % (2048 * ks) == 0 && K / (2048 * ks) % 2 != 0);
    return (M <= 224 || N >= 5120) && general_cuts >= ks && general_cuts <= 2 * ks;
}
static hipError_t launch_mid_parts(hipStream_t s, int M, int N, int K, const void* A, const void* W, float* parts, int cuts) {
    switch ((M + 31) / 32) {
        case 2: return launch_mid<2, 2, false, 4>(s, M, N, K, A, W, nullptr, parts, cuts);
        case 3: return launch_mid<3, 2, false, 4>(s, M, N, K, A, W, nullptr, parts, cuts);
        case 4: return launch_mid<4, 2, false, 4>(s, M, N, K, A, W, nullptr, parts, cuts);
        case 5: return launch_mid<5, 4, false, 2>(s, M, N, K, A, W, nullptr, parts, cuts);
        case 6: return launch_mid<6, 4, false, 2>(s, M, N, K, A, W, nullptr, parts, cuts);
        case 7: return launch_mid<7, 4, false, 2>(s, M, N, K, A, W, nullptr, parts, cuts);
        case 8: return launch_mid<8, 4, false, 2>(s, M, N, K, A, W, nullptr, parts, cuts);
    }
    return hipErrorInvalidValue;
}

// What whole rounds of 256-column tiles leave of a product of 33 to 128 rows, up to 96 columns per CU: the narrowest tiles that come out at one per CU, K
// summed in the one order of all tiles (so the bits are those of 128x128 tiles, whose 164 workgroups held a third less of the weights in flight).
// Whole product on cold weights, us: N 152064, K 3584 40 rows 201 -> 195, 96 206 -> 202, 128 216 -> 213; K 5120 281 -> 269, 305 -> 298, 316 -> 311; N
// 90112, K 4096 164 -> 160, 173 -> 169, 179 -> 173.
static hipError_t launch_mid_rest(hipStream_t s, int M, int N, int K, const void* A, const void* W, void* C, int ldc) {
#define TLT_MID(nw, n) if ((M + 31) / 32 == nw && (N + 32 * n - 1) / (32 * n) <= 256) return launch_mid<nw, n, false, 1>(s, M, N, K, A, W, nullptr, C, 1, ldc);
    TLT_MID(2, 2) TLT_MID(2, 3)
    TLT_MID(3, 2) TLT_MID(3, 3)
    TLT_MID(4, 2) TLT_MID(4, 3)
#undef TLT_MID
    return hipErrorInvalidValue;
}

template <int WGM, int WGN, int WTM, int WTN, int SA, int SB, bool GLU = false, bool NTW = false>
static hipError_t launch_pipe(hipStream_t s, int out_mode, int M, int N, int K, const void* A, const void* W, void* C,
                              const void* W2 = nullptr, int ksplit = 1, int ldc = 0, int kskew = 0) {
    // N counts the output columns this launch covers; ldc (default N) is the row stride of C
    constexpr int BM = 32 * WTM * WGM, BN = 32 * WTN * WGN;
    if (ldc == 0) ldc = N;
    constexpr int BNO = GLU ? BN / 2 : BN;
    // (only tile widths that do not divide 64 handle a partial last column tile; N % 32 == 0 either way)
    if ((BNO % 64 == 0 && N % BNO != 0) || N % 32 != 0) return hipErrorInvalidValue;
    const int nbm = (M + BM - 1) / BM, nbn = (N + BNO - 1) / BNO;
    const int total = nbm * nbn * ksplit;
    const int per_xcd = (total + 7) / 8;
    const size_t lds = ((size_t)SA * BM + (size_t)SB * BN) * 64 * sizeof(uint16_t);
    // persistent workgroups: as many as the chip holds at once (32 CUs per XCD, LDS-limited occupancy)
    const int occupancy = lds <= 80 * 1024 ? 2 : 1;
    // (a workgroup that walks several tiles needs as many K tiles in each as either cursor may run ahead)
    const bool persistent = (K / 64) / ksplit >= (SA > SB ? SA : SB);
    const int wg_per_xcd = (!persistent || per_xcd < 32 * occupancy) ? per_xcd : 32 * occupancy;
    dim3 grid(wg_per_xcd * 8), block(64 * WGM * WGN);
#define LAUNCH(OUT)                                                                                                   \
    {                                                                                                                 \
        auto kern = gemm_bf16_pipe_k<WGM, WGN, WTM, WTN, SA, SB, OUT, GLU, NTW && (OUT == OUT_T || OUT == OUT_F32 || OUT == OUT_SPLIT_F32)>; \
        static bool attr_set = false;                                                                                 \
        if (!attr_set) {                                                                                              \
            hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
            if (e != hipSuccess) return e;                                                                            \
            attr_set = true;                                                                                          \
        }                                                                                                             \
        hipLaunchKernelGGL(kern, grid, block, lds, s, M, ldc, K, (const uint16_t*)A, (const uint16_t*)W,              \
                           (const uint16_t*)W2, C, nbm, total, per_xcd, ksplit, wg_per_xcd, (int32_t*)nullptr, kskew,              \
                           (int64_t)M * ldc, N);                                                                     \
    }
    if (GLU || out_mode == OUT_T) LAUNCH(OUT_T)
    else if (out_mode == OUT_F32) LAUNCH(OUT_F32)
    else if (out_mode == OUT_SPLIT_F32) LAUNCH(OUT_SPLIT_F32)
    else if (ksplit == 1) LAUNCH(OUT_ADD_F32)
    else LAUNCH(OUT_ATOMIC_ADD_F32)
#undef LAUNCH
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_generic(hipStream_t s, int out_mode, int M, int N, int K, const void* A, const void* W, void* C) {
    dim3 grid((N + 63) / 64, (M + 63) / 64), block(256);
    if (out_mode == OUT_T)
        hipLaunchKernelGGL((gemm_generic_k<T, OUT_T>), grid, block, 0, s, M, N, K, (const T*)A, (const T*)W, C);
    else if (out_mode == OUT_F32)
        hipLaunchKernelGGL((gemm_generic_k<T, OUT_F32>), grid, block, 0, s, M, N, K, (const T*)A, (const T*)W, C);
    else
        hipLaunchKernelGGL((gemm_generic_k<T, OUT_ADD_F32>), grid, block, 0, s, M, N, K, (const T*)A, (const T*)W, C);
    return hipGetLastError();
}

// 256x256 tiles over the columns that fill whole rounds of the chip's 256 CUs, 128x128 tiles (two
// workgroups per CU) over the rest: a last round that would leave most CUs idle is replaced by a
// shorter one.  glu: W/W2 are the gate/up matrices and N counts gate columns (a 256-row weight tile
// then yields 128 output columns, a 128-row one 64).
static hipError_t launch_tiled(hipStream_t s, int out_mode, int M, int N, int K, const void* A, const void* W,
                               const void* W2, void* C, bool glu) {
    const int bno256 = glu ? 128 : 256, bno128 = glu ? 64 : 128;
    const int nbm256 = (M + 255) / 256, nbm128 = (M + 127) / 128;
    const int nbn256 = N / bno256;   // whole 256-wide column tiles
    const size_t c_elt = (glu || out_mode == OUT_T) ? 2 : 4;
    auto small = [&](int n_cols, int col0) -> hipError_t {
        const int tiles = nbm128 * (n_cols / bno128);
        const void* w = (const uint16_t*)W + (int64_t)col0 * K;
        const void* w2 = W2 ? (const uint16_t*)W2 + (int64_t)col0 * K : nullptr;
        void* c = (char*)C + (size_t)col0 * c_elt;
        // (a single row of tiles: every weight row is read once, by one workgroup: non-temporal loads, see NTW)
        if (glu && nbm128 == 1) {
            if (tiles > 256) return launch_pipe<2, 2, 2, 2, 3, 2, true, true>(s, OUT_T, M, n_cols, K, A, w, c, w2, 1, N);
            return launch_pipe<2, 2, 2, 2, 3, 3, true, true>(s, OUT_T, M, n_cols, K, A, w, c, w2, 1, N);
        }
        if (glu) {
            if (tiles > 256) return launch_pipe<2, 2, 2, 2, 3, 2, true>(s, OUT_T, M, n_cols, K, A, w, c, w2, 1, N);
            return launch_pipe<2, 2, 2, 2, 3, 3, true>(s, OUT_T, M, n_cols, K, A, w, c, w2, 1, N);
        }
        // up to 64 rows: tiles of 64 rows (half of a 128-row tile would be padding), four waves side by side; the LDS that is freed holds a
        // third weight slot with two workgroups per CU, or five (and four of activations) with one.  What bounds it is how much of the weight
        // stream a CU has in flight.  Against 128x128 tiles, whose two workgroups per CU had two slots (us, same buffers, cold weights): N
        // 152064, K 3584: 1 row 183 -> 162 (6.7 TB/s), 16 rows 189 -> 173, 32 rows 202 -> 188; N 128256, K 8192: 358 -> 339, 352 -> 336, 365 -> 350;
        // N 32000, K 4096: 56 -> 55; one tile per CU: N 16384, K 4096 40 -> 33 at 1 row, 39.3 -> 37.3 at 64; N 8192, K 8192 61 -> 48, 64 -> 57.
        // (With one tile per CU four activation slots leave two K steps' loads outstanding, see kInFlight, and five weight slots are what that
        // takes; with eight the first burst was longer: N 16384, K 4096, 1 row 30.8 -> 30.1, 64 rows 37.8 -> 37.0; N 8192, K 8192 46.7 -> 45.9
        // and 58.7 -> 58.1; N 32768, K 2048 31.1 -> 30.3, 33.8 -> 32.7.  With four, 10 loads instead of 12: 1 row 30.7, 48.7 and 30.3.)
        if (M <= 64) {
            if (tiles > 256) return launch_pipe<1, 4, 2, 1, 3, 3, false, true>(s, out_mode, M, n_cols, K, A, w, c, nullptr, 1, N);
            return launch_pipe<1, 4, 2, 1, 4, 5, false, true>(s, out_mode, M, n_cols, K, A, w, c, nullptr, 1, N);
        }
        if (nbm128 == 1) {
            if (tiles > 256) return launch_pipe<2, 2, 2, 2, 3, 2, false, true>(s, out_mode, M, n_cols, K, A, w, c, nullptr, 1, N);
            return launch_pipe<2, 2, 2, 2, 3, 3, false, true>(s, out_mode, M, n_cols, K, A, w, c, nullptr, 1, N);
        }
        // more 128-row tiles than CUs (some CUs would hold two workgroups and take twice as long as the others), but
        // 192- or 256-row tiles fit the chip once: one workgroup per CU with the CU to itself, whichever of the two
        // fills more of the CUs (o projection at M = 1536: 336 tiles -> 224 of 192 rows, 49.9 -> 43.0 us; qkv at
        // M = 1536: 432 -> 216 of 256 rows, 59.8 -> 54.2 us; o at M = 2048: 448 -> 224 of 256 rows, 62.4 -> 51.0 us;
        // best of four interleaved runs on cold weights)
        if (tiles > 256) {
            const int t192 = ((M + 191) / 192) * (n_cols / bno128), t256 = nbm256 * (n_cols / bno128);
            const bool fit192 = t192 <= 256, fit256 = t256 <= 256 && t256 >= 200;
            if (fit256 && (!fit192 || t256 >= t192))
                return launch_pipe<2, 2, 4, 2, 3, 4>(s, out_mode, M, n_cols, K, A, w, c, nullptr, 1, N);
            if (fit192) return launch_pipe<2, 2, 3, 2, 3, 4>(s, out_mode, M, n_cols, K, A, w, c, nullptr, 1, N);
        }
        if (tiles > 256) return launch_pipe<2, 2, 2, 2, 3, 2>(s, out_mode, M, n_cols, K, A, w, c, nullptr, 1, N);
        return launch_pipe<2, 2, 2, 2, 3, 3>(s, out_mode, M, n_cols, K, A, w, c, nullptr, 1, N);
    };
    auto big = [&](int n_cols) -> hipError_t {
        if (nbm256 == 1) {
            if (glu) return launch_pipe<2, 2, 4, 4, 3, 2, true, true>(s, OUT_T, M, n_cols, K, A, W, C, W2, 1, N);
            return launch_pipe<2, 2, 4, 4, 3, 2, false, true>(s, out_mode, M, n_cols, K, A, W, C, nullptr, 1, N);
        }
        if (glu) return launch_pipe<2, 2, 4, 4, 3, 2, true>(s, OUT_T, M, n_cols, K, A, W, C, W2, 1, N);
        return launch_pipe<2, 2, 4, 4, 3, 2>(s, out_mode, M, n_cols, K, A, W, C, nullptr, 1, N);
    };
    const int tiles256 = nbm256 * nbn256;
    // one row of big tiles, a hundred or more of them, streams cold weights faster than twice as
    // many TA-bound small ones
    if (nbm256 == 1 && M > 128 && tiles256 >= 100 && N % bno256 == 0) {
        // more than a round of them (the LM head: 594 tiles): the whole rounds, then what is left in 256x128 tiles,
        // so that the last, partly filled round is half as long (best of four interleaved runs, M = 160 .. 256:
        // 287-312 us in one launch, 267-296 this way, 267-311 with a rest of 128x128 tiles; 32B shape 401-436 /
        // 372-410 / 369-435)
        const int main_tiles = tiles256 / 256 * 256;
        if (!glu && main_tiles > 0 && main_tiles < tiles256) {
            hipError_t e = big(main_tiles * 256);
            if (e != hipSuccess) return e;
            const void* w = (const uint16_t*)W + (int64_t)main_tiles * 256 * K;
            void* c = (char*)C + (size_t)main_tiles * 256 * c_elt;
            return launch_pipe<2, 2, 4, 2, 3, 4, false, true>(s, out_mode, M, N - main_tiles * 256, K, A, w, c, nullptr, 1, N);
        }
        // gate/up with well under a round of big tiles: 256 rows x 80 output columns per workgroup (four waves of
        // 64 rows x 5 column blocks of 16 gate and 16 up rows, the last tile partial) puts the weights on nearly all CUs, and the
        // narrower tile leaves room for a third weight slot.  What bounds it is a CU's load path, which the activation rows that
        // every workgroup re-reads from L2 share with the cold weights: 3.0 MB per workgroup in 64-69 us here (43-47 GB/s), 3.2 MB
        // in 77-79 us (41-42) with 96 columns and two slots.
        // Against 96 columns with two slots (three alternating runs on cold weights, M = 129 .. 256): 7B shape (198 -> 237
        // tiles) 77-79 -> 64-69 us, N 13824, K 5120 97-99 -> 80-85, N 20480, K 4096 88-93 -> 75-82.  Past 160 big tiles 80
        // columns would make more than a round (and 96 there gain nothing over the big tiles: N = 24576 102-105 -> 102-110).
        if (glu && tiles256 <= 160)
            return launch_pipe<4, 1, 2, 5, 3, 3, true, true>(s, OUT_T, M, N, K, A, W, C, W2, 1, N);
        return big(N);
    }
    // up to 128 rows: half of a 256-row tile would be padding, and the LDS it frees holds a third weight slot
    // (gate/up at M = 128: 85 -> 70 us, LM head: 261 -> 251; at the 32B shape 406 -> 343)
    // (from 33 rows on where whole rounds of them leave less than half a round: the wider tile re-reads the activation rows half as often.
    // N 152064, K 3584: 48 rows 201 us in 64-row tiles, 192 this way, 64 rows 210 and 198; K 5120: 300 and 277; at K 896 58.8 and 62.9)
    const bool wide64 = !glu && M > 32 && M <= 64 && K >= 2048 && tiles256 > 256 && tiles256 % 256 <= 128;
    if (((M > 64 && M <= 128) || wide64) && tiles256 >= 100 && N % bno256 == 0) {
        if (glu) return launch_pipe<2, 2, 2, 4, 3, 3, true, true>(s, OUT_T, M, N, K, A, W, C, W2, 1, N);
        // (more than a round: whole rounds, the rest in 128x128 tiles: LM head 227-250 -> 219-241 us, 32B shape 313-343 -> 297-325)
        const int main_tiles = tiles256 / 256 * 256;
        if (main_tiles > 0 && main_tiles < tiles256) {
            hipError_t e = launch_pipe<2, 2, 2, 4, 3, 3, false, true>(s, out_mode, M, main_tiles * 256, K, A, W, C, nullptr, 1, N);
            if (e != hipSuccess) return e;
            const void* w = (const uint16_t*)W + (int64_t)main_tiles * 256 * K;
            void* c = (char*)C + (size_t)main_tiles * 256 * c_elt;
            if (out_mode == OUT_F32 && N - main_tiles * 256 <= 96 * 256) return launch_mid_rest(s, M, N - main_tiles * 256, K, A, w, c, N);
            return launch_pipe<2, 2, 2, 2, 3, 3, false, true>(s, out_mode, M, N - main_tiles * 256, K, A, w, c, nullptr, 1, N);
        }
        return launch_pipe<2, 2, 2, 4, 3, 3, false, true>(s, out_mode, M, N, K, A, W, C, nullptr, 1, N);
    }
    if (M <= 64 || tiles256 < 256) return small(N, 0);
    const int full_rounds = tiles256 / 256;
    const int main_nbn = full_rounds * 256 / nbm256;          // column tiles that make up the whole rounds
    const int rest_cols = N - main_nbn * bno256;
    const int rest_tiles256 = tiles256 - main_nbn * nbm256 + (N % bno256 ? nbm256 : 0);
    if (main_nbn == 0) return N % bno256 == 0 ? big(N) : small(N, 0);
    if (rest_cols == 0) return big(N);
    if (rest_tiles256 >= 140 && N % bno256 == 0) return big(N);   // the last round is well filled as it is
    hipError_t e = big(main_nbn * bno256);
    if (e != hipSuccess) return e;
    // the rest in 256x128 tiles, one per CU (gate/up, best of four interleaved runs: M = 1536, a rest of 120 big
    // tiles: 331 us with 128x128 tiles, 323 this way, 347 in one launch of big tiles; M = 1024, rest 80: 249 /
    // 232 / 255; M = 2048, rest 160: 468 / 454 / 435)
    if (rest_cols % bno256 == 0) {
        const int col0 = main_nbn * bno256;
        const void* w = (const uint16_t*)W + (int64_t)col0 * K;
        const void* w2 = W2 ? (const uint16_t*)W2 + (int64_t)col0 * K : nullptr;
        void* c = (char*)C + (size_t)col0 * c_elt;
        if (glu) return launch_pipe<2, 2, 4, 2, 3, 4, true>(s, OUT_T, M, rest_cols, K, A, w, c, w2, 1, N);
        return launch_pipe<2, 2, 4, 2, 3, 4>(s, out_mode, M, rest_cols, K, A, w, c, nullptr, 1, N);
    }
    return small(rest_cols, main_nbn * bno256);
}

// How a product whose fp32 result is summed by its consumer is cut along K (bf16 MFMA path).  kind 0: not at all;
// 1: 256x128 tiles; 2: 256x256 tiles; 3: 128x128 tiles.
//
// The plan is the minimum of a small cost model over (tile shape, number of cuts).  A launch takes a ramp plus, for
// every round of workgroups the chip has to run (one per CU; 128x128 tiles past 256 workgroups share CUs in pairs and
// run slower), the K steps of a cut at the tile shape's clocks per step plus its epilogue; every cut after the first
// adds M*N*4 bytes that the consumer (the norm or rotary kernel that sums the slices) reads at ~4 TB/s.  The
// constants were fitted to a sweep on the chip (nine projection shapes of the 7B / 32B / 70B models, M = 96 .. 1536,
// kinds 1-3, 1-12 cuts, cold weights, best of three interleaved runs, even cuts): the model's pick is within 0.9 %
// of the best measured plan on average (worst case 11 %), where the rules it replaces were 7.8 % off on average and
// up to 49 % (M = 384 .. 1024).  Uneven cuts, which paid when the cuts accumulated with atomics, lost 3-5 % to even
// ones in the same sweep, so the cuts are even.
struct SplitPlan {
    int kind = 0, ks = 1, skew = 0;
};
static SplitPlan plan_split(int M, int N, int K, int max_ks = 12, double uncut_credit_us = 0.0) {
    SplitPlan sp;
    if (N % 128 != 0 || M < 1) return sp;
    const int nk = K / kBK;
    const int nbm256 = (M + 255) / 256, nbm128 = (M + 127) / 128;
    auto cost_us = [&](int kind, int ks) -> double {
        int tiles;
        double step_clk, epilogue_clk;
        if (kind == 1) tiles = nbm256 * (N / 128), step_clk = 1396, epilogue_clk = 9827;
        else if (kind == 2) tiles = nbm256 * (N / 256), step_clk = 2266, epilogue_clk = 18240;
        else tiles = nbm128 * (N / 128), step_clk = 988, epilogue_clk = 5754;
        const int wgs = tiles * ks;
        const double steps = (double)nk / ks;
        double clk;
        if (kind == 3 && wgs > 256) clk = (double)((wgs + 511) / 512) * (steps * 2390 + epilogue_clk);
        else clk = (double)((wgs + 255) / 256) * (steps * step_clk + epilogue_clk);
        return 1.6 + clk / 1800.0 + (ks - 1) * (double)M * N * 4.0 / 4.0e6;
    };
    // (not cut at all, the product takes the tiled launcher's own pick of a tile shape: the best of the three here
    // and of the 192x128 tiles that launcher has besides, 1259 clocks per step and 4000 of epilogue)
    double best = cost_us(1, 1);
    if (cost_us(3, 1) < best) best = cost_us(3, 1);
    if (N % 256 == 0 && cost_us(2, 1) < best) best = cost_us(2, 1);
    {
        const int t192 = ((M + 191) / 192) * (N / 128);
        const double c192 = 1.6 + (double)((t192 + 255) / 256) * (nk * 1259.0 + 4000.0) / 1800.0;
        if (c192 < best) best = c192;
    }
    best -= uncut_credit_us;   // (what the uncut product saves its caller besides, e.g. an output in the model dtype)
    if (max_ks > 12) max_ks = 12;
    for (int kind = 1; kind <= 3; ++kind) {
        if (kind == 2 && N % 256 != 0) continue;
        for (int ks = 2; ks <= max_ks && nk / ks >= 6; ++ks) {
            const double c = cost_us(kind, ks);
            if (c < best) {
                best = c;
                sp.kind = kind, sp.ks = ks, sp.skew = 0;
            }
        }
    }
    return sp;
}

static bool pipe_ok(int N, int K, const void* A, const void* W) {
    const bool aligned = (((uintptr_t)A | (uintptr_t)W) & 15) == 0;
    // per-lane DMA offsets are 32-bit byte offsets inside a 256-row panel
    return aligned && K % kBK == 0 && N % 128 == 0 && (int64_t)258 * K * 2 < ((int64_t)1 << 31);
}

hipError_t gemm(hipStream_t s, int dtype, int out_mode, int M, int N, int K, const void* A, const void* W, void* C) {
    if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
    if (dtype == F32)
        return f32_few_ok(M, K, A, W) && !f32_tiles_pay(M, N, K) ? launch_f32_few(s, out_mode, M, N, K, A, W, nullptr, C)
                                                                 : launch_generic<float>(s, out_mode, M, N, K, A, W, C);
    if (pipe_ok(N, K, A, W)) {
        // (accumulating into C: the K splits add their partial sums with fp32 atomics, in any order, so the
        // last bit of the result is not fixed.  The step itself uses gemm_parts, which is reproducible.)
        if (out_mode == OUT_ADD_F32) {
            const SplitPlan sp = plan_split(M, N, K);
            if (sp.kind == 1) return launch_pipe<2, 2, 4, 2, 3, 4>(s, out_mode, M, N, K, A, W, C, nullptr, sp.ks, 0, sp.skew);
            if (sp.kind == 2) return launch_pipe<2, 2, 4, 4, 3, 2>(s, out_mode, M, N, K, A, W, C, nullptr, sp.ks, 0, sp.skew);
            if (sp.kind == 3) return launch_pipe<2, 2, 2, 2, 3, 3>(s, out_mode, M, N, K, A, W, C, nullptr, sp.ks, 0, sp.skew);
        }
        return launch_tiled(s, out_mode, M, N, K, A, W, nullptr, C, false);
    }
    return launch_generic<bf16>(s, out_mode, M, N, K, A, W, C);
}

// room for the slices of the few-row products (at 256 rows 8 cuts of a 4608-wide product take 38 MB); a plan that
// does not fit the caller's buffer is cut less
// Whether the product as K-cut fp32 slices (gemm_parts) is expected to beat the same product stored once in the
// model dtype, counting the bytes the slices cost their reader and the writer over a bf16 result.
bool gemm_parts_pays(int dtype, int M, int N, int K) {
    if (dtype != BF16 || M < 1 || N % 128 != 0 || K % kBK != 0) return false;
    return plan_split(M, N, K, 12, (double)M * N * 4.0 / 4.0e6).kind != 0;
}

size_t gemm_parts_max_bytes() { return (size_t)256 * 65536 * 4 + 4096; }

hipError_t gemm_parts(hipStream_t s, int dtype, int M, int N, int K, const void* A, const void* W, float* parts,
                      size_t parts_bytes, int* n_parts) {
    *n_parts = 1;
    if (M <= 0 || N <= 0 || K <= 0) return hipSuccess;
    if ((size_t)M * N * 4 > parts_bytes) return hipErrorInvalidValue;
    if (dtype == BF16 && pipe_ok(N, K, A, W)) {
        const size_t room = parts_bytes / ((size_t)M * N * 4);
        const SplitPlan sp = plan_split(M, N, K, room > 12 ? 12 : (int)room);
        if (M <= 32) {
            int cuts = 1;
            const int wtn = few_split_plan(N, K, sp.ks, room > 12 ? 12 : (int)room, &cuts);
            if (wtn != 0) *n_parts = cuts;
            if (wtn == 2) return launch_few<2, false>(s, M, N, K, A, W, nullptr, parts, cuts);
            if (wtn == 3) return launch_few<3, false>(s, M, N, K, A, W, nullptr, parts, cuts);
            if (wtn == 4) return launch_few<4, false>(s, M, N, K, A, W, nullptr, parts, cuts);
        }
        int mid_cuts = 0;
        if (mid_split_plan(M, N, K, sp.ks, room > 12 ? 12 : (int)room, &mid_cuts)) {
            *n_parts = mid_cuts;
            return launch_mid_parts(s, M, N, K, A, W, parts, mid_cuts);
        }
        if (sp.kind != 0 && (size_t)sp.ks * M * N * 4 <= parts_bytes) {
            *n_parts = sp.ks;
            if (sp.kind == 1) return launch_pipe<2, 2, 4, 2, 3, 4>(s, OUT_SPLIT_F32, M, N, K, A, W, parts, nullptr, sp.ks, 0, sp.skew);
            // (tiles of 64 rows, see launch_tiled: N = K = 3584 9.9 -> 9.3 us at 64 rows, N 4608 10.6 -> 10.0, N 3584, K 18944 26.8 -> 24.8 at
            // 40 rows and 26.5 -> 26.2 at 64; the sums are the same bit for bit)
            if (sp.kind == 3 && M <= 64)
                return launch_pipe<1, 4, 2, 1, 3, 3, false, true>(s, OUT_SPLIT_F32, M, N, K, A, W, parts, nullptr, sp.ks, 0, sp.skew);
            if (sp.kind == 3 && M <= 128)
                return launch_pipe<2, 2, 2, 2, 3, 3, false, true>(s, OUT_SPLIT_F32, M, N, K, A, W, parts, nullptr, sp.ks, 0, sp.skew);
            if (sp.kind == 3) return launch_pipe<2, 2, 2, 2, 3, 3>(s, OUT_SPLIT_F32, M, N, K, A, W, parts, nullptr, sp.ks, 0, sp.skew);
            return launch_pipe<2, 2, 4, 4, 3, 2>(s, OUT_SPLIT_F32, M, N, K, A, W, parts, nullptr, sp.ks, 0, sp.skew);
        }
    }
    return gemm(s, dtype, OUT_F32, M, N, K, A, W, parts);
}

// ---- fused row argmax (big tiles only: every 256-row weight tile yields two 128-column blocks)
// (a workgroup per row: its blocks, five per thread at 152064 columns, are all requested at once; a wave per row took 11.4 us
// at 84 rows, this 4.9)
__global__ __launch_bounds__(256) void argmax_blocks_k(int P, const float* __restrict__ pv, const int32_t* __restrict__ pi, int32_t* __restrict__ out) {
    __shared__ float sv[4];
    __shared__ int si[4];
    const int64_t row = (int64_t)blockIdx.x * P;
    float v = -INFINITY;
    int i = 0x7fffffff;
    for (int p0 = threadIdx.x; p0 < P; p0 += 256 * 8) {
        float ov[8];
        int oi[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool on = p0 + 256 * u < P;
            ov[u] = on ? pv[row + p0 + 256 * u] : -INFINITY;
            oi[u] = on ? pi[row + p0 + 256 * u] : 0x7fffffff;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (better(ov[u], oi[u], v, i)) v = ov[u], i = oi[u];
    }
    wave_best(v, i);
    if ((threadIdx.x & 63) == 0) sv[threadIdx.x >> 6] = v, si[threadIdx.x >> 6] = i;
    __syncthreads();
    if (threadIdx.x != 0) return;
#pragma unroll
    for (int w = 1; w < 4; ++w)
        if (better(sv[w], si[w], v, i)) v = sv[w], i = si[w];
    out[blockIdx.x] = i;
}

bool gemm_argmax_supported(int dtype, int M, int N, int K, const void* A, const void* W) {
    const bool aligned = (((uintptr_t)A | (uintptr_t)W) & 15) == 0;
    return dtype == BF16 && M > 64 && aligned && K % kBK == 0 && K / kBK >= 3 && N % 256 == 0 &&
           (int64_t)258 * K * 2 < ((int64_t)1 << 31);
}

size_t gemm_argmax_workspace_bytes(int M, int N) { return (size_t)M * (N / 128) * 8; }

// One launch of the row-maximum kernel over the columns col0 .. col0 + n_cols - 1, a multiple of its tile's width.
template <int WGM, int WGN, int WTM, int SA, int SB, bool NTW>
static hipError_t launch_rowmax(hipStream_t s, int M, int N, int K, const void* A, const void* W, float* pv, int32_t* pi, int col0, int n_cols) {
    constexpr int BM = 32 * WTM * WGM, BN = 128 * WGN;   // (four column tiles per wave: blocks of 128 columns)
    const int P = N / 128, nbm = (M + BM - 1) / BM, total = nbm * (n_cols / BN), per_xcd = (total + 7) / 8;
    const size_t lds = ((size_t)SA * BM + (size_t)SB * BN) * 64 * sizeof(uint16_t);
    const bool persistent = K / 64 >= (SA > SB ? SA : SB);   // (see launch_pipe)
    const int wg_per_xcd = !persistent || per_xcd < 32 ? per_xcd : 32;
    auto kern = gemm_bf16_pipe_k<WGM, WGN, WTM, 4, SA, SB, OUT_ROWMAX, false, NTW>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(wg_per_xcd * 8), dim3(64 * WGM * WGN), lds, s, M, P, K, (const uint16_t*)A, (const uint16_t*)W + (int64_t)col0 * K,
                       (const uint16_t*)nullptr, (void*)(pv + col0 / 128), nbm, total, per_xcd, 1, wg_per_xcd, pi + col0 / 128, 0, (int64_t)col0,
                       n_cols);
    return hipGetLastError();
}

hipError_t gemm_argmax(hipStream_t s, int M, int N, int K, const void* A, const void* W, void* ws, int32_t* out) {
    const int P = N / 128;
    float* pv = (float*)ws;
    int32_t* pi = (int32_t*)(pv + (size_t)M * P);
    hipError_t e;
    if (M <= 256) {
        // one row of tiles: whole rounds of the chip in 256-column tiles, what is left in 128-column ones (as launch_tiled cuts the stored
        // product), weights with the non-temporal hint; up to 128 rows in tiles of 128 rows.  N 152064, K 3584, us against 256x256 tiles in
        // one launch: 65 rows 280 -> 232, 128 rows 277 -> 233, 129 rows 281 -> 251, 256 rows 301 -> 283.
        const int tiles = N / 256, main_cols = (tiles > 256 ? tiles / 256 * 256 : tiles) * 256;
        if (M <= 128) e = launch_rowmax<2, 2, 2, 3, 3, true>(s, M, N, K, A, W, pv, pi, 0, main_cols);
        else e = launch_rowmax<2, 2, 4, 3, 2, true>(s, M, N, K, A, W, pv, pi, 0, main_cols);
        if (e != hipSuccess) return e;
        if (main_cols < N) {
            if (M <= 128) e = launch_rowmax<2, 1, 2, 3, 4, true>(s, M, N, K, A, W, pv, pi, main_cols, N - main_cols);
            else e = launch_rowmax<4, 1, 2, 3, 4, true>(s, M, N, K, A, W, pv, pi, main_cols, N - main_cols);
        }
    } else {
        e = launch_rowmax<2, 2, 4, 3, 2, false>(s, M, N, K, A, W, pv, pi, 0, N);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(argmax_blocks_k, dim3(M), dim3(256), 0, s, P, pv, pi, out);
    return hipGetLastError();
}

bool gemm_glu_supported(int dtype, int M, int N, int K, const void* A, const void* Wg, const void* Wu) {
    if (dtype == F32) return M > 0 && f32_few_ok(M, K, A, Wg, Wu);
    const bool aligned = (((uintptr_t)A | (uintptr_t)Wg | (uintptr_t)Wu) & 15) == 0;
    return M > 0 && aligned && K % kBK == 0 && N % 128 == 0 && (int64_t)258 * K * 2 < ((int64_t)1 << 31);
}

// act[M][N] = silu(A Wg^T) * (A Wu^T), dtype in and out; call only when gemm_glu_supported().
hipError_t gemm_glu(hipStream_t s, int dtype, int M, int N, int K, const void* A, const void* Wg, const void* Wu, void* act) {
    if (dtype == F32) return launch_f32_few(s, OUT_F32, M, N, K, A, Wg, Wu, act);
    if (const int wtn = mid_glu_width(M, N, K)) return launch_mid_glu(s, wtn, M, N, K, A, Wg, Wu, act);
    if (const int wtn = few_glu_width(M, N, K)) return launch_few_glu(s, wtn, M, N, K, A, Wg, Wu, act);
    return launch_tiled(s, OUT_T, M, N, K, A, Wg, Wu, act, true);
}

// ---- measurement aid: what the matrix pipes sustain with nothing else running ----
// Every wave (one per SIMD of every CU) loops over the 16 x 4 MFMAs of a 128x128 wave tile and a 64-wide K tile,
// in the GEMM kernel's issue order, on register operands that never change: no LDS, no memory, no waits.  On
// random data the chip holds about 1.8 GHz under its power limit here, so the rate this loop reaches, not the
// 2.4 GHz figure, is what a GEMM kernel's share of the peak is to be read against.
__global__ __launch_bounds__(256) void mfma_stream_k(const u32x4_t* __restrict__ frags, float* __restrict__ out, int iters) {
    const int lane = threadIdx.x & 63;
    bf16x8_t fa[4][4], fb[4][4];   // [K slice of 16][fragment]
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            fa[s][i] = __builtin_bit_cast(bf16x8_t, frags[(s * 8 + i) * 64 + lane]);
            fb[s][i] = __builtin_bit_cast(bf16x8_t, frags[(s * 8 + 4 + i) * 64 + lane]);
        }
    f32x16_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int jj = (i & 1) ? 3 - j : j;
                    acc[i][jj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][i], fb[s][jj], acc[i][jj], 0, 0, 0);
                }
        __builtin_amdgcn_sched_barrier(0);
    }
    float sum = 0.f;   // in a fixed order: i, then j, then the lane's 16 elements
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) sum += acc[i][j][v];
    out[blockIdx.x * 256 + threadIdx.x] = sum;
}

hipError_t mfma_stream(hipStream_t s, const void* frags, float* out, int iters) {
    hipLaunchKernelGGL(mfma_stream_k, dim3(kMfmaStreamBlocks), dim3(256), 0, s, (const u32x4_t*)frags, out, iters);
    return hipGetLastError();
}

}  // namespace tlt

// bf16 GEMM tiles for gfx950 on eight wavefronts that take turns at the matrix cores: 256 x 256, 256 x 128 and 128 x 256, K in
// steps of 64.
//
// What bounds them.  On random operands board power (see gemm_bf16.hip): per flop the large tile moves the fewest bytes through
// LDS and L2 of the kernels here, and its matrix instruction (16x16x32) is the cheap one.  On zeros 1880 (NT), 1900 (NN) and
// 1870 TFLOP/s (TN) at 8192^3, random 1413, 1497 and 1431, where the best kernel of gemm_bf16.hip for each layout reaches
// 1337, 1360 and 1359 (fetch and math wavefronts NT, the 256 x 256 tile of four wavefronts NN and TN); at 4096^3, one tile per
// compute unit, 100 us (NT) and 103 us (TN) against 116 and 110.
//
// Turns (the schedule publicly described as ping-pong for this family of chips; fragments, units and waits are worked out here).
// Wavefronts w and w + 4 share a SIMD.  The product of a step is cut into clusters (a unit of A times a unit of B); for
// each a wavefront first reads what is missing of its fragments and issues loads (memory phase), then runs 16 matrix
// instructions on them (matrix phase), with a workgroup barrier behind either phase.  Wavefronts 4..7 are one phase behind, so
// of the two on a SIMD one always has matrix instructions to issue while the other waits for LDS.  The fragments of a cluster
// are read right before it: 128 accumulators, 80 fragment registers and the addresses fit 256.
//
// LDS.  A stage holds 64 k (a whole cache line of a K-major row) in units that are handed back to the loads one by one: a unit
// that is read in one cluster is loaded again from the next on.
//   256 x 256: wavefronts 2 x 4, two stages of B0, A0, B1, A1, 128 rows (columns) each; four clusters per step, and two loads in
//              each, eight clusters before their unit is read: 12 to 14 KiB per wavefront in flight
//   256 x 128: wavefronts 4 x 2, three stages of A (256 rows), B0, B1 (64 columns each); two clusters per step; loads five
//              clusters ahead.  Half the columns are for GEMMs of few tiles.
//   128 x 256: wavefronts 2 x 4, three stages of A (128 rows), B0, B1 (128 columns each), else as 256 x 128.  For GEMMs of at most 128
//              rows, which stream B: a step takes 1.0 us, and 168 workgroups of it 4.8 TB/s, 210 5.4.
//
// Which rows and columns a wavefront owns: rows 64 wm .. + 63 of each unit of A, columns 32 wn .. + 31 of each unit of B.  The
// blocks of C are computed transposed, and the two blocks of such 32 columns take turns at groups of four columns, so that a
// lane ends up with 8 consecutive columns of a row: 16 bytes of bf16.  So results go from the accumulators to memory without
// passing through LDS, 64 contiguous bytes per row.
#pragma once
#include "gemm_bf16_common.h"

namespace tpl {

template <int WM_, int UA_>
struct PPTile {
    static constexpr int WM = WM_, WN = 8 / WM_;                          // wavefronts by rows and columns
    static constexpr int UA = UA_, STAGES = UA == 2 ? 2 : 3;              // units of A in a stage
    static constexpr int A_ROWS = 64 * WM, B_COLS = 32 * WN;              // rows (columns) of a unit
    static constexpr int BM = UA * A_ROWS, BN = 2 * B_COLS;
    static constexpr int A_UNIT = A_ROWS * 128, B_UNIT = B_COLS * 128;    // bytes
    static constexpr int A_STAGE = UA * A_UNIT, B_STAGE = 2 * B_UNIT;
    static constexpr int LA = A_ROWS / 64, LB = B_COLS / 64;              // loads of a unit by one wavefront, 1 KiB each
    static constexpr int CS_BYTES = WN * 16 * 4 * 2 * 4;                  // column sums of the finished runs
    static constexpr int LDS_BYTES = STAGES * (A_STAGE + B_STAGE) + CS_BYTES;
    static constexpr int FLOATS = BM * BN;
};
template <typename TL> using PPAcc = f32x4[TL::UA][4][4];                 // [unit of A][16 rows][block of 16 columns: B0, B0, B1, B1]

// Some of a GEMM's tiles: `count` from `tile0` on, K cut into shares of nk k-steps (an even number where there are several).
// partial: the sums of (share, tile) as the accumulators hold them, see pp_partial; null where K is whole.
struct PPRun { int tile0, count, nk; float* partial; };

// acc += F_b F_a: rows of the block are columns of C
__device__ __forceinline__ void mfma16_pp(f32x4& acc, const bf16x8& b, const bf16x8& a) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}

// Positions of the 16-byte chunks of a unit in LDS, free of bank conflicts for the reads below.
// K-major, 128-byte rows: chunk c of row r at c ^ f(r).  The 16 rows of a fragment of B are groups of four, one of every eight.
template <bool IS_B> __device__ __forceinline__ int pp_swz_k(int row) {
    return IS_B ? ((row >> 1) & 1) | (((row >> 3) & 3) << 1) : swz_k64(row);
}
// MN-major, R columns per k: chunk c of row k at c ^ f(k).  A fragment of B takes one half of every chunk of a 64-byte group, so
// the rows k and k + 8 that are read together swap neighbouring chunks.
template <bool IS_B, int R> __device__ __forceinline__ int pp_swz_mn(int c, int k) {
    if (!IS_B) return mn_swz<R>(c, k);
    return c ^ (R == 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2) ^ ((k >> 3) & 1);
}
// K-major: the k chunk that a lane loads of block `block` (1 KiB, 8 rows) of a unit
template <bool IS_B> __device__ __forceinline__ int pp_chunk(int block, int lane) {
    return (lane & 7) ^ pp_swz_k<IS_B>(block * 8 + (lane >> 3));
}
// Byte offsets of the R / 64 loads of a unit (R rows or columns x 64 k) by one wavefront.
template <bool KMAJ, bool IS_B, int R>
__device__ __forceinline__ void pp_offsets(unsigned (&off)[R / 64], int ld, int mn0, int MN, int wave, int lane) {
#pragma unroll
    for (int j = 0; j < R / 64; ++j) {
        const int block = wave * (R / 64) + j;
        if (KMAJ) {
            const int row = block * 8 + (lane >> 3);
            off[j] = mn0 + row < MN ? (unsigned)(((int64_t)(mn0 + row) * ld + pp_chunk<IS_B>(block, lane) * 8) * 2) : OOB_HALF;
        } else {
            const int idx = block * 64 + lane, k = idx / (R / 8), c = pp_swz_mn<IS_B, R>(idx % (R / 8), k);   // its own inverse
            off[j] = mn0 + c * 8 < MN ? (unsigned)(((int64_t)k * ld + mn0 + c * 8) * 2) : OOB_HALF;
        }
    }
}
// Loads 64 k from k0 on of a unit.  K-major: past the end of the K share a lane reads nothing; it may lie inside the last step.
// MN-major: a share ends with a step or with the buffer.
template <bool KMAJ, bool IS_B, int NL>
__device__ __forceinline__ void pp_load(i32x4 r, unsigned dst, const unsigned (&off)[NL], int k0, int kend, unsigned kbytes, int wave, int lane) {
    const unsigned so = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)k0 * kbytes));
    if (!KMAJ) r[2] = k0 < kend ? r[2] : 0;
    if (!KMAJ || k0 + 64 <= kend) {
#pragma unroll
        for (int j = 0; j < NL; ++j) buffer_load_lds_b128_s(r, dst + (wave * NL + j) * 1024, off[j], so);
    } else {
        int l = lane;
        asm volatile("" : "+v"(l));                                       // worked out here, not kept in registers over the loop
#pragma unroll
        for (int j = 0; j < NL; ++j)
            buffer_load_lds_b128(r, dst + (wave * NL + j) * 1024,
                                 k0 + pp_chunk<IS_B>(wave * NL + j, l) * 8 < kend && off[j] != OOB_HALF ? off[j] + so : OOB_HALF);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// A fragment (16 rows x 32 k) at LDS address addr + IMM; PITCH: bytes per k of an MN-major unit.
template <bool KMAJ, int IMM, int PITCH>
__device__ __forceinline__ bf16x8 pp_read(unsigned addr) {
    if constexpr (KMAJ) {
        typedef __attribute__((address_space(3))) const bf16x8* p_t;
        return *reinterpret_cast<p_t>((uintptr_t)(addr + IMM));
    } else {
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(addr + IMM));
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(addr + IMM + 4 * PITCH));
        const bf16x4 b0 = __builtin_bit_cast(bf16x4, v0), b1 = __builtin_bit_cast(bf16x4, v1);
        bf16x8 o;
        o[0] = b0[0]; o[1] = b0[1]; o[2] = b0[2]; o[3] = b0[3];
        o[4] = b1[0]; o[5] = b1[1]; o[6] = b1[2]; o[7] = b1[3];
        return o;
    }
}

// ---- epilogue ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ int pp_wave() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }
// What a lane writes: row `row` + 16 i of each unit of A, 8 columns from `col[u]` on for either unit of B.
struct PPLane {
    int row, col[2];
    bool odd;                         // the blocks of a pair hold their column groups in swapped order in odd lane groups
    float bias[16];
};
template <typename TL>
__device__ __forceinline__ PPLane pp_lane(const GemmParams& p, int m0, int n0) {
    const int lane = threadIdx.x & 63, wave = pp_wave(), wm = wave / TL::WN, wn = wave % TL::WN, g = lane >> 4;
    PPLane el;
    el.row = m0 + wm * 64 + (lane & 15);
    el.odd = g & 1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        el.col[u] = n0 + u * TL::B_COLS + wn * 32 + 8 * g;
        float b8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (p.bias && el.col[u] < p.N) unpack8(*reinterpret_cast<const uint4*>(p.bias + el.col[u]), b8);
#pragma unroll
        for (int e = 0; e < 8; ++e) el.bias[8 * u + e] = b8[e];
    }
    return el;
}
template <int KIND>
__device__ __forceinline__ uint4 pp_fetch(const GemmParams& p, int row, int col) {       // residual or GeLU input
    uint4 v = make_uint4(0, 0, 0, 0);
    if ((KIND == KIND_RESID || KIND == KIND_DGELU) && row < p.M && col < p.N)
        v = *reinterpret_cast<const uint4*>((KIND == KIND_RESID ? p.resid : p.aux) + (int64_t)row * p.N + col);
    return v;
}
template <int KIND>
__device__ __forceinline__ void pp_emit(const GemmParams& p, int row, int col, float (&v)[8], const float* bias, const uint4& in) {
    if (row >= p.M || col >= p.N) return;
    const int64_t idx = (int64_t)row * p.N + col;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += bias[e];
    if (KIND == KIND_RESID || (KIND == KIND_ANY && p.resid)) {
        float r8[8];
        unpack8(KIND == KIND_RESID ? in : *reinterpret_cast<const uint4*>(p.resid + idx), r8);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += r8[e];
    }
    if (KIND == KIND_GELU || (KIND == KIND_ANY && p.epi == EPI_GELU)) {
        *reinterpret_cast<uint4*>(p.aux + idx) = pack8(v);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = gelu_f(v[e]);
    } else if (KIND == KIND_DGELU || (KIND == KIND_ANY && p.epi == EPI_DGELU)) {
        float u8[8];
        unpack8(KIND == KIND_DGELU ? in : *reinterpret_cast<const uint4*>(p.aux + idx), u8);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_f(u8[e]);
    }
    const uint4 o = pack8(v);
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 o4 = {o.x, o.y, o.z, o.w};
    if (p.nt_store) __builtin_nontemporal_store(o4, reinterpret_cast<u32x4*>(p.C + idx));
    else *reinterpret_cast<u32x4*>(p.C + idx) = o4;
}
// A block of 16 rows of the wavefront: x[j] holds 4 columns of block j.
template <int KIND>
__device__ __forceinline__ void pp_row_block(const GemmParams& p, const PPLane& el, int row, const f32x4 (&x)[4], const uint4 (&in)[2]) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = el.odd ? x[2 * u + 1][e] : x[2 * u][e];
            v[4 + e] = el.odd ? x[2 * u][e] : x[2 * u + 1][e];
        }
        pp_emit<KIND>(p, row, el.col[u], v, el.bias + 8 * u, in[u]);
    }
}
template <typename TL, int KIND>
__device__ __forceinline__ void pp_rows(const GemmParams& p, const PPAcc<TL>& acc, const PPLane& el) {
    uint4 in[4][2];                       // requested a unit of A ahead
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u) in[i][u] = pp_fetch<KIND>(p, el.row + i * 16, el.col[u]);
    f32x4 x[4][4];                        // the present unit: one body for both, code that runs once per tile comes from memory
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[i][j] = acc[0][i][j];
#pragma unroll 1
    for (int h = 0; h < TL::UA; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = el.row + h * TL::A_ROWS + i * 16;
            pp_row_block<KIND>(p, el, row, x[i], in[i]);
            if (h + 1 < TL::UA) {
#pragma unroll
                for (int u = 0; u < 2; ++u) in[i][u] = pp_fetch<KIND>(p, row + TL::A_ROWS, el.col[u]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) x[i][j] = acc[TL::UA - 1][i][j];
        }
    }
}
// Partial sums of a K share: 16 bytes per lane, block by block; blocks of rows past M are left out.
__device__ __forceinline__ float4* pp_partial(float* tile, int block) {
    return reinterpret_cast<float4*>(tile) + block * 4 * 512 + threadIdx.x;
}
template <typename TL, int BLOCK>
__device__ __forceinline__ void pp_store_partial(const GemmParams& p, const PPAcc<TL>& acc, int row0, float* partial) {
    if constexpr (BLOCK < 4 * TL::UA) {
        if (row0 + (BLOCK >> 2) * TL::A_ROWS + (BLOCK & 3) * 16 < p.M) {
            float4* dst = pp_partial(partial, BLOCK);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4& a = acc[BLOCK >> 2][BLOCK & 3][j];
                dst[j * 512] = make_float4(a[0], a[1], a[2], a[3]);
            }
        }
        pp_store_partial<TL, BLOCK + 1>(p, acc, row0, partial);
    }
}
template <typename TL>
__device__ __forceinline__ void pp_epilogue(const GemmParams& p, const PPAcc<TL>& acc, int m0, int n0, float* partial) {
    if (partial) {
        pp_store_partial<TL, 0>(p, acc, m0 + pp_wave() / TL::WN * 64, partial);
        return;
    }
    const PPLane el = pp_lane<TL>(p, m0, n0);
    if (p.epi == EPI_NONE && !p.resid) pp_rows<TL, KIND_PLAIN>(p, acc, el);
    else if (p.epi == EPI_NONE) pp_rows<TL, KIND_RESID>(p, acc, el);
    else if (p.epi == EPI_GELU && !p.resid) pp_rows<TL, KIND_GELU>(p, acc, el);
    else if (p.epi == EPI_DGELU && !p.resid) pp_rows<TL, KIND_DGELU>(p, acc, el);
    else pp_rows<TL, KIND_ANY>(p, acc, el);
}
// Row block `block` of tile `local` of a run whose K was cut: the shares' sums in share order, then the epilogue.
template <typename TL>
__device__ __forceinline__ void pp_sum_rows(const GemmParams& p, const PPRun& r, int shares, int local, int block) {
    int tm, tn;
    tile_coords(r.tile0 + local, p.tiles_m, p.tiles_n, p.band, tm, tn);
    const int m0 = tm * TL::BM, n0 = tn * TL::BN;
    const PPLane el = pp_lane<TL>(p, m0, n0);
    const int row = el.row + (block >> 2) * TL::A_ROWS + (block & 3) * 16;
    if (__builtin_amdgcn_readfirstlane(row - (int)(threadIdx.x & 15)) < p.M) {
        f32x4 x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[j][v] = 0.0f;
        for (int s = 0; s < shares; ++s) {
            const float4* src = pp_partial(r.partial + ((int64_t)s * r.count + local) * TL::FLOATS, block);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 y = src[j * 512];
                x[j][0] += y.x; x[j][1] += y.y; x[j][2] += y.z; x[j][3] += y.w;
            }
        }
        const uint4 none[2] = {};
        pp_row_block<KIND_ANY>(p, el, row, x, none);
    }
    const int col = n0 + (int)threadIdx.x;
    if (block == 0 && tm == 0 && p.colsum && threadIdx.x < TL::BN && col < p.N) {
        float v = 0.0f;
        for (int s = 0; s < shares; ++s) v += p.colsum_part[(int64_t)s * p.N + col];
        p.colsum[col] = (bf16_t)v;
    }
}

// ---- products ---------------------------------------------------------------------------------------------------------
struct PPWork { int tm, m0, n0, k0, kend, share; float* partial; };
template <typename TL>
__device__ __forceinline__ PPWork pp_work(const GemmParams& p, const PPRun& r, int pos) {
    PPWork w;
    w.share = pos / r.count;
    int tn;
    tile_coords(r.tile0 + pos - w.share * r.count, p.tiles_m, p.tiles_n, p.band, w.tm, tn);
    w.m0 = w.tm * TL::BM;
    w.n0 = tn * TL::BN;
    w.k0 = w.share * r.nk * DK;
    w.kend = w.k0 + r.nk * DK < p.K ? w.k0 + r.nk * DK : p.K;
    w.partial = r.partial ? r.partial + (int64_t)pos * TL::FLOATS : nullptr;
    return w;
}

// COLSUM: with p.colsum set, the wavefronts that hold the first rows of tile row 0 also add up the columns of B over k (the bias
// gradient that goes with a weight gradient) from the fragments they multiply, in their own copy of the loop.
template <typename TL, bool A_KMAJ, bool B_KMAJ, bool COLSUM>
__device__ __forceinline__ void pp_products(const GemmParams& p, const PPWork& w, char* smem, PPAcc<TL>& acc) {
    constexpr int AR = TL::A_ROWS, BC = TL::B_COLS;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = pp_wave(), wm = wave / TL::WN, wn = wave % TL::WN;
    const bool late = wave >= 4;                                          // one phase behind
    const int m0 = w.m0, n0 = w.n0, ns = (w.kend - w.k0 + 63) / 64;

    const i32x4 ra = make_rsrc(p.A, (unsigned)((int64_t)(A_KMAJ ? p.M : p.K) * p.lda * 2));
    const i32x4 rb = make_rsrc(p.B, (unsigned)((int64_t)(B_KMAJ ? p.N : p.K) * p.ldb * 2));
    const unsigned lds_a = (unsigned)(uintptr_t)(lds_void_ptr)smem, lds_b = lds_a + TL::STAGES * TL::A_STAGE;
    unsigned oa[TL::UA][TL::LA], ob[2][TL::LB];
#pragma unroll
    for (int u = 0; u < TL::UA; ++u) pp_offsets<A_KMAJ, false, AR>(oa[u], p.lda, m0 + u * AR, p.M, wave, lane);
#pragma unroll
    for (int u = 0; u < 2; ++u) pp_offsets<B_KMAJ, true, BC>(ob[u], p.ldb, n0 + u * BC, p.N, wave, lane);
    const unsigned ka_bytes = A_KMAJ ? 2u : (unsigned)p.lda * 2u, kb_bytes = B_KMAJ ? 2u : (unsigned)p.ldb * 2u;
    auto load_a = [&](auto uc, int s, int stage) __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value;
        pp_load<A_KMAJ, false>(ra, lds_a + stage * TL::A_STAGE + U * TL::A_UNIT, oa[U], w.k0 + 64 * s, w.kend, ka_bytes, wave, lane);
    };
    auto load_b = [&](auto uc, int s, int stage) __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value;
        pp_load<B_KMAJ, true>(rb, lds_b + stage * TL::B_STAGE + U * TL::B_UNIT, ob[U], w.k0 + 64 * s, w.kend, kb_bytes, wave, lane);
    };

    // LDS addresses of this lane's fragment reads in unit 0 of stage 0.  K-major: by half of the 64 k (and block of B);
    // MN-major: by block.
    unsigned aaddr[4], baddr[2][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = wm * 64 + l16, k = 8 * lq + (l16 >> 2), mn = wm * 64 + i * 16 + 4 * (l16 & 3);
        if (A_KMAJ) aaddr[i] = lds_a + row * 128 + (((lq + 4 * (i & 1)) ^ pp_swz_k<false>(row)) << 4);
        else aaddr[i] = lds_a + k * (2 * AR) + (pp_swz_mn<false, AR>(mn >> 3, k) << 4) + (mn & 7) * 2;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            if (B_KMAJ) {
                const int q = l16 >> 2, row = wn * 32 + 8 * q + 4 * ((q ^ j) & 1) + (l16 & 3);
                baddr[j][ks] = lds_b + row * 128 + (((lq + 4 * ks) ^ pp_swz_k<true>(row)) << 4);
            } else {
                const int k = 8 * lq + (l16 >> 2), q = l16 & 3;
                baddr[j][ks] = lds_b + k * (2 * BC) + (pp_swz_mn<true, BC>(wn * 4 + q, k) << 4) + 8 * ((q ^ j) & 1);
            }
        }

#pragma unroll
    for (int h = 0; h < TL::UA; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[h][i][j][v] = 0.0f;
    bf16x8 fa[4][2], fb0[TL::UA][2][2], fb1[2][2];                        // [..][half of the 64 k]
    auto read_a = [&](auto uc, auto pc) __attribute__((always_inline)) {
        constexpr int UNIT = decltype(pc)::value * TL::A_STAGE + decltype(uc)::value * TL::A_UNIT;
        if constexpr (A_KMAJ) {
            fa[0][0] = pp_read<true, UNIT, 0>(aaddr[0]); fa[0][1] = pp_read<true, UNIT, 0>(aaddr[1]);
            fa[1][0] = pp_read<true, UNIT + 2048, 0>(aaddr[0]); fa[1][1] = pp_read<true, UNIT + 2048, 0>(aaddr[1]);
            fa[2][0] = pp_read<true, UNIT + 4096, 0>(aaddr[0]); fa[2][1] = pp_read<true, UNIT + 4096, 0>(aaddr[1]);
            fa[3][0] = pp_read<true, UNIT + 6144, 0>(aaddr[0]); fa[3][1] = pp_read<true, UNIT + 6144, 0>(aaddr[1]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                fa[i][0] = pp_read<false, UNIT, 2 * AR>(aaddr[i]);
                fa[i][1] = pp_read<false, UNIT + 32 * 2 * AR, 2 * AR>(aaddr[i]);
            }
        }
    };
    auto read_b = [&](auto uc, auto pc, bf16x8 (&dst)[2][2]) __attribute__((always_inline)) {
        constexpr int UNIT = decltype(pc)::value * TL::B_STAGE + decltype(uc)::value * TL::B_UNIT;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if constexpr (B_KMAJ) {
                dst[j][0] = pp_read<true, UNIT, 0>(baddr[j][0]);
                dst[j][1] = pp_read<true, UNIT, 0>(baddr[j][1]);
            } else {
                dst[j][0] = pp_read<false, UNIT, 2 * BC>(baddr[j][0]);
                dst[j][1] = pp_read<false, UNIT + 32 * 2 * BC, 2 * BC>(baddr[j][0]);
            }
        }
    };
    auto meet = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    // End of a memory phase: all but the NEWER last loads have landed (what the next cluster reads among them), and this
    // cluster's fragments are in registers.
    auto arrived = [&](auto newer) __attribute__((always_inline)) {
        wait_vmcnt<decltype(newer)::value>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        meet();
    };
    float cs[4];                                                          // a lane's part of the column sums, see end_run
    auto mul = [&](auto ac, auto bc, const bf16x8 (&fb)[2][2], auto csc) __attribute__((always_inline)) {
        constexpr int U = decltype(ac)::value, J0 = 2 * decltype(bc)::value;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    mfma16_pp(acc[U][i][J0 + j], fb[j][ks], fa[i][ks]);
                    __builtin_amdgcn_sched_barrier(0);
                }
        if constexpr (decltype(csc)::value && U == 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j) cs[J0 + j] = add_elements(fb[j][1], add_elements(fb[j][0], cs[J0 + j]));
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        meet();
    };
    using C0 = std::integral_constant<int, 0>; using C1 = std::integral_constant<int, 1>; using C2 = std::integral_constant<int, 2>;
    auto step = [&](int s, auto pc, auto csc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        if constexpr (TL::UA == 2) {
            // loads in issue order: B0(s+2), A0(s+2), B1(s+2), A1(s+2), two each; six units newer than the one that is read next
            constexpr int NEXT = P ^ 1;
            using W = std::integral_constant<int, 12>;
            read_a(C0{}, pc);
            load_b(C0{}, s + 2, P);
            arrived(W{});                                                 // B1(s)
            mul(C0{}, C0{}, fb0[P], csc);
            read_b(C1{}, pc, fb1);
            load_a(C0{}, s + 2, P);
            arrived(W{});                                                 // A1(s)
            mul(C0{}, C1{}, fb1, csc);
            read_a(C1{}, pc);
            load_b(C1{}, s + 2, P);
            arrived(W{});                                                 // B0(s+1)
            mul(C1{}, C1{}, fb1, csc);
            read_b(C0{}, std::integral_constant<int, NEXT>{}, fb0[NEXT]);
            load_a(C1{}, s + 2, P);
            arrived(W{});                                                 // A0(s+1)
            mul(C1{}, C0{}, fb0[P], csc);
        } else {
            // loads in issue order: B1(s+2), B0(s+3), LB each, and A(s+3), LA; newer than what is read next: two pairs and two of A
            static_assert(4 * TL::LB + 2 * TL::LA == 12, "12 loads stay in flight");
            using W = std::integral_constant<int, 12>;
            read_a(C0{}, pc);
            load_b(C1{}, s + 2, (P + 2) % 3);
            load_b(C0{}, s + 3, P);
            arrived(W{});                                                 // B1(s), B0(s+1)
            mul(C0{}, C0{}, fb0[0], csc);
            read_b(C1{}, pc, fb1);
            read_b(C0{}, std::integral_constant<int, (P + 1) % 3>{}, fb0[0]);
            load_a(C0{}, s + 3, P);
            arrived(W{});                                                 // A(s+1)
            mul(C0{}, C1{}, fb1, csc);
        }
    };
    if constexpr (TL::UA == 2) {
#pragma unroll
        for (int s = 0; s < 2; ++s) { load_b(C0{}, s, s); load_a(C0{}, s, s); load_b(C1{}, s, s); load_a(C1{}, s, s); }
        wait_vmcnt<12>();                                                 // B0(0), A0(0)
    } else {
        load_b(C0{}, 0, 0); load_a(C0{}, 0, 0);
        load_b(C1{}, 0, 0); load_b(C0{}, 1, 1); load_a(C0{}, 1, 1);
        load_b(C1{}, 1, 1); load_b(C0{}, 2, 2); load_a(C0{}, 2, 2);
        wait_vmcnt<12>();                                                 // B0(0), A(0)
    }
    meet();
    read_b(C0{}, C0{}, fb0[0]);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    meet();
    if (late) meet();

    // The sums of the runs before the present one (8 or 9 steps, see CS_RUN) and what their additions lost wait in LDS.
    float* cs_runs = reinterpret_cast<float*>(smem + TL::STAGES * (TL::A_STAGE + TL::B_STAGE)) + (wn * 16 + l16) * 8;
    auto end_run = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float x = cs[j];
            x += __shfl_xor(x, 16, 64);
            x += __shfl_xor(x, 32, 64);
            if (lq == 0) {
                float sum = cs_runs[2 * j], lost = cs_runs[2 * j + 1];
                add_carrying(sum, lost, x);
                cs_runs[2 * j] = sum;
                cs_runs[2 * j + 1] = lost;
            }
            cs[j] = 0.0f;
        }
    };
    auto run = [&](auto csc) __attribute__((always_inline)) {
        constexpr bool CS = decltype(csc)::value;
        int s = 0;
        if constexpr (CS) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                cs[j] = 0.0f;
                if (lq == 0) cs_runs[2 * j] = cs_runs[2 * j + 1] = 0.0f;
            }
        }
        if constexpr (TL::STAGES == 2) {
            for (; s + 1 < ns; s += 2) {
                step(s, C0{}, csc);
                step(s + 1, C1{}, csc);
                if (CS && s % 8 == 6) end_run();
            }
            if (s < ns) step(s, C0{}, csc);
        } else {
            for (; s + 2 < ns; s += 3) {
                step(s, C0{}, csc);
                step(s + 1, C1{}, csc);
                step(s + 2, C2{}, csc);
                if (CS && s % 9 == 6) end_run();
            }
            if (s < ns) step(s, C0{}, csc);
            if (s + 1 < ns) step(s + 1, C1{}, csc);
        }
    };
    const bool cs_on = COLSUM && p.colsum && w.tm == 0 && wm == 0;        // uniform over the wavefront; both copies have the same barriers
    if constexpr (COLSUM) {
        if (cs_on) run(std::true_type{});
        else run(std::false_type{});
    } else {
        run(std::false_type{});
    }
    if (!late) meet();
    mfma16_drain();
    wait_vmcnt<0>();
    if (COLSUM && cs_on) {
        end_run();
        if (lq == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int q = l16 >> 2, col = n0 + (j >> 1) * BC + wn * 32 + 8 * q + 4 * ((q ^ j) & 1) + (l16 & 3);
                if (col < p.N) {
                    const float v = cs_runs[2 * j] - cs_runs[2 * j + 1];
                    if (w.partial) p.colsum_part[(int64_t)w.share * p.N + col] = v;
                    else p.colsum[col] = (bf16_t)v;
                }
            }
        }
    }
}

}  // namespace tpl

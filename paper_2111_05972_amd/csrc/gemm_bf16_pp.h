// bf16 GEMM tile for gfx950 on eight wavefronts that take turns at the matrix cores: 256 x 256, K in steps of 64.
//
// What bounds it.  On random operands board power (see gemm_bf16.hip): per flop the tile moves the fewest bytes through LDS
// and L2 of the kernels here, and its matrix instruction (16x16x32) is the cheap one.  On zeros 1880 (NT), 1900 (NN) and
// 1870 TFLOP/s (TN) at 8192^3, random 1413, 1497 and 1431, where the best kernel of gemm_bf16.hip for each layout reaches
// 1337, 1360 and 1359 (fetch and math wavefronts NT, the 256 x 256 tile of four wavefronts NN and TN); at 4096^3, one tile per
// compute unit, 100 us (NT) and 103 us (TN) against 116 and 110.
//
// Turns.  Wavefronts w and w + 4 share a SIMD.  The product of a step is four clusters (a half of A's rows times a half of
// B's columns); for each a wavefront first reads what is missing of its fragments and issues two loads (memory phase), then
// runs 16 matrix instructions on them (matrix phase), with a workgroup barrier behind either phase.  Wavefronts 4..7 are one
// phase behind, so of the two on a SIMD one always has matrix instructions to issue while the other waits for LDS: no
// fragment is read ahead, and 128 accumulators, 80 fragment registers and the addresses fit 256.
//
// LDS.  Two stages of 64 k, each in four units: the halves B0, A0, B1, A1, 128 rows (columns) of 64 k.  64 k are a whole cache
// line of a K-major row.  A unit is read in one cluster and handed back to the loads in the next, eight clusters before
// it is read again, so six to seven units (12 KiB per wavefront) are always in flight although there are only two stages.
//
// Which rows and columns a wavefront owns: rows 64 wm .. + 63 of either half of A, columns 32 wn .. + 31 of either half of B.
// The blocks of C are computed transposed, and the two blocks of such 32 columns take turns at groups of four columns, so that
// a lane ends up with 8 consecutive columns of a row: 16 bytes of bf16.  So results go from the accumulators to memory
// without passing through LDS, 64 contiguous bytes per row.
#pragma once
#include "gemm_bf16_common.h"

namespace tpl {

template <int NB0_, int NB1_>
struct PPTile {
    static constexpr int NB0 = NB0_, NB1 = NB1_, NB = NB0 + NB1;          // 16-column blocks of a wavefront in the two B units
    static constexpr int BM = 256, BN = 64 * NB;
    static constexpr int A_UNIT = 128 * 128, B0_UNIT = 64 * NB0 * 128, B1_UNIT = 64 * NB1 * 128;   // bytes: rows (columns) x 64 k
    static constexpr int A_STAGE = 2 * A_UNIT, B_STAGE = B0_UNIT + B1_UNIT;
    static constexpr int CS_BYTES = 4 * 16 * NB * 2 * 4;                  // column sums of the finished runs
    static constexpr int LDS_BYTES = 2 * (A_STAGE + B_STAGE) + CS_BYTES;
};

// Some of a GEMM's tiles: `count` from `tile0` on, K cut into shares of nk k-steps (an even number where there are several).
// partial: the sums of (share, tile) as the accumulators hold them, see pp_partial; null where K is whole.
struct PPRun { int tile0, count, nk; float* partial; };
template <typename TL> constexpr int pp_tile_floats() { return TL::BM * TL::BN; }

// acc += F_b F_a: rows of the block are columns of C
__device__ __forceinline__ void mfma16_pp(f32x4& acc, const bf16x8& b, const bf16x8& a) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}
__device__ __forceinline__ int pp_swz_pair(int row) { return ((row >> 1) & 1) | (((row >> 3) & 3) << 1); }

// A unit is R rows (columns) x 64 k of an operand; a wavefront loads R / 64 blocks of 1 KiB of it.
// K-major: the k chunk that a lane loads of block `block`.  MN-major: byte offsets only, k is the block's row.
template <bool PAIR> __device__ __forceinline__ int pp_chunk(int block, int lane) {
    const int row = block * 8 + (lane >> 3);
    return (lane & 7) ^ (PAIR ? pp_swz_pair(row) : swz_k64(row));
}
template <bool KMAJ, bool PAIR, int R>
__device__ __forceinline__ void pp_offsets(unsigned (&off)[R / 64], int ld, int mn0, int MN, int wave, int lane) {
#pragma unroll
    for (int j = 0; j < R / 64; ++j) {
        const int block = wave * (R / 64) + j;
        if (KMAJ) {
            const int row = block * 8 + (lane >> 3), c = pp_chunk<PAIR>(block, lane);
            off[j] = mn0 + row < MN ? (unsigned)(((int64_t)(mn0 + row) * ld + c * 8) * 2) : OOB_HALF;
        } else {
            const int idx = block * 64 + lane, k = idx / (R / 8), pos = idx % (R / 8);
            const int c = PAIR ? pos ^ ((k & 3) << 2) ^ ((k >> 3) & 1) : mn_unswz<R>(pos, k);
            off[j] = mn0 + c * 8 < MN ? (unsigned)(((int64_t)k * ld + mn0 + c * 8) * 2) : OOB_HALF;
        }
    }
}
// Loads step s (64 k from k00 + 64 s) of a unit.  K-major: past the end of the K share a lane reads nothing; it may lie inside
// the last step.  MN-major: a share ends with a step or with the buffer.
template <bool KMAJ, bool PAIR, int NL>
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
                                 k0 + pp_chunk<PAIR>(wave * NL + j, l) * 8 < kend && off[j] != OOB_HALF ? off[j] + so : OOB_HALF);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Fragment reads of one operand.  addr: per-lane LDS addresses (see pp_bases), IMM: the unit's byte offset.
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

// Epilogue straight from the accumulators.  The blocks of C are computed transposed (lane = row of C), and the two blocks of
// a pair hold interleaved groups of four columns, so a lane has 8 consecutive columns of one row: 16 bytes of bf16, 64
// contiguous bytes over the four lanes of a row.  Nothing passes through LDS.
template <typename TL>
struct PPLane {
    int row, col0, col1;              // first row; first column in the two B units
    bool odd;                         // pair blocks hold their column groups in swapped order in odd lane groups
    float bias[TL::NB * 4];
};
template <int KIND, int W>
__device__ __forceinline__ uint4 pp_fetch(const GemmParams& p, int row, int col) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if ((KIND == KIND_RESID || KIND == KIND_DGELU) && row < p.M && col < p.N) {
        const bf16_t* src = (KIND == KIND_RESID ? p.resid : p.aux) + (int64_t)row * p.N + col;
        if (W == 8) v = *reinterpret_cast<const uint4*>(src);
        else { const uint2 h = *reinterpret_cast<const uint2*>(src); v.x = h.x; v.y = h.y; }
    }
    return v;
}
template <int W>
__device__ __forceinline__ void pp_store(bf16_t* dst, const uint4& v, bool nt) {
    if (W == 8) {
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 o = {v.x, v.y, v.z, v.w};
        if (nt) __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(dst));
        else *reinterpret_cast<u32x4*>(dst) = o;
    } else {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 o = {v.x, v.y};
        if (nt) __builtin_nontemporal_store(o, reinterpret_cast<u32x2*>(dst));
        else *reinterpret_cast<u32x2*>(dst) = o;
    }
}
template <int KIND, int W>
__device__ __forceinline__ void pp_emit(const GemmParams& p, int row, int col, float (&v)[8], const float* bias, uint4 in) {
    if (row >= p.M || col >= p.N) return;
    const int64_t idx = (int64_t)row * p.N + col;
#pragma unroll
    for (int e = 0; e < W; ++e) v[e] += bias[e];
    if (KIND == KIND_RESID || (KIND == KIND_ANY && p.resid)) {
        float r8[8];
        if (KIND == KIND_ANY) {
            const uint2* src = reinterpret_cast<const uint2*>(p.resid + idx);
            const uint2 a = src[0], b = W == 8 ? src[1] : a;
            in = make_uint4(a.x, a.y, b.x, b.y);
        }
        unpack8(in, r8);
#pragma unroll
        for (int e = 0; e < W; ++e) v[e] += r8[e];
    }
    if (KIND == KIND_GELU || (KIND == KIND_ANY && p.epi == EPI_GELU)) {
        pp_store<W>(p.aux + idx, pack8(v), false);
#pragma unroll
        for (int e = 0; e < W; ++e) v[e] = gelu_f(v[e]);
    } else if (KIND == KIND_DGELU || (KIND == KIND_ANY && p.epi == EPI_DGELU)) {
        float u8[8];
        if (KIND == KIND_ANY) {
            const uint2* src = reinterpret_cast<const uint2*>(p.aux + idx);
            const uint2 a = src[0], b = W == 8 ? src[1] : a;
            in = make_uint4(a.x, a.y, b.x, b.y);
        }
        unpack8(in, u8);
#pragma unroll
        for (int e = 0; e < W; ++e) v[e] *= gelu_grad_f(u8[e]);
    }
    pp_store<W>(p.C + idx, pack8(v), p.nt_store);
}
// A block of 16 rows of the wavefront: x[j] holds 4 columns of block j.
template <typename TL, int KIND>
__device__ __forceinline__ void pp_row_block(const GemmParams& p, const PPLane<TL>& el, int row, const f32x4 (&x)[TL::NB], const uint4 (&in)[2]) {
    auto unit = [&](auto uc) __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value, N_ = U ? TL::NB1 : TL::NB0, J = U ? TL::NB0 : 0;
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float lo = x[J][e], hi = N_ == 2 ? x[J + N_ - 1][e] : 0.0f;
            v[e] = N_ == 2 && el.odd ? hi : lo;
            v[4 + e] = N_ == 2 && el.odd ? lo : hi;
        }
        pp_emit<KIND, 4 * N_>(p, row, U ? el.col1 : el.col0, v, el.bias + 4 * J, in[U]);
    };
    unit(std::integral_constant<int, 0>{});
    unit(std::integral_constant<int, 1>{});
}
template <typename TL, int KIND>
__device__ __forceinline__ void pp_rows(const GemmParams& p, const f32x4 (&acc)[2][4][TL::NB], const PPLane<TL>& el) {
    constexpr int NB0 = TL::NB0, NB1 = TL::NB1, NB = TL::NB, W0 = 4 * NB0, W1 = 4 * NB1;
    uint4 in[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        in[i][0] = pp_fetch<KIND, W0>(p, el.row + i * 16, el.col0);
        in[i][1] = pp_fetch<KIND, W1>(p, el.row + i * 16, el.col1);
    }
    f32x4 x[4][NB];                       // the present half: one body for both, code that runs once per tile comes from memory
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) x[i][j] = acc[0][i][j];
#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = el.row + h * 128 + i * 16;
            pp_row_block<TL, KIND>(p, el, row, x[i], in[i]);
            if (h == 0) {
                in[i][0] = pp_fetch<KIND, W0>(p, row + 128, el.col0);
                in[i][1] = pp_fetch<KIND, W1>(p, row + 128, el.col1);
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) x[i][j] = acc[1][i][j];
        }
    }
}
template <typename TL>
__device__ __forceinline__ PPLane<TL> pp_lane(const GemmParams& p, int m0, int n0) {
    constexpr int NB0 = TL::NB0, NB1 = TL::NB1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave >> 2, wn = wave & 3;
    PPLane<TL> el;
    const int g = lane >> 4;
    el.row = m0 + wm * 64 + (lane & 15);
    el.col0 = n0 + wn * 16 * NB0 + 4 * NB0 * g;
    el.col1 = n0 + 64 * NB0 + wn * 16 * NB1 + 4 * NB1 * g;
    el.odd = g & 1;
#pragma unroll
    for (int e = 0; e < 4 * NB0; ++e) el.bias[e] = p.bias && el.col0 < p.N ? (float)p.bias[el.col0 + e] : 0.0f;
#pragma unroll
    for (int e = 0; e < 4 * NB1; ++e) el.bias[4 * NB0 + e] = p.bias && el.col1 < p.N ? (float)p.bias[el.col1 + e] : 0.0f;
    return el;
}
// Partial sums of a K share: 16 bytes per lane, block by block; blocks of rows past M are left out.
template <typename TL>
__device__ __forceinline__ float4* pp_partial(float* tile, int h, int i) {
    return reinterpret_cast<float4*>(tile) + ((h * 4 + i) * TL::NB) * 512 + threadIdx.x;
}
template <typename TL, int B>
__device__ __forceinline__ void pp_store_partial(const GemmParams& p, const f32x4 (&acc)[2][4][TL::NB], int row0, float* partial) {
    if constexpr (B < 8) {
        constexpr int H = B >> 2, I = B & 3;
        if (row0 + H * 128 + I * 16 < p.M) {
            float4* dst = pp_partial<TL>(partial, H, I);
#pragma unroll
            for (int j = 0; j < TL::NB; ++j) dst[j * 512] = make_float4(acc[H][I][j][0], acc[H][I][j][1], acc[H][I][j][2], acc[H][I][j][3]);
        }
        pp_store_partial<TL, B + 1>(p, acc, row0, partial);
    }
}
template <typename TL>
__device__ __forceinline__ void pp_epilogue(const GemmParams& p, const f32x4 (&acc)[2][4][TL::NB], int m0, int n0, float* partial) {
    if (partial) {
        pp_store_partial<TL, 0>(p, acc, m0 + (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) >> 2) * 64, partial);
        return;
    }
    const PPLane<TL> el = pp_lane<TL>(p, m0, n0);
    if (p.epi == EPI_NONE && !p.resid) pp_rows<TL, KIND_PLAIN>(p, acc, el);
    else if (p.epi == EPI_NONE) pp_rows<TL, KIND_RESID>(p, acc, el);
    else if (p.epi == EPI_GELU && !p.resid) pp_rows<TL, KIND_GELU>(p, acc, el);
    else if (p.epi == EPI_DGELU && !p.resid) pp_rows<TL, KIND_DGELU>(p, acc, el);
    else pp_rows<TL, KIND_ANY>(p, acc, el);
}
// Row block `part` (0..7) of a tile whose K was cut: the shares' sums in share order, then the epilogue.
template <typename TL>
__device__ __forceinline__ void pp_sum_rows(const GemmParams& p, const PPRun& r, int shares, int local, int part) {
    int tm, tn;
    tile_coords(r.tile0 + local, p.tiles_m, p.tiles_n, p.band, tm, tn);
    const int m0 = tm * TL::BM, n0 = tn * TL::BN, h = part >> 2, i = part & 3;
    const PPLane<TL> el = pp_lane<TL>(p, m0, n0);
    const int row = el.row + h * 128 + i * 16;
    if (__builtin_amdgcn_readfirstlane(row - (int)(threadIdx.x & 15)) < p.M) {
        f32x4 x[TL::NB];
#pragma unroll
        for (int j = 0; j < TL::NB; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[j][v] = 0.0f;
        for (int s = 0; s < shares; ++s) {
            const float4* src = pp_partial<TL>(r.partial + ((int64_t)s * r.count + local) * pp_tile_floats<TL>(), h, i);
#pragma unroll
            for (int j = 0; j < TL::NB; ++j) {
                const float4 y = src[j * 512];
                x[j][0] += y.x; x[j][1] += y.y; x[j][2] += y.z; x[j][3] += y.w;
            }
        }
        const uint4 none[2] = {};
        pp_row_block<TL, KIND_ANY>(p, el, row, x, none);
    }
    const int col = n0 + (int)threadIdx.x;
    if (part == 0 && tm == 0 && p.colsum && threadIdx.x < TL::BN && col < p.N) {
        float v = 0.0f;
        for (int s = 0; s < shares; ++s) v += p.colsum_part[(int64_t)s * p.N + col];
        p.colsum[col] = (bf16_t)v;
    }
}

template <typename TL>
struct PPWork { int tm, m0, n0, k0, kend, share; float* partial; };
template <typename TL>
__device__ __forceinline__ PPWork<TL> pp_work(const GemmParams& p, const PPRun& r, int pos) {
    PPWork<TL> w;
    w.share = pos / r.count;
    const int local = pos - w.share * r.count;
    int tn;
    tile_coords(r.tile0 + local, p.tiles_m, p.tiles_n, p.band, w.tm, tn);
    w.m0 = w.tm * TL::BM;
    w.n0 = tn * TL::BN;
    w.k0 = w.share * r.nk * DK;
    w.kend = w.k0 + r.nk * DK < p.K ? w.k0 + r.nk * DK : p.K;
    w.partial = r.partial ? r.partial + (int64_t)pos * pp_tile_floats<TL>() : nullptr;
    return w;
}

template <typename TL, bool A_KMAJ, bool B_KMAJ, bool COLSUM>
__device__ __forceinline__ void pp_products(const GemmParams& p, const PPWork<TL>& w, char* smem, f32x4 (&acc)[2][4][TL::NB]) {
    constexpr int NB0 = TL::NB0, NB1 = TL::NB1, NB = TL::NB;
    const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wm = wave >> 2, wn = wave & 3;
    const int m0 = w.m0, n0 = w.n0, k00 = w.k0, ns = (w.kend - w.k0 + 63) / 64;

    const i32x4 ra = make_rsrc(p.A, (unsigned)((int64_t)(A_KMAJ ? p.M : p.K) * p.lda * 2));
    const i32x4 rb = make_rsrc(p.B, (unsigned)((int64_t)(B_KMAJ ? p.N : p.K) * p.ldb * 2));
    const unsigned lds_a = (unsigned)(uintptr_t)(lds_void_ptr)smem, lds_b = lds_a + 2 * TL::A_STAGE;
    unsigned oa0[2], oa1[2], ob0[NB0], ob1[NB1];
    pp_offsets<A_KMAJ, false, 128>(oa0, p.lda, m0, p.M, wave, lane);
    pp_offsets<A_KMAJ, false, 128>(oa1, p.lda, m0 + 128, p.M, wave, lane);
    pp_offsets<B_KMAJ, NB0 == 2, 64 * NB0>(ob0, p.ldb, n0, p.N, wave, lane);
    pp_offsets<B_KMAJ, NB1 == 2, 64 * NB1>(ob1, p.ldb, n0 + 64 * NB0, p.N, wave, lane);
    const unsigned ka_bytes = A_KMAJ ? 2u : (unsigned)p.lda * 2u, kb_bytes = B_KMAJ ? 2u : (unsigned)p.ldb * 2u;
    // unit u of step s: 0: B0, 1: A0, 2: B1, 3: A1
    auto issue = [&](auto uc, int s, int stage) __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value;
        if constexpr (U == 0) pp_load<B_KMAJ, NB0 == 2>(rb, lds_b + stage * TL::B_STAGE, ob0, k00 + 64 * s, w.kend, kb_bytes, wave, lane);
        else if constexpr (U == 1) pp_load<A_KMAJ, false>(ra, lds_a + stage * TL::A_STAGE, oa0, k00 + 64 * s, w.kend, ka_bytes, wave, lane);
        else if constexpr (U == 2) pp_load<B_KMAJ, NB1 == 2>(rb, lds_b + stage * TL::B_STAGE + TL::B0_UNIT, ob1, k00 + 64 * s, w.kend, kb_bytes, wave, lane);
        else pp_load<A_KMAJ, false>(ra, lds_a + stage * TL::A_STAGE + TL::A_UNIT, oa1, k00 + 64 * s, w.kend, ka_bytes, wave, lane);
    };
    using U0 = std::integral_constant<int, 0>; using U1 = std::integral_constant<int, 1>;
    using U2 = std::integral_constant<int, 2>; using U3 = std::integral_constant<int, 3>;

    // LDS addresses of this lane's fragment reads
    unsigned aaddr[4], b0addr[2 * NB0], b1addr[2 * NB1];                  // K-major: [ks] ([block][ks]); MN-major: [row block] ([block])
    if (A_KMAJ) {
        const int row = wm * 64 + l16;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) aaddr[ks] = lds_a + row * 128 + (((lq + 4 * ks) ^ swz_k64(row)) << 4);
        aaddr[2] = aaddr[3] = 0;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 8 * lq + (l16 >> 2), mn = wm * 64 + i * 16 + 4 * (l16 & 3);
            aaddr[i] = lds_a + k * 256 + (mn_swz<128>(mn >> 3, k) << 4) + (mn & 7) * 2;
        }
    }
    auto b_bases = [&](auto nbc, unsigned base, unsigned* addr) __attribute__((always_inline)) {
        constexpr int N_ = decltype(nbc)::value;
#pragma unroll
        for (int j = 0; j < N_; ++j) {
            if (B_KMAJ) {
                const int q = l16 >> 2;
                const int row = N_ == 2 ? wn * 32 + 8 * q + 4 * ((q ^ j) & 1) + (l16 & 3) : wn * 16 + l16;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
                    addr[2 * j + ks] = base + row * 128 + (((lq + 4 * ks) ^ (N_ == 2 ? pp_swz_pair(row) : swz_k64(row))) << 4);
            } else {
                const int k = 8 * lq + (l16 >> 2), q = l16 & 3;
                if (N_ == 2) {
                    const int c = (wn * 4 + q) ^ ((k & 3) << 2) ^ ((k >> 3) & 1);
                    addr[j] = base + k * 256 + (c << 4) + 8 * ((q ^ j) & 1);
                } else {
                    const int mn = wn * 16 + 4 * q;
                    addr[j] = base + k * 128 + (mn_swz<64>(mn >> 3, k) << 4) + (mn & 7) * 2;
                }
            }
        }
    };
    b_bases(std::integral_constant<int, NB0>{}, lds_b, b0addr);
    b_bases(std::integral_constant<int, NB1>{}, lds_b + TL::B0_UNIT, b1addr);

#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[h][i][j][v] = 0.0f;
    bf16x8 fa[4][2], fb0[2][NB0][2], fb1[NB1][2];                         // [..][ks]

    auto read_a = [&](auto hc, auto pc) __attribute__((always_inline)) {
        constexpr int UNIT = decltype(pc)::value * TL::A_STAGE + decltype(hc)::value * TL::A_UNIT;
        if constexpr (A_KMAJ) {
            fa[0][0] = pp_read<true, UNIT, 0>(aaddr[0]); fa[0][1] = pp_read<true, UNIT, 0>(aaddr[1]);
            fa[1][0] = pp_read<true, UNIT + 2048, 0>(aaddr[0]); fa[1][1] = pp_read<true, UNIT + 2048, 0>(aaddr[1]);
            fa[2][0] = pp_read<true, UNIT + 4096, 0>(aaddr[0]); fa[2][1] = pp_read<true, UNIT + 4096, 0>(aaddr[1]);
            fa[3][0] = pp_read<true, UNIT + 6144, 0>(aaddr[0]); fa[3][1] = pp_read<true, UNIT + 6144, 0>(aaddr[1]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                fa[i][0] = pp_read<false, UNIT, 256>(aaddr[i]);
                fa[i][1] = pp_read<false, UNIT + 32 * 256, 256>(aaddr[i]);
            }
        }
    };
    auto read_b = [&](auto nbc, auto unitc, const unsigned* addr, auto& dst) __attribute__((always_inline)) {
        constexpr int N_ = decltype(nbc)::value, UNIT = decltype(unitc)::value, PITCH = 128 * N_;
#pragma unroll
        for (int j = 0; j < N_; ++j) {
            if constexpr (B_KMAJ) {
                dst[j][0] = pp_read<true, UNIT, 0>(addr[2 * j]);
                dst[j][1] = pp_read<true, UNIT, 0>(addr[2 * j + 1]);
            } else {
                dst[j][0] = pp_read<false, UNIT, PITCH>(addr[j]);
                dst[j][1] = pp_read<false, UNIT + 32 * PITCH, PITCH>(addr[j]);
            }
        }
    };
    auto read_b0 = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        read_b(std::integral_constant<int, NB0>{}, std::integral_constant<int, P * TL::B_STAGE>{}, b0addr, fb0[P]);
    };
    auto read_b1 = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        read_b(std::integral_constant<int, NB1>{}, std::integral_constant<int, P * TL::B_STAGE>{}, b1addr, fb1);
    };
    // end of a memory phase: this cluster's fragments are in registers, the next cluster's unit has landed
    auto meet = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto arrived = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        meet();
    };
    // Column sums of B over k (bias gradients): a lane adds up what it holds of its column, see end_run
    float cs[COLSUM ? NB : 1];
    auto mul = [&](auto hc, auto jc, auto nbc, const auto& fb, auto csc) __attribute__((always_inline)) {
        constexpr int H = decltype(hc)::value, J0 = decltype(jc)::value, N_ = decltype(nbc)::value;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < N_; ++j) {
                    mfma16_pp(acc[H][i][J0 + j], fb[j][ks], fa[i][ks]);
                    __builtin_amdgcn_sched_barrier(0);
                }
        if constexpr (decltype(csc)::value && H == 0) {
#pragma unroll
            for (int j = 0; j < N_; ++j) cs[J0 + j] = add_elements(fb[j][1], add_elements(fb[j][0], cs[J0 + j]));
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        meet();
    };
    using C0 = std::integral_constant<int, 0>; using C1 = std::integral_constant<int, 1>;
    using N0 = std::integral_constant<int, NB0>; using N1 = std::integral_constant<int, NB1>;
    constexpr int W01 = 6 + 2 * NB0 + NB1, W23 = 6 + NB0 + 2 * NB1;
    auto step = [&](int s, auto pc, auto csc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        read_a(C0{}, pc);
        issue(U0{}, s + 2, P);
        wait_vmcnt<W01>();
        arrived();
        mul(C0{}, C0{}, N0{}, fb0[P], csc);
        read_b1(pc);
        issue(U1{}, s + 2, P);
        wait_vmcnt<W01>();
        arrived();
        mul(C0{}, N0{}, N1{}, fb1, csc);
        read_a(C1{}, pc);
        issue(U2{}, s + 2, P);
        wait_vmcnt<W23>();
        arrived();
        mul(C1{}, N0{}, N1{}, fb1, csc);
        read_b0(std::integral_constant<int, P ^ 1>{});
        issue(U3{}, s + 2, P);
        wait_vmcnt<W23>();
        arrived();
        mul(C1{}, C0{}, N0{}, fb0[P], csc);
    };
    issue(U0{}, 0, 0); issue(U1{}, 0, 0); issue(U2{}, 0, 0); issue(U3{}, 0, 0);
    issue(U0{}, 1, 1); issue(U1{}, 1, 1); issue(U2{}, 1, 1); issue(U3{}, 1, 1);
    wait_vmcnt<W23>();
    meet();
    read_b0(C0{});
    arrived();
    if (wm == 1) meet();
    // The sums of the runs before the present one (CS_RUN k-steps of 32 each) and what their additions lost wait in LDS.
    float* cs_runs = reinterpret_cast<float*>(smem + 2 * (TL::A_STAGE + TL::B_STAGE)) + (wn * 16 + l16) * NB * 2;
    auto end_run = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < (COLSUM ? NB : 1); ++j) {
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
            for (int j = 0; j < NB; ++j) {
                cs[j] = 0.0f;
                if (lq == 0) cs_runs[2 * j] = cs_runs[2 * j + 1] = 0.0f;
            }
        }
        for (; s + 1 < ns; s += 2) {
            step(s, C0{}, csc);
            step(s + 1, C1{}, csc);
            if (CS && s % (CS_RUN / 2) == CS_RUN / 2 - 2) end_run();
        }
        if (s < ns) step(s, C0{}, csc);
    };
    const bool cs_on = COLSUM && p.colsum && w.tm == 0 && wm == 0;        // uniform over the wavefront; both copies have the same barriers
    if constexpr (COLSUM) {
        if (cs_on) run(std::true_type{});
        else run(std::false_type{});
    } else {
        run(std::false_type{});
    }
    if (wm == 0) meet();
    mfma16_drain();
    wait_vmcnt<0>();
    if (COLSUM && cs_on) {
        end_run();
        if (lq == 0) {
#pragma unroll
            for (int j = 0; j < (COLSUM ? NB : 1); ++j) {
                const bool b1 = j >= NB0;
                const int nb = b1 ? NB1 : NB0, jj = b1 ? j - NB0 : j, q = l16 >> 2;
                const int col = n0 + (b1 ? 64 * NB0 : 0) + wn * 16 * nb + (nb == 2 ? 8 * q + 4 * ((q ^ jj) & 1) + (l16 & 3) : l16);
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

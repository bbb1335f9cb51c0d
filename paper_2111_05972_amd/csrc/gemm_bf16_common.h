// Shared by the bf16 GEMM kernels for gfx950: launch parameters, LDS layouts, direct loads and conversions.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_math.h"
#include "kernels.h"
#include "lds_dma.h"
#include "tile_order.h"

namespace tpl {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

enum EpiKind { KIND_PARTIAL, KIND_PLAIN, KIND_RESID, KIND_GELU, KIND_DGELU, KIND_ANY };

constexpr int DK = 32;                      // k per stage
constexpr unsigned OOB_OFFSET = 0xFFFFFFF0u;   // beyond any buffer this kernel accepts

struct GemmParams {
    const bf16_t* A; const bf16_t* B; bf16_t* C;
    const bf16_t* bias; const bf16_t* resid; bf16_t* aux;
    int M, N, K;
    int lda, ldb;          // row strides (elements) of A and B as stored
    int epi;
    int tiles_m, tiles_n;
    int band;              // tile rows per band of the tile order (see tile_coords)
    int nt_store;          // C stored with the non-temporal hint
    int nk;                // k-steps of one workgroup (one K share when K is split)
    int nk_total;          // k-steps of the whole K
    float* partial;        // K split over several workgroups: float partial sums [share][M][N], else null
    bf16_t* colsum;        // [N]: sum over k of B[k][n], written by the kernels that can (see gemm_bf16), else null
    float* colsum_part;    // with K split: [share][N], the same sums of one share; gemm_group_sum_kernel adds them
};

// Which K share a workgroup computes.  The workgroup list is share-major (all tiles of share 0, then all
// tiles of share 1, ...), so the tiles in flight together on an XCD walk the same k range and share panels.
struct KShare { int tile, share, kt0, nk, kend; float* partial; };
__device__ __forceinline__ KShare k_share(const GemmParams& p, int list_pos) {
    KShare s;
    const int ntiles = p.tiles_m * p.tiles_n;
    const int share = list_pos / ntiles;
    s.tile = list_pos - share * ntiles;
    s.share = share;
    s.kt0 = share * p.nk;
    s.nk = p.nk_total - s.kt0 < p.nk ? p.nk_total - s.kt0 : p.nk;
    s.kend = (s.kt0 + s.nk) * DK < p.K ? (s.kt0 + s.nk) * DK : p.K;
    s.partial = p.partial ? p.partial + (int64_t)share * p.M * p.N : nullptr;
    return s;
}

// ---- LDS layouts -------------------------------------------------------------------------------
// K-major stage tile: 64-byte rows (32 k), four 16-byte chunks, swizzled by row.
__device__ __forceinline__ int swz_k32(int row) { return (row >> 2) & 3; }
// MN-major stage tile: one row of R (m or n) bf16 per k = R/8 16-byte chunks, R*2 bytes per k.
// A transposing read touches four consecutive k at the same 64 bytes of columns (two 16-lane groups,
// 32 bytes each); the four k must land in four different 64-byte quarters of the 256-byte bank line.
//  * R*2 a multiple of 256 (R = 128, 256): every k starts at the same bank offset, so the 64-byte
//    column group is XORed with k & 3.
//  * R = 192 (384-byte rows): k and k+1 already differ by 128 bytes, so k+2, k+3 are moved one
//    64-byte group further (cyclically over the row's 6 groups; 6 = 2 mod 4 keeps the four distinct).
//  * R = 64 (128-byte rows): k and k+1 differ by 128 bytes, k+2, k+3 take the other 64-byte group of the row.
template <int R> __device__ __forceinline__ int mn_swz(int c, int k) {
    constexpr int CPR = R / 8;
    const int half = ((k >> 3) & 1) << 1;       // k and k + 8 (16x16x32 fragments read both at once): other 32 bytes
    if (CPR >= 16 && (CPR & (CPR - 1)) == 0) return c ^ ((k & 3) << 2) ^ half;
    int g = (c >> 2) + ((k >> 1) & 1);
    g = g >= CPR / 4 ? g - CPR / 4 : g;
    return (g << 2) | ((c & 3) ^ half);
}
template <int R> __device__ __forceinline__ int mn_unswz(int c, int k) {
    constexpr int CPR = R / 8;
    const int half = ((k >> 3) & 1) << 1;
    if (CPR >= 16 && (CPR & (CPR - 1)) == 0) return c ^ ((k & 3) << 2) ^ half;
    int g = (c >> 2) - ((k >> 1) & 1);
    g = g < 0 ? g + CPR / 4 : g;
    return (g << 2) | ((c & 3) ^ half);
}

constexpr unsigned OOB_HALF = 0x80000000u;     // out of bounds for operands below 2 GiB, and no wrap when a
                                               // scalar offset below 2 GiB is added

// Byte offsets (relative to the operand base, for tile origin mn0 and k = 0) of the T 16-byte chunks
// this lane fetches per stage (operand tile of R = 64 T rows); chunk j of wavefront w lands in LDS
// block w*T + j (1 KiB blocks) at 16*lane.
// XOR16: MN-major chunk positions for the kernel that reads 16x16x32 fragments with per-lane base registers
// (chunk c of row k at position c ^ xor16(k)); otherwise mn_swz.
__device__ __forceinline__ int xor16(int k) { return (((k >> 1) & 1) << 1) | (((k >> 3) & 1) << 2); }
// K16: K-major chunk positions for tiles read as 16-row fragments (swz_k32_16 below).
__device__ __forceinline__ int swz_k32_16(int row) { return (row >> 1) & 3; }
// k row (0..31) of the MN-major stage tile of R = 64 T columns that load j of wavefront `wave` fetches for this lane.
template <int T> __device__ __forceinline__ int mn_krow(int wave, int j, int lane) {
    return ((wave * T + j) * 64 + lane) / (64 * T / 8);
}
template <bool KMAJ, int T, bool XOR16 = false, bool K16 = false>
__device__ __forceinline__ void dma_offsets(unsigned (&off)[T], bool (&mn_ok)[T], int& kcol, int ld,
                                            int mn0, int MN, int wave, int lane) {
    constexpr int R = 64 * T;
#pragma unroll
    for (int j = 0; j < T; ++j) {
        int block = wave * T + j;
        if (KMAJ) {
            int row = block * 16 + (lane >> 2);
            int c = (lane & 3) ^ (K16 ? swz_k32_16(row) : swz_k32(row));
            kcol = c * 8;                                   // same for every j
            mn_ok[j] = true;                                // rows beyond MN point past the buffer
            off[j] = mn0 + row < MN ? (unsigned)(((int64_t)(mn0 + row) * ld + c * 8) * 2) : OOB_HALF;
        } else {
            int idx = block * 64 + lane;                    // physical chunk index inside the stage tile
            int k = idx / (R / 8);
            int c = XOR16 ? (idx % (R / 8)) ^ xor16(k) : mn_unswz<R>(idx % (R / 8), k);   // logical chunk stored there
            kcol = 0;
            mn_ok[j] = mn0 + c * 8 < MN;
            off[j] = (unsigned)(((int64_t)k * ld + mn0 + c * 8) * 2);
        }
    }
}

// LDS -> MFMA fragment: rows mn_base + (lane % 32), k = ks*16 + 8*(lane/32) + 0..7.
template <bool KMAJ, int R>
__device__ __forceinline__ bf16x8 dma_frag(const char* tile, int mn_base, int ks, int lane) {
    if (KMAJ) {
        int row = mn_base + (lane & 31);
        int c = 2 * ks + (lane >> 5);
        return *reinterpret_cast<const bf16x8*>(tile + row * 64 + ((c ^ swz_k32(row)) << 4));
    } else {
        // Two transposing reads; in each 16-lane group lane l points at (k = kb + l/4, 4 columns at
        // 4*(l%4)) and receives k = kb..kb+3 of column l.
        int l16 = lane & 15;
        int mn = mn_base + (lane & 16) + 4 * (l16 & 3);
        int kq = l16 >> 2;
        int kb = ks * 16 + 8 * (lane >> 5);
        bf16x8 out;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int k = kb + 4 * h + kq;
            int off = k * (R * 2) + (mn_swz<R>(mn >> 3, k) << 4) + (mn & 7) * 2;
            s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(tile + off));
            bf16x4 b = __builtin_bit_cast(bf16x4, v);
            out[4 * h + 0] = b[0]; out[4 * h + 1] = b[1]; out[4 * h + 2] = b[2]; out[4 * h + 3] = b[3];
        }
        return out;
    }
}

// LDS -> fragment of the 16x16x32 matrix instruction: rows mn_base + (lane % 16), k = 8*(lane/16) + 0..7 of
// the 32-k stage.  For this lane pattern a K-major tile of 64-byte rows is free of bank conflicts with the chunk
// XOR (row >> 1) & 3 (measured: 223 B/clk/CU, against 125 with the (row >> 2) & 3 of the 32-row fragments).
template <bool KMAJ, int R>
__device__ __forceinline__ bf16x8 dma_frag16(const char* tile, int mn_base, int lane) {
    if (KMAJ) {
        int row = mn_base + (lane & 15);
        int c = lane >> 4;
        return *reinterpret_cast<const bf16x8*>(tile + row * 64 + ((c ^ swz_k32_16(row)) << 4));
    } else {
        int l16 = lane & 15;
        int mn = mn_base + 4 * (l16 & 3);
        int kq = l16 >> 2;
        int kb = 8 * (lane >> 4);
        bf16x8 out;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int k = kb + 4 * h + kq;
            int off = k * (R * 2) + (mn_swz<R>(mn >> 3, k) << 4) + (mn & 7) * 2;
            s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(tile + off));
            bf16x4 b = __builtin_bit_cast(bf16x4, v);
            out[4 * h + 0] = b[0]; out[4 * h + 1] = b[1]; out[4 * h + 2] = b[2]; out[4 * h + 3] = b[3];
        }
        return out;
    }
}

template <int N> __device__ __forceinline__ void wait_vmcnt() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

__device__ __forceinline__ void unpack8(const uint4& v, float (&f)[8]) {
    const unsigned u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(u[i] << 16);
        f[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
    unsigned u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bf16_t lo = (bf16_t)f[2 * i], hi = (bf16_t)f[2 * i + 1];
        u[i] = (unsigned)__builtin_bit_cast(unsigned short, lo) |
               ((unsigned)__builtin_bit_cast(unsigned short, hi) << 16);
    }
    return make_uint4(u[0], u[1], u[2], u[3]);
}

// K-major tile with rows of 128 bytes (64 k): 16-byte chunk c of row r sits at position c ^ ((r >> 1) & 7),
// so the 16 rows a quarter-wavefront reads at one k are spread over all banks.
__device__ __forceinline__ int swz_k64(int row) { return (row >> 1) & 7; }

// Wait states between the last matrix instruction and a read of its accumulator.
__device__ __forceinline__ void mfma16_drain() { asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory"); }

// Column sums are added in runs of CS_RUN k-steps (512 rows), then the runs: as one running sum over all rows they lose more
// to rounding than the column-sum kernels (rms error over 32768 rows of unit variance that cancel: 1.8e-5 to 2.0e-5, those
// kernels 1.3e-5, so 0.35e-5; BERT-large TP 4 step 165.2 -> 166.1 us).
constexpr int CS_RUN = 16;
// s += x; what the rounding loses goes into the next call.
__device__ __forceinline__ void add_carrying(float& s, float& lost, float x) {
    const float y = x - lost, t = s + y, l = (t - s) - y;
    lost = l == l ? l : 0.0f;                  // infinite sums: inf - inf
    s = t;
}
// c + the sum of the eight elements of a fragment (float accumulation)
__device__ __forceinline__ float add_elements(const bf16x8& f, float c) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    bf16x2 ones;
    ones[0] = ones[1] = (bf16_t)1.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        bf16x2 v;
        v[0] = f[2 * e]; v[1] = f[2 * e + 1];
        c = __builtin_amdgcn_fdot2_f32_bf16(v, ones, c, false);
    }
    return c;
}
__device__ __forceinline__ void store_colsum(const GemmParams& p, const KShare& sh, int col, float v) {
    if (col >= p.N) return;
    if (sh.partial) p.colsum_part[(int64_t)sh.share * p.N + col] = v;
    else p.colsum[col] = (bf16_t)v;
}

}  // namespace tpl

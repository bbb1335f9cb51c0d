// bf16 flash-style softmax attention for gfx950, forward and backward, head sizes that are a multiple of 8 up to 128.
//
// DH is the head size rounded up to 32, 64, 96 or 128: tiles, fragments and accumulators are DH wide, columns past the
// head size dh read as zero (they must not be the next head's) and are not stored.  (8 heads x 3 x 1001 tokens x 80: the
// training step around it took 3.52 ms with one wavefront per row on vector arithmetic, 0.51 ms on the 96-wide kernels.)
//
// Precision of the weights.  At head sizes 64 and 128 probabilities and dS are rounded to bf16 before the products with V,
// dO, K and Q.  At every other head size (FLOATW) they keep their 24 bits: an operand is the sum of three bf16 terms
// (split_terms), each multiplied by a matrix instruction of its own (that step: 0.48 ms with rounded weights, 0.51 so).
//
// Infinities and NaN.  Zero times infinity is NaN, and a matrix instruction multiplies masked weights, which are zero, with
// their rows: in the tile that the diagonal crosses, a token would reach tokens before it.  So does a term of a split weight
// that happens to be zero: an infinite sum would become NaN.  With FLOATW a wavefront that ends with a value that is not finite therefore computes its 32 rows again, row by row, where a masked row
// is not read (attn_rows.h).  Head sizes 64 and 128 have the matrix instruction's behaviour.
//
// qkv is [B*S, 3*nl*dh] with columns (q | k | v, local head, dh); o is [B*S, nl*dh].  The S x S
// score matrix is never stored: scores are recomputed tile by tile on the matrix cores (MFMA
// 32x32x16 bf16, float accumulation), softmax statistics stay in registers, and only
// LSE = max + log(sum) per row is kept for the backward pass.
//
// Register layouts.  An MFMA 32x32 accumulator gives lane l column (l % 32) and rows
// 8*i + 4*(l/32) + j (register 4*i + j).  The forward and the dQ kernel compute the TRANSPOSED score
// tile (rows = keys, columns = queries), so one lane owns one query: row max / row sum are in-lane
// reductions plus one exchange with lane l^32, and the probabilities are already laid out as the
// K-operand of the next MFMA (P never passes through LDS).  The dK/dV kernel computes the
// untransposed tile (lane = key) for the same reason, and hands P to the wavefront of dK in float.  Operands that are needed with the other
// dimension contiguous (V in forward, Q and dO in dK/dV, K in dQ) are read from LDS with the
// transposing ds_read_b64_tr_b16.
//
// Backward is one launch whose workgroups are dK/dV workgroups (per key block) or dQ workgroups (per query block), each
// accumulating in registers in a fixed order: no atomics, results are run-to-run identical.  D = rowsum(dO * O) comes from a
// kernel before it, or where strips are short from the workgroups themselves (own_dsum).
//
// Streaming.  K/V (or Q/dO) tiles of 64 rows go from global memory straight into a ring of two or three LDS stages (buffer
// loads with the LDS flag), the tile of step t+1 requested at the start of step t; fragments are read from LDS a
// phase ahead of the MFMAs that use them.  A tile step is bound by vector arithmetic (exp2, scaling, conversions),
// not by the matrix cores.
//
// Strips and chunks.  The tile steps of one (128-row block, head) form a strip; under the causal mask
// strips are triangular (2 to S/64 steps) and the longest one is the critical path of the launch.  When
// the caller supplies a workspace, strips longer than a chunk length are cut into chunks of equal length,
// each chunk is a workgroup of its own that writes float partials (forward: running max, sum and
// unnormalised O; backward: partial dQ or dK, dV), and a second kernel combines the chunks of a strip in
// chunk order.  Strips of one chunk write their result directly, as without a workspace.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "attn_rows.h"
#include "device_math.h"
#include "kernels.h"
#include "lds_dma.h"

namespace tpl {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

constexpr int AW = 4;              // wavefronts per workgroup
constexpr int ATHREADS = 64 * AW;
constexpr int BLK = 32 * AW;       // rows (queries or keys) owned by a workgroup
constexpr int TILE = 64;           // rows of the streamed operand staged in LDS per step
constexpr float LOG2E = 1.44269504088896340736f;
constexpr float LN2 = 0.69314718055994530942f;
constexpr float RESCALE_LAG = 8.0f;  // forward: how far (log2) the row maximum may run ahead of the reference point

// ---- LDS tile of TILE rows x DH bf16, 16-byte chunks XOR-swizzled by row -------------------------
// Two kinds of read hit these tiles: 16-byte reads of 16 consecutive rows at one chunk (operand with
// the head dimension as K), and transposing 8-byte reads of 4 consecutive rows at two neighbouring
// 32-byte column groups.  The XOR below makes both conflict-free over the 64 banks (256 bytes): the
// bits that separate the 4 rows of a transposing read move the 64-byte column group, the remaining
// row bits move the chunk inside it.
template <int DH> __device__ __forceinline__ int swz(int row) {
    return DH == 64    ? ((((row >> 1) & 1) << 2) | ((row >> 2) & 3))     // 128-byte rows, 8 chunks
           : DH == 128 ? (((row & 3) << 2) | ((row >> 2) & 3))            // 256-byte rows, 16 chunks
                       : ((row >> 2) & 3);    // 64- and 192-byte rows: 4 rows already start in 4 different column groups
}
template <int DH> constexpr int tile_bytes() { return TILE * DH * 2; }
template <int DH, int NT> constexpr int NCHUNKS = (TILE * DH / 8 + NT - 1) / NT;   // 16-byte chunks per thread and tile (at most)

// ---- global -> LDS without passing through registers ---------------------------------------------
// A tile is TILE rows x DH bf16 = TILE*DH/8 chunks of 16 bytes; a buffer load with the LDS flag writes the 64
// chunks of a wavefront to 64 consecutive LDS positions.  Position p = t + NT*i (row p / NC, slot p % NC) must
// hold chunk (slot ^ swz(row)) of its row, so the swizzle is applied to the global offset each lane requests.
// Offsets are relative to row 0 of this (batch, head); the descriptor ends after the head's slice of row S-1,
// which makes rows >= S read as zero.
constexpr unsigned HEAD_OOB = 0x80000000u;      // past every slice (below 2 GiB), also with a row offset added
template <int DH, int NT>
__device__ __forceinline__ void dma_offsets(unsigned (&off)[(NCHUNKS<DH, NT>)], int64_t ld, int dh, int t) {
    constexpr int NC = DH / 8;
#pragma unroll
    for (int i = 0; i < NCHUNKS<DH, NT>; ++i) {
        const int p = t + NT * i, row = p / NC, c = (p % NC) ^ swz<DH>(row);
        off[i] = c * 8 < dh ? (unsigned)row * (unsigned)(ld * 2) + (unsigned)c * 16u : HEAD_OOB;
    }
}
__device__ __forceinline__ i32x4 head_rsrc(const bf16_t* base, int64_t ld, int S, int dh) {
    return make_rsrc(base, (unsigned)(((int64_t)(S - 1) * ld + dh) * 2));
}
// rows [row0, row0 + TILE) -> LDS tile at byte address lds_tile; wave = wavefront index (uniform)
template <int DH, int NT>
__device__ __forceinline__ void tile_dma(i32x4 rsrc, unsigned lds_tile, const unsigned (&off)[(NCHUNKS<DH, NT>)],
                                         unsigned row0_bytes, int wave) {
#pragma unroll
    for (int i = 0; i < NCHUNKS<DH, NT>; ++i)
        if ((i + 1) * NT <= TILE * DH / 8 || i * NT + wave * 64 < TILE * DH / 8)   // the last round may need some wavefronts only
            buffer_load_lds_b128(rsrc, lds_tile + (unsigned)(i * NT + wave * 64) * 16u, off[i] + row0_bytes);
}
// A use of v that the compiler must order after the load that produces v: placed before a streaming loop, it
// makes the compiler wait for prologue loads there, instead of inside the loop at their first use, where the
// wait (a count of all loads in flight) would also drain the tile requested for the next step.
template <typename T> __device__ __forceinline__ void settle(const T& v) { asm volatile("" ::"v"(v)); }
// The loads above are invisible to the compiler's own wait counting: wait for all of them before the barrier
// that hands the tile to the readers.
__device__ __forceinline__ void dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Two kinds of read, as byte offsets inside a tile that stay in registers across the streaming loop (computed per read they are
// ~100 vector instructions per tile step, more than the softmax arithmetic itself; matrix and vector instructions do not overlap
// on a SIMD, so every one of them is matrix time lost; backward over 8192 tokens, 12 heads of 128, causal: 771 and 761 us with
// dQ's computed per read and kept).  Both are unchanged by adding a multiple of 16 to the row (the swizzle uses row bits 0..3
// only): a second block of 16 rows is the same offset plus 16 rows.
//   frag_k_off   MFMA operand with the head dimension as K: row (row_base + lane%32), dh = 16*ks + 8*(lane/32) + 0..7
//   frag_t_off   MFMA operand with the tile's ROW index as K: column (d_base + lane%32); element e = 4h + j holds row
//                r_base + 8h + 4*(lane/32) + j, which is the order accumulator registers 0..7 hold their rows
template <int DH> __device__ __forceinline__ unsigned frag_k_off(int row_base, int ks, int lane) {
    int row = row_base + (lane & 31);
    int c = 2 * ks + (lane >> 5);
    return (unsigned)(row * (DH * 2) + ((c ^ swz<DH>(row)) << 4));
}
template <int DH> __device__ __forceinline__ unsigned frag_t_off(int d_base, int r_base, int h, int lane) {
    int l16 = lane & 15;
    int d = d_base + (lane & 16) + 4 * (l16 & 3);
    int row = r_base + 8 * h + 4 * (lane >> 5) + (l16 >> 2);
    return (unsigned)(row * (DH * 2) + ((((d >> 3) ^ swz<DH>(row))) << 4) + (d & 7) * 2);
}
typedef __attribute__((address_space(3))) const bf16x8* lds_bf16x8_cptr;
// The reads themselves from a 32-bit LDS address held in a register plus a compile-time byte offset (an immediate).
template <int IMM> __device__ __forceinline__ bf16x8 lds_frag_k(unsigned addr) {
    return *reinterpret_cast<lds_bf16x8_cptr>((uintptr_t)(addr + IMM));
}
template <int IMM> __device__ __forceinline__ bf16x8 lds_frag_t(unsigned addr0, unsigned addr1) {
    s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(addr0 + IMM));
    s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(addr1 + IMM));
    bf16x4 b0 = __builtin_bit_cast(bf16x4, v0), b1 = __builtin_bit_cast(bf16x4, v1);
    bf16x8 out;
    out[0] = b0[0]; out[1] = b0[1]; out[2] = b0[2]; out[3] = b0[3];
    out[4] = b1[0]; out[5] = b1[1]; out[6] = b1[2]; out[7] = b1[3];
    return out;
}
typedef __attribute__((ext_vector_type(4))) float f32x4;
__device__ __forceinline__ f32x4 lds_f4(unsigned addr) {
    typedef __attribute__((address_space(3))) const f32x4* p_t;
    return *reinterpret_cast<p_t>((uintptr_t)addr);
}
template <typename T> __device__ __forceinline__ void keep_in_register(T& v) { asm volatile("" : "+v"(v)); }
// The same operand straight from global memory (loop-invariant fragments kept in registers).
__device__ __forceinline__ bf16x8 frag_k_global(const bf16_t* base, int64_t ld, int row, int nrows, int dh,
                                                int ks, int lane) {
    bf16x8 z;
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = (bf16_t)0.0f;
    if (row >= nrows || 16 * ks + 8 * (lane >> 5) >= dh) return z;
    return *reinterpret_cast<const bf16x8*>(base + (int64_t)row * ld + 16 * ks + 8 * (lane >> 5));
}
// The sum of the products of two runs of eight elements (float accumulation).  Runs are added to each other in pairs: one after another the
// sums of 64 lost a tenth more to rounding than the row-dot kernel's.
__device__ __forceinline__ float dot8(const bf16x8& x, const bf16x8& y) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    float c = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        bf16x2 u, v;
        u[0] = x[e]; u[1] = x[e + 1];
        v[0] = y[e]; v[1] = y[e + 1];
        c = __builtin_amdgcn_fdot2_f32_bf16(u, v, c, false);
    }
    return c;
}
// The sum of v over each aligned group of eight lanes, in all of them.
__device__ __forceinline__ float sum_of_8_lanes(float v) {
    auto step = [](float x, auto ctrl) { return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true)); };
    v = step(v, std::integral_constant<int, 0xB1>{});      // lane ^ 1
    v = step(v, std::integral_constant<int, 0x4E>{});      // lane ^ 2
    return step(v, std::integral_constant<int, 0x141>{});  // 7 - lane: the other four
}
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)
__device__ __forceinline__ bf16x8 pack_regs(const f32x16& a, int first) {
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16_t)a[first + e];
    return o;
}
// The weights of a second product (probabilities or dS, accumulator order) as matrix operands: terms g[0] + g[1] + ...
// of rows 0..15 (g[.][0]) and 16..31 (g[.][1]).  FLOATW: a float's 24 significant bits are cut into three runs of 8, which
// are bf16 exactly, so the products and their float sums are those of float weights (results that differ from the
// correctly rounded bf16 one at head size 80: 0.05 % of dV, as with float arithmetic; 42 % with rounded weights).  The
// upper halves are taken by truncation: one lane permute per pair, and an infinity stays one.
template <bool FLOATW> constexpr int weight_terms() { return FLOATW ? 3 : 1; }
template <bool FLOATW>
__device__ __forceinline__ void split_terms(f32x16 w, bf16x8 (&g)[weight_terms<FLOATW>()][2]) {
    if constexpr (!FLOATW) {
        g[0][0] = pack_regs(w, 0);
        g[0][1] = pack_regs(w, 8);
    } else {
#pragma unroll
        for (int n = 0; n < 3; ++n)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                unsigned u[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    u[e] = __builtin_amdgcn_perm(__float_as_uint(w[8 * h + 2 * e + 1]), __float_as_uint(w[8 * h + 2 * e]), 0x07060302u);
                g[n][h] = __builtin_bit_cast(bf16x8, make_uint4(u[0], u[1], u[2], u[3]));
                if (n == 2) continue;
#pragma unroll
                for (int e = 8 * h; e < 8 * h + 8; ++e) {
                    const float top = __uint_as_float(__float_as_uint(w[e]) & 0xffff0000u);
                    w[e] = top == w[e] ? 0.0f : w[e] - top;      // not inf - inf
                }
            }
    }
}
// acc += F W for the weight rows 16 h ... of F's columns
template <bool FLOATW>
__device__ __forceinline__ f32x16 mfma_terms(const bf16x8& f, const bf16x8 (&g)[weight_terms<FLOATW>()][2], int h, f32x16 acc) {
#pragma unroll
    for (int n = 0; n < weight_terms<FLOATW>(); ++n) acc = MFMA(f, g[n][h], acc);
    return acc;
}
__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.0f;
    return z;
}
__device__ __forceinline__ void store4(bf16_t* p, float a, float b, float c, float d) {
    bf16x4 o;
    o[0] = (bf16_t)a; o[1] = (bf16_t)b; o[2] = (bf16_t)c; o[3] = (bf16_t)d;
    *reinterpret_cast<bf16x4*>(p) = o;
}
// max(v[l], v[l ^ 32]) in every lane by one lane-swap instruction (no trip through the LDS crossbar, whose latency would
// sit in the middle of the softmax chain): swapping the upper half of a with the lower half of b, for a = b = v, leaves
// (v.lo, v.lo) and (v.hi, v.hi).
__device__ __forceinline__ float cross_half_max(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// z stays 0 while the values are finite, and becomes NaN otherwise.
__device__ __forceinline__ void note4(float& z, const float (&r)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) z = fmaf(r[j], 0.0f, z);
}
__device__ __forceinline__ bool any_nonfinite(float z) { return __any(z != 0.0f); }
// 2^x on the hardware transcendental unit (arguments here are <= ~0; results below 2^-126 flush to 0).
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Log-sum-exp of a row from its reference point (log2) and sum.
template <bool FLOATW> __device__ __forceinline__ float strip_lse(float m, float l) {
    return FLOATW ? fmaf(m, LN2, logf(l)) : (m + log2f(l)) * LN2;
}

// ---- strips and chunks (host and device agree through these) --------------------------------------
// Blocks are ranked heaviest first: query blocks from the last one down (forward, dQ), key blocks from the
// first one up (dK/dV).  Workgroup `slot` of a head is chunk c of the block of rank r, slots numbered
// rank-major, so that the heaviest chunks are dispatched first.
__host__ __device__ inline int strip_block(bool kv_side, int nblk, int rank) { return kv_side ? rank : nblk - 1 - rank; }
__host__ __device__ inline int strip_tiles(bool causal, bool kv_side, int S, int blk) {
    const int nt = (S + TILE - 1) / TILE;
    if (!causal) return nt;
    if (kv_side) return nt - (blk * BLK) / TILE;          // query tiles from the diagonal to the end
    const int end = (blk + 1) * BLK < S ? (blk + 1) * BLK : S;
    return (end + TILE - 1) / TILE;                       // key tiles from 0 to the diagonal
}
// Chunk length with the multiplier that replaces the division by it (the slot search runs in every workgroup):
// magic = floor(2^32 / ch) + 1 gives floor(n / ch) = (n * magic) >> 32 exactly for n * ch < 2^32 (here n, ch < 2^16).
struct ChunkLen { int ch; unsigned magic; };
inline ChunkLen make_chunk_len(int ch) {
    return ChunkLen{ch, ch > 1 && ch < (1 << 16) ? (unsigned)((1ull << 32) / (unsigned)ch) + 1u : 0u};
}
__host__ __device__ inline int strip_chunks(int tiles, ChunkLen ch) {
    if (tiles <= ch.ch) return 1;
    if (ch.ch == 1) return tiles;
    return (int)(((unsigned long long)(unsigned)(tiles + ch.ch - 1) * ch.magic) >> 32);
}
__host__ __device__ inline int strip_slots(bool causal, bool kv_side, int S, ChunkLen ch) {
    const int nblk = (S + BLK - 1) / BLK;
    int n = 0;
    for (int r = 0; r < nblk; ++r) n += strip_chunks(strip_tiles(causal, kv_side, S, strip_block(kv_side, nblk, r)), ch);
    return n;
}
struct Chunk {
    int blk;        // query block (forward, dQ) or key block (dK/dV)
    int nch;        // chunks of this block's strip
    int slot0;      // slot of the strip's chunk 0
    int t0, t1;     // tile steps [t0, t1) of this chunk
};
// Chunk of workgroup `slot`; with slot < 0: the strip of block `want_blk` (t0, t1 = whole strip).
__device__ inline Chunk find_chunk(bool causal, bool kv_side, int S, ChunkLen ch, int slot, int want_blk) {
    const int nblk = (S + BLK - 1) / BLK;
    const int nt = (S + TILE - 1) / TILE;
    Chunk k{0, 1, 0, 0, 0};
    int acc = 0;
    for (int r = 0; r < nblk; ++r) {
        const int blk = strip_block(kv_side, nblk, r);
        const int tiles = strip_tiles(causal, kv_side, S, blk);
        const int nch = strip_chunks(tiles, ch);
        const bool hit = slot >= 0 ? slot < acc + nch : blk == want_blk;
        if (hit) {
            const int first = kv_side ? nt - tiles : 0;
            k.blk = blk; k.nch = nch; k.slot0 = acc;
            if (slot >= 0) {
                const int c = slot - acc, len = (tiles + nch - 1) / nch;
                k.t0 = first + c * len;
                k.t1 = first + ((c + 1) * len < tiles ? (c + 1) * len : tiles);
            } else {
                k.t0 = first; k.t1 = first + tiles;
            }
            return k;
        }
        acc += nch;
    }
    return k;
}
__device__ __forceinline__ void store_f4(float* p, float a, float b, float c, float d) {
    *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}

// =================================================================================================
// Forward.  Workgroup = (query block of 128, batch*head), 8 wavefronts: wavefront w owns the 32
// queries of sub-block w % 4 and, of every 64-key tile streamed through double-buffered LDS, the key
// half w / 4.  The two wavefronts of a query sub-block therefore walk half the keys each (half the
// dependent chain, two wavefronts per SIMD to overlap softmax arithmetic with matrix-core work) and
// their (max, sum, O) partials are merged through LDS at the end, always in the same order.
// =================================================================================================
constexpr int FTHREADS = 512;

template <int DH> constexpr int fwd_lds_bytes() {
    constexpr int ring = 4 * tile_bytes<DH>();
    constexpr int merge = 4 * 64 * (2 + DH / 2) * 4;      // per query sub-block and lane: m, l, O[DH/2]
    return ring > merge ? ring : merge;
}

template <int DH, bool CAUSAL, bool FLOATW>
__global__ __launch_bounds__(FTHREADS, DH <= 64 ? 4 : 2) void attn_fwd_kernel(const bf16_t* __restrict__ qkv,
                                                            bf16_t* __restrict__ o,
                                                            float* __restrict__ lse, int S, int nl, int dh, float c2f, int BH,
                                                            float* __restrict__ part, ChunkLen ch) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int TB = tile_bytes<DH>();
    constexpr int NCH = NCHUNKS<DH, FTHREADS>;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, half = lane >> 5;
    const int qs = wave & 3, kvh = wave >> 2;
    const int bh = blockIdx.x % BH, slot = blockIdx.x / BH;      // head fastest: heaviest chunks of all heads first
    const Chunk ck = find_chunk(CAUSAL, false, S, ch, slot, 0);
    const int qb = ck.blk;
    const int b = bh / nl, h = bh % nl;
    const int64_t ld = 3LL * nl * dh;
    const bf16_t* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * dh;
    const bf16_t* kbase = qbase + (int64_t)nl * dh;
    const bf16_t* vbase = kbase + (int64_t)nl * dh;
    const int q0 = qb * BLK + qs * 32;                    // first query of this wavefront
    const int q = q0 + (lane & 31);                       // this lane's query
    const float c2 = FLOATW ? c2f : LOG2E / sqrtf((float)dh);

    bf16x8 qf[DH / 16];
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) qf[ks] = frag_k_global(qbase, ld, q, S, dh, ks, lane);

    f32x16 oacc[DH / 32];
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) oacc[dt] = zero16();
    float m = -INFINITY, lsum = 0.0f;

    const int kv_end = CAUSAL ? min(S, (qb + 1) * BLK) : S;
    const int tile0 = ck.t0, ntiles = ck.t1;
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const i32x4 desc_k = head_rsrc(kbase, ld, S, dh), desc_v = head_rsrc(vbase, ld, S, dh);
    unsigned off[NCH];
    dma_offsets<DH, FTHREADS>(off, ld, dh, t);
    auto fetch_tile = [&](int kt, unsigned stage) {       // K and V rows of tile kt -> LDS stage
        const unsigned r0 = (unsigned)kt * TILE * (unsigned)(ld * 2);
        tile_dma<DH, FTHREADS>(desc_k, stage, off, r0, wave_u);
        tile_dma<DH, FTHREADS>(desc_v, stage + TB, off, r0, wave_u);
    };
    // LDS addresses of this lane's fragment reads in stage 0 (K tile at lds0, V tile one tile further), kept in registers
    unsigned ka[DH / 16], va[DH / 32][2];
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) { ka[ks] = lds0 + frag_k_off<DH>(kvh * 32, ks, lane); keep_in_register(ka[ks]); }
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int h = 0; h < 2; ++h) { va[dt][h] = lds0 + TB + frag_t_off<DH>(dt * 32, kvh * 32, h, lane); keep_in_register(va[dt][h]); }
    fetch_tile(tile0, lds0);
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) settle(qf[ks]);
    dma_wait();
    __syncthreads();
    // one tile step on ring stage STG (a compile-time constant, so that the stage is an immediate of every fragment read)
    auto step = [&](int kt, auto stg) __attribute__((always_inline)) {
        constexpr int STG = decltype(stg)::value;
        constexpr int SOFF = STG * 2 * TB;
        // the other stage was last read before the barrier that ended the previous step
        if (kt + 1 < ntiles) fetch_tile(kt + 1, lds0 + (1 - STG) * 2 * TB);
        const int kv0 = kt * TILE + kvh * 32;
        if (kv0 < kv_end && !(CAUSAL && kv0 > q0 + 31)) {                 // wavefront-uniform
            // All K fragments are requested before the first MFMA and all V fragments before the softmax arithmetic,
            // so that LDS latency is paid once per phase instead of once per MFMA (the fences keep that order).
            f32x16 s = zero16();
            bf16x8 fr[DH / 16];
#pragma unroll
            for (int ks = 0; ks < DH / 16; ++ks) fr[ks] = lds_frag_k<SOFF>(ka[ks]);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int ks = 0; ks < DH / 16; ++ks) s = MFMA(fr[ks], qf[ks], s);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int dt = 0; dt < DH / 32; ++dt) {
                fr[2 * dt] = lds_frag_t<SOFF>(va[dt][0], va[dt][1]);
                fr[2 * dt + 1] = lds_frag_t<SOFF + 16 * DH * 2>(va[dt][0], va[dt][1]);
            }
            __builtin_amdgcn_sched_barrier(0);
            // masking is needed only in tiles that straddle the diagonal or the end of the sequence
            if (kv0 + 31 >= S || (CAUSAL && kv0 + 31 > q0)) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    int kv = kv0 + (v >> 2) * 8 + half * 4 + (v & 3);
                    bool ok = kv < S && (!CAUSAL || kv <= q);
                    s[v] = ok ? s[v] : -INFINITY;
                }
            }
            float mb = s[0];
#pragma unroll
            for (int v = 1; v < 16; ++v) mb = fmaxf(mb, s[v]);
            mb = cross_half_max(mb) * c2;                     // c2 > 0: scaling commutes with max
            // The reference point m of the running sums moves only when the maximum has grown by more than
            // RESCALE_LAG (log2 units): probabilities then reach 2^RESCALE_LAG at most, which float sums and
            // bf16 operands hold without loss, and the accumulators are rescaled in a few early tiles only
            // instead of in most of them.  Any reference point gives the same O and LSE up to rounding.
            const float mn = (mb - m > RESCALE_LAG) ? mb : m;   // false for NaN (-inf - -inf): m stays
            float mu = mn == -INFINITY ? 0.0f : mn;
            float alpha = fast_exp2(m - mu);
            m = mn;
            float ps = 0.0f;
#pragma unroll
            for (int v = 0; v < 16; ++v) { s[v] = fast_exp2(fmaf(s[v], c2, -mu)); ps += s[v]; }
            lsum = lsum * alpha + ps;
            if (__any(alpha != 1.0f)) {                       // the running maximum rarely moves
#pragma unroll
                for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
            }
            bf16x8 pb[weight_terms<FLOATW>()][2];
            split_terms<FLOATW>(s, pb);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int dt = 0; dt < DH / 32; ++dt) {
                oacc[dt] = mfma_terms<FLOATW>(fr[2 * dt], pb, 0, oacc[dt]);
                oacc[dt] = mfma_terms<FLOATW>(fr[2 * dt + 1], pb, 1, oacc[dt]);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        dma_wait();
        __syncthreads();
    };
    {
        int kt = tile0;
        for (; kt + 1 < ntiles; kt += 2) {
            step(kt, std::integral_constant<int, 0>{});
            step(kt + 1, std::integral_constant<int, 1>{});
        }
        if (kt < ntiles) step(kt, std::integral_constant<int, 0>{});
    }
    lsum += __shfl_xor(lsum, 32, 64);
    // merge the two key halves: wavefronts 4..7 hand (m, l, O) to wavefronts 0..3 through LDS
    constexpr int NV = 2 + DH / 2;
    float* mg = reinterpret_cast<float*>(smem) + (qs * NV) * 64 + lane;   // element i at mg[i * 64]
    if (kvh == 1) {
        mg[0] = m; mg[64] = lsum;
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) mg[(2 + dt * 16 + v) * 64] = oacc[dt][v];
    }
    __syncthreads();
    if (kvh == 0) {
        const float m1 = mg[0], l1 = mg[64];
        const float mn = fmaxf(m, m1);
        const float mu = mn == -INFINITY ? 0.0f : mn;
        const float f0 = fast_exp2(m - mu), f1 = fast_exp2(m1 - mu);
        const float ltot = lsum * f0 + l1 * f1;
        const float inv = FLOATW || ltot > 0.0f ? 1.0f / ltot : 0.0f;
        float z = 0.0f;
        if (ck.nch > 1) {
            // one chunk of a longer strip: (max, sum, unnormalised O) of this chunk's keys, float, [query][dh]
            float* pp = part + ((int64_t)slot * BH + bh) * (BLK * (DH + 2));
            const int ql = qs * 32 + (lane & 31);
#pragma unroll
            for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float r[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        r[j] = oacc[dt][4 * i + j] * f0 + mg[(2 + dt * 16 + 4 * i + j) * 64] * f1;
                    if (FLOATW) note4(z, r);
                    store_f4(pp + ql * DH + dt * 32 + 8 * i + 4 * half, r[0], r[1], r[2], r[3]);
                }
            if (half == 0) { pp[BLK * DH + ql] = mn; pp[BLK * DH + BLK + ql] = ltot; }
        } else if (q < S) {
            bf16_t* op = o + ((int64_t)b * S + q) * ((int64_t)nl * dh) + (int64_t)h * dh;
#pragma unroll
            for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float r[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        r[j] = (oacc[dt][4 * i + j] * f0 + mg[(2 + dt * 16 + 4 * i + j) * 64] * f1) * inv;
                    if (FLOATW) note4(z, r);
                    if (dt * 32 + 8 * i + 4 * half < dh) store4(op + dt * 32 + 8 * i + 4 * half, r[0], r[1], r[2], r[3]);
                }
            if (half == 0) lse[((int64_t)b * nl + h) * S + q] = strip_lse<FLOATW>(mn, ltot);
        }
        if (!FLOATW || !any_nonfinite(z)) return;
        rows_stored();
        float* q_s = reinterpret_cast<float*>(smem) + qs * NV * 64;      // this wavefront alone reads its merge area
        float* pp = part + ((int64_t)slot * BH + bh) * (BLK * (DH + 2));
        const bool whole = ck.nch == 1;
        for (int i = q0; i < q0 + 32 && i < S; ++i) {
            load_row(q_s, qbase + (int64_t)i * ld, dh, lane);
            row_loaded();
            bf16_t* op = o + ((int64_t)b * S + i) * ((int64_t)nl * dh) + (int64_t)h * dh;
            const int ql = i - qb * BLK;
            float mr, lr;
            attn_row_fwd<(DH + 63) / 64>(q_s, kbase, vbase, ld, dh, tile0 * TILE, min(CAUSAL ? i + 1 : S, ntiles * TILE), 1.0f / sqrtf((float)dh), whole,
                                         lane, mr, lr, [&](int d, float v) { if (whole) op[d] = (bf16_t)v; else pp[ql * DH + d] = v; });
            if (lane == 0) {
                if (whole) lse[((int64_t)b * nl + h) * S + i] = mr + logf(lr);
                else { pp[BLK * DH + ql] = mr * LOG2E; pp[BLK * DH + BLK + ql] = lr; }
            }
            row_loaded();
        }
    }
}

// Threads per row of the combine kernels, four columns each: a power of two.
template <int DH> constexpr int combine_tpr() { return DH == 96 ? 32 : DH / 4; }

// Forward, second kernel: merges the chunks of every strip that was cut (max, rescale, add, in chunk order),
// normalises and writes O and LSE.  Workgroup = (256 / TPR query rows of a block, batch*head), TPR threads per row.
template <int DH, bool CAUSAL, bool FLOATW>
__global__ __launch_bounds__(256) void attn_fwd_combine_kernel(const float* __restrict__ part, bf16_t* __restrict__ o,
                                                               float* __restrict__ lse, int S, int nl, int dh, int BH, ChunkLen ch,
                                                               int blk0) {
    constexpr int TPR = combine_tpr<DH>(), PSZ = BLK * (DH + 2), RPW = 256 / TPR, WPB = BLK / RPW;
    const Chunk ck = find_chunk(CAUSAL, false, S, ch, -1, blk0 + (int)blockIdx.x / WPB);
    if (ck.nch == 1) return;
    const int bh = blockIdx.y, b = bh / nl, h = bh % nl;
    const int tc = threadIdx.x % TPR;
    {
        const int ql = ((int)blockIdx.x % WPB) * RPW + threadIdx.x / TPR;
        const int q = ck.blk * BLK + ql;
        if (q >= S || 4 * tc >= dh) return;
        const float* p0 = part + ((int64_t)ck.slot0 * BH + bh) * PSZ;
        float mtot = -INFINITY;
        for (int c = 0; c < ck.nch; ++c) mtot = fmaxf(mtot, p0[(int64_t)c * BH * PSZ + BLK * DH + ql]);
        const float mu = mtot == -INFINITY ? 0.0f : mtot;
        float ltot = 0.0f, a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
        for (int c = 0; c < ck.nch; ++c) {
            const float* pc = p0 + (int64_t)c * BH * PSZ;
            const float f = fast_exp2(pc[BLK * DH + ql] - mu);
            ltot = fmaf(pc[BLK * DH + BLK + ql], f, ltot);
            const float4 v = *reinterpret_cast<const float4*>(pc + ql * DH + 4 * tc);
            a0 = fmaf(v.x, f, a0); a1 = fmaf(v.y, f, a1); a2 = fmaf(v.z, f, a2); a3 = fmaf(v.w, f, a3);
        }
        const float inv = FLOATW || ltot > 0.0f ? 1.0f / ltot : 0.0f;
        store4(o + ((int64_t)b * S + q) * ((int64_t)nl * dh) + (int64_t)h * dh + 4 * tc, a0 * inv, a1 * inv, a2 * inv,
               a3 * inv);
        if (tc == 0) lse[((int64_t)b * nl + h) * S + q] = strip_lse<FLOATW>(mtot, ltot);
    }
}

// Backward, last kernel: dQ, dK, dV of every strip that was cut = sum of its chunks' partials in chunk order.
// blockIdx.z = 0: dQ (query-block strips), 1: dK, 2: dV (key-block strips; a slot holds [dK | dV]); workgroup =
// (256 / TPR rows of a block, batch*head), TPR threads per row.
template <int DH, bool CAUSAL>
__global__ __launch_bounds__(256) void attn_bwd_combine_kernel(const float* __restrict__ part_q,
                                                               const float* __restrict__ part_kv,
                                                               bf16_t* __restrict__ dqkv, int S, int nl, int dh, int BH,
                                                               ChunkLen ch_q, ChunkLen ch_kv,
                                                               int blk0_q, int ncut_q, int blk0_kv, int ncut_kv) {
    constexpr int TPR = combine_tpr<DH>(), RPW = 256 / TPR, WPB = BLK / RPW;
    const int which = blockIdx.z;
    if ((int)blockIdx.x / WPB >= (which == 0 ? ncut_q : ncut_kv)) return;
    const Chunk ck = find_chunk(CAUSAL, which != 0, S, which == 0 ? ch_q : ch_kv, -1,
                                (which == 0 ? blk0_q : blk0_kv) + (int)blockIdx.x / WPB);
    if (ck.nch == 1) return;
    const int bh = blockIdx.y, b = bh / nl, h = bh % nl;
    const int psz = which == 0 ? BLK * DH : 2 * BLK * DH;
    const float* p0 = (which == 0 ? part_q : part_kv) + ((int64_t)ck.slot0 * BH + bh) * psz + (which == 2 ? BLK * DH : 0);
    const float f = which == 2 ? 1.0f : 1.0f / sqrtf((float)dh);
    const int64_t ld = 3LL * nl * dh;
    const int tc = threadIdx.x % TPR;
    {
        const int rl = ((int)blockIdx.x % WPB) * RPW + threadIdx.x / TPR;
        const int row = ck.blk * BLK + rl;
        if (row >= S || 4 * tc >= dh) return;
        float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f, a3 = 0.0f;
        for (int c = 0; c < ck.nch; ++c) {
            const float4 v = *reinterpret_cast<const float4*>(p0 + (int64_t)c * BH * psz + rl * DH + 4 * tc);
            a0 += v.x; a1 += v.y; a2 += v.z; a3 += v.w;
        }
        store4(dqkv + ((int64_t)b * S + row) * ld + (int64_t)which * nl * dh + (int64_t)h * dh + 4 * tc, a0 * f, a1 * f,
               a2 * f, a3 * f);
    }
}

// =================================================================================================
// D[b,h,s] = sum_d dO[s,d] * O[s,d]: LPH lanes per (token, head), 8 elements each; reads dO and O once, coalesced.
// =================================================================================================
template <int DH>
__global__ __launch_bounds__(256) void attn_dsum_kernel(const bf16_t* __restrict__ o,
                                                        const bf16_t* __restrict__ d_o,
                                                        float* __restrict__ dsum, int B, int S, int nl, int dh) {
    constexpr int LPH = DH <= 32 ? 4 : DH == 64 ? 8 : 16;
    const int64_t item = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LPH, items = (int64_t)B * S * nl;   // token-major, then head
    const int c = (threadIdx.x % LPH) * 8;
    float acc = 0.0f;
    if (item < items && c < dh) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(o + item * dh + c);
        const bf16x8 g = *reinterpret_cast<const bf16x8*>(d_o + item * dh + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = fmaf((float)a[e], (float)g[e], acc);
    }
#pragma unroll
    for (int off = LPH / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (item < items && c == 0) {
        const int64_t row = item / nl;
        const int h = (int)(item - row * nl), b = (int)(row / S), s = (int)(row - (int64_t)b * S);
        dsum[((int64_t)b * nl + h) * S + s] = acc;
    }
}

// =================================================================================================
// dK, dV.  Workgroup = (key block of 128, batch*head), 8 wavefronts: wavefronts w and w + 4 share the 32 keys of sub-block w.
// Wavefront w works out the scores and probabilities P and accumulates dV = P^T dO; wavefront w + 4 works out dP and
// accumulates dK = dS^T Q from the same P, which it gets through LDS in float, one sub-tile of 32 queries later.  That is
// two products of a sub-tile on either, half of the accumulators and fragments each (two wavefronts per SIMD), and one's
// exponentials beside the other's products.  A SIMD's matrix work and vector work still add up for the most part.  Backward
// with the scores worked out by both and so, us: 8192 tokens, 12 heads of 128, causal 831 and 771; 2 x 2048, 10 heads 115 and
// 110; 8 x 512, 8 heads without a mask 52.4 and 50.0, heads of 64 level (4 heads 19.1 and 18.0; 2 x 1024, 16 heads 35.7 and 36.8).
// Q, dO (and LSE, D) are streamed in tiles of 64 queries through three stages: dK still reads the tile before.
// Score tile is untransposed: lane = key (l%32), registers = queries 8i + 4*(l/32) + j.
// =================================================================================================
constexpr int DKV_P_BYTES = 32 * 32 * 4;                  // P of a sub-tile and sub-block of keys
template <int DH> constexpr int dkv_lds_bytes() { return 3 * (2 * tile_bytes<DH>() + 2 * TILE * 4) + 2 * 4 * DKV_P_BYTES; }
template <int DH, bool CAUSAL, bool FLOATW, bool OWN_D, bool DK_ROLE>
__device__ __forceinline__ void attn_dkv_body(char* smem, const bf16_t* __restrict__ qkv,
                                              const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o,
                                              const float* __restrict__ lse, const float* __restrict__ dsum, bf16_t* __restrict__ dqkv,
                                              int S, int nl, int dh, float c2f, int bh, const Chunk& ck, float* __restrict__ pslot) {
    constexpr int TB = tile_bytes<DH>(), NF = DH / 16, NT = DH / 32, HALF = 32 * DH * 2;
    constexpr int NCH = NCHUNKS<DH, FTHREADS>;
    constexpr int TERMS = 6 * TB, PS = TERMS + 3 * 2 * TILE * 4;      // three Q tiles, three dO tiles, three times LSE*log2e and D, P
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, half = lane >> 5;
    const int kb = ck.blk;
    const int b = bh / nl, h = bh % nl;
    const int64_t ld = 3LL * nl * dh, ldo = (int64_t)nl * dh;
    const bf16_t* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * dh;
    const bf16_t* kbase = qbase + (int64_t)nl * dh;
    const bf16_t* vbase = kbase + (int64_t)nl * dh;
    const bf16_t* dobase = d_o + (int64_t)b * S * ldo + (int64_t)h * dh;
    const float* lrow = lse + ((int64_t)b * nl + h) * S;
    const float* drow = dsum + ((int64_t)b * nl + h) * S;
    const bf16_t* obase = OWN_D ? o + (int64_t)b * S * ldo + (int64_t)h * dh : nullptr;   // not OWN_D: D has been summed
    const int k0 = kb * BLK + (wave & 3) * 32;
    const int kv = k0 + (lane & 31);
    const float scale = 1.0f / sqrtf((float)dh);
    const float c2 = FLOATW ? c2f : LOG2E * scale;

    bf16x8 own[NF];                                        // K for the scores, V for dP
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) own[ks] = frag_k_global(DK_ROLE ? vbase : kbase, ld, kv, S, dh, ks, lane);
    f32x16 acc[NT];                                        // dK (DK_ROLE) or dV
#pragma unroll
    for (int dt = 0; dt < NT; ++dt) acc[dt] = zero16();

    const int qt0 = ck.t0, ntiles = ck.t1;                // query tiles of this chunk (the strip starts at the diagonal)
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const i32x4 desc_q = head_rsrc(qbase, ld, S, dh), desc_do = head_rsrc(dobase, ldo, S, dh);
    unsigned off_q[NCH], off_do[NCH];
    dma_offsets<DH, FTHREADS>(off_q, ld, dh, t);
    dma_offsets<DH, FTHREADS>(off_do, ldo, dh, t);
    // Q and dO rows of tile qt straight into LDS; LSE and D of its rows through registers (r2s stores them), or D from the rows of O,
    // which eight threads a row keep in registers until dO has landed.
    constexpr int OCH = (DH / 8 + 7) / 8;
    const int orow = t >> 3, oc = t & 7;
    float rl = 0.0f, rd = 0.0f;
    bf16x8 of[OCH];
    auto fetch_o = [&](int qt) __attribute__((always_inline)) {
        const int qi = qt * TILE + orow;
#pragma unroll
        for (int i = 0; i < OCH; ++i) {
            const int c = (oc + 8 * i) * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) of[i][e] = (bf16_t)0.0f;
            if (qi < S && c < dh) of[i] = *reinterpret_cast<const bf16x8*>(obase + (int64_t)qi * ldo + c);
        }
    };
    auto write_d = [&](auto stg) __attribute__((always_inline)) {
        constexpr int STG = decltype(stg)::value;
        float d = 0.0f;
#pragma unroll
        for (int i = 0; i < OCH; ++i)
            if (DH % 64 == 0 || oc + 8 * i < DH / 8)
                d += dot8(of[i], lds_frag_k<(3 + STG) * TB>(lds0 + orow * (DH * 2) + (((oc + 8 * i) ^ swz<DH>(orow)) << 4)));
        d = sum_of_8_lanes(d);
        if (oc == 0) reinterpret_cast<float*>(smem + TERMS)[STG * 2 * TILE + TILE + orow] = d;
    };
    auto g2r = [&](int qt, int stage) {
        tile_dma<DH, FTHREADS>(desc_q, lds0 + stage * TB, off_q, (unsigned)qt * TILE * (unsigned)(ld * 2), wave_u);
        tile_dma<DH, FTHREADS>(desc_do, lds0 + (3 + stage) * TB, off_do, (unsigned)qt * TILE * (unsigned)(ldo * 2), wave_u);
        if (t < TILE) {
            int qi = qt * TILE + t;
            rl = qi < S ? lrow[qi] * LOG2E : 0.0f;
            if (!OWN_D) rd = qi < S ? drow[qi] : 0.0f;
        }
    };
    auto r2s = [&](int stage) {
        if (t < TILE) {
            float* st = reinterpret_cast<float*>(smem + TERMS) + stage * 2 * TILE;
            st[t] = rl;
            if (!OWN_D) st[TILE + t] = rd;
        }
    };
    // LDS addresses in stage 0: rows as they are (scores: Q, dP: dO), transposed (dV: dO, dK: Q), LSE or D, P
    unsigned ka[NF], ta[NT][2];
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) { ka[ks] = lds0 + (DK_ROLE ? 3 * TB : 0) + frag_k_off<DH>(0, ks, lane); keep_in_register(ka[ks]); }
#pragma unroll
    for (int dt = 0; dt < NT; ++dt)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            ta[dt][g] = lds0 + (DK_ROLE ? 0 : 3 * TB) + frag_t_off<DH>(dt * 32, 0, g, lane);
            keep_in_register(ta[dt][g]);
        }
    unsigned terms = lds0 + TERMS + (DK_ROLE ? TILE * 4 : 0) + half * 16;
    char* pbuf = smem + PS + (wave_u & 3) * DKV_P_BYTES + lane * 16;
    if (qt0 < ntiles) { g2r(qt0, 0); r2s(0); if (OWN_D) fetch_o(qt0); }
    if (OWN_D) {
#pragma unroll
        for (int i = 0; i < OCH; ++i) settle(of[i]);
    }
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) settle(own[ks]);
    dma_wait();
    __syncthreads();

    f32x16 x;                                              // scores, then P; or dP, then dS
    bool pending = false;                                  // dP of the sub-tile before waits for its P
    auto product = [&](auto stg, auto sbc) __attribute__((always_inline)) {
        constexpr int OFF = decltype(stg)::value * TB + decltype(sbc)::value * HALF;
        bf16x8 fr[NF];
#pragma unroll
        for (int i = 0; i < NF; ++i) fr[i] = lds_frag_k<OFF>(ka[i]);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        x = zero16();
#pragma unroll
        for (int i = 0; i < NF; ++i) x = MFMA(fr[i], own[i], x);
        __builtin_amdgcn_s_setprio(0);
    };
    // x, P or dS, times the rows of its sub-tile, transposed
    auto fetch_t = [&](auto stg, auto sbc, bf16x8 (&fr)[NF]) __attribute__((always_inline)) {
        constexpr int OFF = decltype(stg)::value * TB + decltype(sbc)::value * HALF;
#pragma unroll
        for (int k = 0; k < NF; ++k)
            fr[k] = k & 1 ? lds_frag_t<OFF + 16 * DH * 2>(ta[k >> 1][0], ta[k >> 1][1]) : lds_frag_t<OFF>(ta[k >> 1][0], ta[k >> 1][1]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto collect = [&](const bf16x8 (&fr)[NF]) __attribute__((always_inline)) {
        bf16x8 g[weight_terms<FLOATW>()][2];
        split_terms<FLOATW>(x, g);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int k = 0; k < NF; ++k) acc[k >> 1] = mfma_terms<FLOATW>(fr[k], g, k & 1, acc[k >> 1]);
        __builtin_amdgcn_s_setprio(0);
    };
    auto finish_dk = [&](auto stg, auto sbc) __attribute__((always_inline)) {
        constexpr int STG = decltype(stg)::value, SB = decltype(sbc)::value;
        f32x4 p[4], d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = *reinterpret_cast<const f32x4*>(pbuf + SB * 4 * DKV_P_BYTES + i * 1024);
            d[i] = lds_f4(terms + STG * 2 * TILE * 4 + SB * 128 + i * 32);
        }
        bf16x8 fr[NF];
        fetch_t(stg, sbc, fr);
#pragma unroll
        for (int v = 0; v < 16; ++v) x[v] = p[v >> 2][v & 3] * (x[v] - d[v >> 2][v & 3]);
        collect(fr);
    };
    // A sub-tile of 32 queries: all of it in the dV role; dP, after the rest of the sub-tile before, in the dK role.
    auto slot = [&](int qt, auto stg, auto sbc, auto before) __attribute__((always_inline)) {
        constexpr int STG = decltype(stg)::value, SB = decltype(sbc)::value;
        const int qs0 = qt * TILE + SB * 32;
        const bool skip = qs0 >= S || (CAUSAL && qs0 + 31 < k0);         // wavefront-uniform, alike in both roles
        if constexpr (DK_ROLE) {
            if (pending) finish_dk(before, std::integral_constant<int, SB ^ 1>{});
            pending = !skip;
            if (!skip) product(stg, sbc);
        } else if (!skip) {
            product(stg, sbc);
            bf16x8 fr[NF];
            fetch_t(stg, sbc, fr);
            if (qs0 + 31 >= S || k0 + 31 >= S || (CAUSAL && k0 + 31 > qs0)) {   // wave-uniform: on the diagonal, at the end of S
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    int qi = qs0 + 8 * (v >> 2) + 4 * half + (v & 3);
                    bool ok = qi < S && kv < S && (!CAUSAL || kv <= qi);
                    x[v] = ok ? x[v] : -INFINITY;         // exp2(-inf) = 0
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4 l = lds_f4(terms + STG * 2 * TILE * 4 + SB * 128 + i * 32);
                f32x4 p;
#pragma unroll
                for (int j = 0; j < 4; ++j) p[j] = x[4 * i + j] = fast_exp2(fmaf(x[4 * i + j], c2, -l[j]));
                *reinterpret_cast<f32x4*>(pbuf + SB * 4 * DKV_P_BYTES + i * 1024) = p;
            }
            collect(fr);
        }
    };
    using C0 = std::integral_constant<int, 0>; using C1 = std::integral_constant<int, 1>; using C2 = std::integral_constant<int, 2>;
    auto step = [&](int qt, auto stg, auto next, auto before) __attribute__((always_inline)) {
        const bool more = qt + 1 < ntiles;
        if (more) g2r(qt + 1, decltype(next)::value);     // read for the last time before the barrier before last
        if (OWN_D) {
            write_d(stg);                                 // read from the next barrier on
            if (more) fetch_o(qt + 1);
        }
        slot(qt, stg, C0{}, before);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // P; the next tile stays in flight
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        slot(qt, stg, C1{}, stg);
        if (more) r2s(decltype(next)::value);
        if (OWN_D) {
#pragma unroll
            for (int i = 0; i < OCH; ++i) settle(of[i]);
        }
        dma_wait();
        __syncthreads();
    };
    for (int qt = qt0; qt < ntiles;) {
        step(qt, C0{}, C1{}, C2{});
        if (++qt >= ntiles) break;
        step(qt, C1{}, C2{}, C0{});
        if (++qt >= ntiles) break;
        step(qt, C2{}, C0{}, C1{});
        ++qt;
    }
    if (DK_ROLE && pending) {
        const int last = (ntiles - 1 - qt0) % 3;          // the stage of the last tile
        terms += last * 2 * TILE * 4;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt) { ta[dt][0] += last * TB; ta[dt][1] += last * TB; }
        finish_dk(C0{}, C1{});
    }
    if (FLOATW) __syncthreads();                          // the ring is overwritten below
    float z = 0.0f;
    if (ck.nch > 1) {
        // one chunk of a longer strip: unscaled float partial, [dK | dV][key][dh]
        float* pp = pslot + (DK_ROLE ? 0 : BLK * DH) + ((wave & 3) * 32 + (lane & 31)) * DH;
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float r[4] = {acc[dt][4 * i], acc[dt][4 * i + 1], acc[dt][4 * i + 2], acc[dt][4 * i + 3]};
                if (FLOATW) note4(z, r);
                store_f4(pp + dt * 32 + 8 * i + 4 * half, r[0], r[1], r[2], r[3]);
            }
    } else if (kv < S) {
        bf16_t* outp = dqkv + ((int64_t)b * S + kv) * ld + (int64_t)(DK_ROLE ? 1 : 2) * nl * dh + (int64_t)h * dh;
        const float f = DK_ROLE ? scale : 1.0f;
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float r[4] = {acc[dt][4 * i] * f, acc[dt][4 * i + 1] * f, acc[dt][4 * i + 2] * f, acc[dt][4 * i + 3] * f};
                if (FLOATW) note4(z, r);
                if (dt * 32 + 8 * i + 4 * half < dh) store4(outp + dt * 32 + 8 * i + 4 * half, r[0], r[1], r[2], r[3]);
            }
    }
    if (!FLOATW || !any_nonfinite(z)) return;
    rows_stored();
    float* k_s = reinterpret_cast<float*>(smem) + wave * 2 * DH;     // the ring has been read
    for (int j = k0; j < k0 + 32 && j < S; ++j) {
        load_row(k_s, kbase + (int64_t)j * ld, dh, lane);
        load_row(k_s + DH, vbase + (int64_t)j * ld, dh, lane);
        row_loaded();
        bf16_t* outp = dqkv + ((int64_t)b * S + j) * ld + (int64_t)(DK_ROLE ? 1 : 2) * nl * dh + (int64_t)h * dh;
        float* pp = pslot + (DK_ROLE ? 0 : BLK * DH) + (j - kb * BLK) * DH;
        auto d_of = [&](int i) {
            if (!OWN_D) return drow[i];
            float d[8];                                   // added in the order of write_d: the same D as in the tiles
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                d[c] = 0.0f;
#pragma unroll
                for (int q = 0; q < OCH; ++q) {
                    const int64_t at = (int64_t)i * ldo + (c + 8 * q) * 8;
                    if ((c + 8 * q) * 8 < dh) d[c] += dot8(*reinterpret_cast<const bf16x8*>(obase + at), *reinterpret_cast<const bf16x8*>(dobase + at));
                }
            }
            return ((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7]));
        };
        attn_row_dkv<(DH + 63) / 64>(k_s, k_s + DH, qbase, ld, dobase, ldo, lrow, d_of, dh, max(CAUSAL ? j : 0, qt0 * TILE), min(S, ntiles * TILE),
                               scale, lane, [&](int d, float dk, float dv) {
                                   const float v = DK_ROLE ? dk : dv;
                                   if (ck.nch > 1) pp[d] = v;
                                   else outp[d] = (bf16_t)(DK_ROLE ? v * scale : v);
                               });
        row_loaded();
    }
}

// dK/dV workgroup number wg (head fastest, then slot)
template <int DH, bool CAUSAL, bool FLOATW, bool OWN_D>
__device__ __forceinline__ void attn_dkv_wg(char* smem, const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                            const bf16_t* __restrict__ d_o, const float* __restrict__ lse, const float* __restrict__ dsum,
                                            bf16_t* __restrict__ dqkv, int S, int nl, int dh, float c2f, int BH,
                                            float* __restrict__ part, ChunkLen ch, int wg) {
    const int bh = wg % BH, slot = wg / BH;
    const Chunk ck = find_chunk(CAUSAL, true, S, ch, slot, 0);
    float* pslot = part + ((int64_t)slot * BH + bh) * (2 * BLK * DH);
    // the role is uniform per wavefront; both bodies run the same loop and the same barriers
    if ((threadIdx.x >> 6) < 4) attn_dkv_body<DH, CAUSAL, FLOATW, OWN_D, false>(smem, qkv, o, d_o, lse, dsum, dqkv, S, nl, dh, c2f, bh, ck, pslot);
    else attn_dkv_body<DH, CAUSAL, FLOATW, OWN_D, true>(smem, qkv, o, d_o, lse, dsum, dqkv, S, nl, dh, c2f, bh, ck, pslot);
}

// =================================================================================================
// dQ.  Same decomposition as the forward: 8 wavefronts, wavefront w owns query sub-block w % 4 (its Q
// and dO fragments stay in registers) and key half w / 4 of every streamed 64-key tile; the two dQ
// partials of a sub-block are added through LDS in a fixed order.  Transposed score tile: lane = query.
// =================================================================================================
template <int DH> constexpr int dq_lds_bytes() {
    constexpr int ring = 4 * tile_bytes<DH>();
    constexpr int merge = 4 * 64 * (DH / 2) * 4;
    return ring > merge ? ring : merge;
}

// dQ workgroup number wg (head fastest, then slot)
template <int DH, bool CAUSAL, bool FLOATW, bool OWN_D>
__device__ __forceinline__ void attn_dq_wg(char* smem, const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                           const bf16_t* __restrict__ d_o, const float* __restrict__ lse, float* __restrict__ dsum,
                                           bf16_t* __restrict__ dqkv, int S, int nl, int dh, float c2f, int BH,
                                           float* __restrict__ part, ChunkLen ch, int wg) {
    constexpr int TB = tile_bytes<DH>();
    constexpr int NCH = NCHUNKS<DH, FTHREADS>;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, half = lane >> 5;
    const int qs = wave & 3, kvh = wave >> 2;
    const int bh = wg % BH, slot = wg / BH;
    const Chunk ck = find_chunk(CAUSAL, false, S, ch, slot, 0);
    const int qb = ck.blk;
    const int b = bh / nl, h = bh % nl;
    const int64_t ld = 3LL * nl * dh, ldo = (int64_t)nl * dh;
    const bf16_t* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * dh;
    const bf16_t* kbase = qbase + (int64_t)nl * dh;
    const bf16_t* vbase = kbase + (int64_t)nl * dh;
    const bf16_t* dobase = d_o + (int64_t)b * S * ldo + (int64_t)h * dh;
    const int q0 = qb * BLK + qs * 32;
    const int q = q0 + (lane & 31);
    const float scale = 1.0f / sqrtf((float)dh);
    const float c2 = FLOATW ? c2f : LOG2E * scale;
    const float l2 = q < S ? lse[((int64_t)b * nl + h) * S + q] * LOG2E : 0.0f;
    bf16x8 qf[DH / 16], dof[DH / 16];
    float dq_d = 0.0f;                                     // D of the query: half of the row in either lane half
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) {
        qf[ks] = frag_k_global(qbase, ld, q, S, dh, ks, lane);
        dof[ks] = frag_k_global(dobase, ldo, q, S, dh, ks, lane);
    }
    if (OWN_D) {
        float part[DH / 16];
#pragma unroll
        for (int ks = 0; ks < DH / 16; ++ks)
            part[ks] = dot8(frag_k_global(o + (int64_t)b * S * ldo + (int64_t)h * dh, ldo, q, S, dh, ks, lane), dof[ks]);
#pragma unroll
        for (int gap = 1; gap < DH / 16; gap *= 2)
#pragma unroll
            for (int ks = 0; ks + gap < DH / 16; ks += 2 * gap) part[ks] += part[ks + gap];
        dq_d = part[0] + __shfl_xor(part[0], 32, 64);
        if (kvh == 0 && half == 0 && q < S) dsum[((int64_t)b * nl + h) * S + q] = dq_d;
    } else if (q < S) {
        dq_d = dsum[((int64_t)b * nl + h) * S + q];
    }
    f32x16 dq[DH / 32];
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt) dq[dt] = zero16();

    const int kv_end = CAUSAL ? min(S, (qb + 1) * BLK) : S;
    const int tile0 = ck.t0, ntiles = ck.t1;
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const i32x4 desc_k = head_rsrc(kbase, ld, S, dh), desc_v = head_rsrc(vbase, ld, S, dh);
    unsigned off[NCH];
    dma_offsets<DH, FTHREADS>(off, ld, dh, t);
    auto fetch_tile = [&](int kt, unsigned stage) {       // K and V rows of tile kt -> LDS stage
        const unsigned r0 = (unsigned)kt * TILE * (unsigned)(ld * 2);
        tile_dma<DH, FTHREADS>(desc_k, stage, off, r0, wave_u);
        tile_dma<DH, FTHREADS>(desc_v, stage + TB, off, r0, wave_u);
    };
    fetch_tile(tile0, lds0);
#pragma unroll
    for (int ks = 0; ks < DH / 16; ++ks) { settle(qf[ks]); settle(dof[ks]); }
    settle(l2);
    settle(dq_d);
    dma_wait();
    __syncthreads();
    // LDS addresses of the fragments in stage 0, this wavefront's 32 keys; V lies TB behind K.  Kept in registers as in forward.
    constexpr int NF = DH / 16;
    unsigned ka[NF], ta[DH / 32][2];
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) { ka[ks] = lds0 + frag_k_off<DH>(kvh * 32, ks, lane); keep_in_register(ka[ks]); }
#pragma unroll
    for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
        for (int g = 0; g < 2; ++g) { ta[dt][g] = lds0 + frag_t_off<DH>(dt * 32, kvh * 32, g, lane); keep_in_register(ta[dt][g]); }
    auto step = [&](int kt, auto stg) __attribute__((always_inline)) {
        constexpr int OFF = decltype(stg)::value * 2 * TB;
        // the other stage was last read before the barrier that ended the previous step
        if (kt + 1 < ntiles) fetch_tile(kt + 1, lds0 + (1 - decltype(stg)::value) * 2 * TB);
        const int kv0 = kt * TILE + kvh * 32;
        if (kv0 < kv_end && !(CAUSAL && kv0 > q0 + 31)) {                 // wavefront-uniform
            // The fragments of the three MFMA phases (K for S, V for dP, K transposed for dQ) form one sequence that
            // is read through a rolling window of W registers: fragment i + W is requested right after the MFMA
            // that used fragment i, so LDS latency hides under W MFMAs instead of being paid before every one.
            f32x16 s = zero16(), dp = zero16();
            constexpr int W = DH <= 64 ? NF : NF / 2;
            bf16x8 fr[W];
            auto fetch = [&](int i) __attribute__((always_inline)) {      // i is a compile-time constant after unrolling
                if (i < NF) return lds_frag_k<OFF>(ka[i]);
                if (i < 2 * NF) return lds_frag_k<OFF + TB>(ka[i - NF]);
                const int k = i - 2 * NF;
                return k & 1 ? lds_frag_t<OFF + 16 * DH * 2>(ta[k >> 1][0], ta[k >> 1][1]) : lds_frag_t<OFF>(ta[k >> 1][0], ta[k >> 1][1]);
            };
#pragma unroll
            for (int i = 0; i < W; ++i) fr[i] = fetch(i);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < 2 * NF; ++i) {
                if (i < NF) s = MFMA(fr[i % W], qf[i], s);
                else dp = MFMA(fr[i % W], dof[i - NF], dp);
                fr[i % W] = fetch(i + W);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_setprio(0);
            const bool need_mask = q0 + 31 >= S || kv0 + 31 >= S || (CAUSAL && kv0 + 31 > q0);
            if (need_mask) {                          // wave-uniform: only tiles on the diagonal or at the end of S
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    int kv = kv0 + (v >> 2) * 8 + half * 4 + (v & 3);
                    bool ok = q < S && kv < S && (!CAUSAL || kv <= q);
                    s[v] = ok ? s[v] : -INFINITY;         // exp2(-inf) = 0
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) dp[v] = fast_exp2(fmaf(s[v], c2, -l2)) * (dp[v] - dq_d);
            bf16x8 g[weight_terms<FLOATW>()][2];
            split_terms<FLOATW>(dp, g);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int k = 0; k < NF; ++k) {
                dq[k >> 1] = mfma_terms<FLOATW>(fr[k % W], g, k & 1, dq[k >> 1]);
                if (k + W < NF) {
                    fr[k % W] = fetch(2 * NF + k + W);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_s_setprio(0);
        }
        dma_wait();
        __syncthreads();
    };
    for (int kt = tile0; kt < ntiles;) {
        step(kt, std::integral_constant<int, 0>{});
        if (++kt >= ntiles) break;
        step(kt, std::integral_constant<int, 1>{});
        ++kt;
    }
    float* mg = reinterpret_cast<float*>(smem) + (qs * (DH / 2)) * 64 + lane;   // element i at mg[i * 64]
    if (kvh == 1) {
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) mg[(dt * 16 + v) * 64] = dq[dt][v];
    }
    __syncthreads();
    float z = 0.0f;
    if (kvh == 0 && ck.nch > 1) {
        // one chunk of a longer strip: unscaled float partial, [query][dh]
        float* pp = part + ((int64_t)slot * BH + bh) * (BLK * DH) + (qs * 32 + (lane & 31)) * DH;
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float r[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) r[j] = dq[dt][4 * i + j] + mg[(dt * 16 + 4 * i + j) * 64];
                if (FLOATW) note4(z, r);
                store_f4(pp + dt * 32 + 8 * i + 4 * half, r[0], r[1], r[2], r[3]);
            }
    } else if (kvh == 0 && q < S) {
        bf16_t* dqp = dqkv + ((int64_t)b * S + q) * ld + (int64_t)h * dh;
#pragma unroll
        for (int dt = 0; dt < DH / 32; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float r[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) r[j] = (dq[dt][4 * i + j] + mg[(dt * 16 + 4 * i + j) * 64]) * scale;
                if (FLOATW) note4(z, r);
                if (dt * 32 + 8 * i + 4 * half < dh) store4(dqp + dt * 32 + 8 * i + 4 * half, r[0], r[1], r[2], r[3]);
            }
    }
    if (!FLOATW || kvh != 0 || !any_nonfinite(z)) return;
    rows_stored();
    float* q_s = reinterpret_cast<float*>(smem) + qs * (DH / 2) * 64;      // this wavefront alone reads its merge area
    for (int i = q0; i < q0 + 32 && i < S; ++i) {
        load_row(q_s, qbase + (int64_t)i * ld, dh, lane);
        load_row(q_s + DH, dobase + (int64_t)i * ldo, dh, lane);
        row_loaded();
        const int64_t row = ((int64_t)b * nl + h) * S + i;
        const float d_row = __shfl(dq_d, i - q0, 64);
        bf16_t* dqp = dqkv + ((int64_t)b * S + i) * ld + (int64_t)h * dh;
        float* pp = part + ((int64_t)slot * BH + bh) * (BLK * DH) + (i - qb * BLK) * DH;
        attn_row_dq<(DH + 63) / 64>(q_s, q_s + DH, kbase, vbase, ld, dh, tile0 * TILE, min(CAUSAL ? i + 1 : S, ntiles * TILE), scale, lse[row],
                              d_row, lane, [&](int d, float v) { if (ck.nch > 1) pp[d] = v; else dqp[d] = (bf16_t)(v * scale); });
        row_loaded();
    }
}

// =================================================================================================
// Backward in one launch: workgroups [0, wgs_kv) compute dK/dV chunks, the rest dQ chunks.  The two are independent,
// both are bound by their longest strip rather than by the amount of work, and a compute unit holds one such
// workgroup at a time: in one launch the units that finish the short chunks of one kind pick up chunks of the other
// instead of idling until the launch ends.  dK/dV first: its steps are the longer ones.
// =================================================================================================
template <int DH, bool CAUSAL, bool FLOATW, bool OWN_D>
__global__ __launch_bounds__(FTHREADS, 2) void attn_bwd_kernel(const bf16_t* __restrict__ qkv,
                                                               const bf16_t* __restrict__ o,
                                                               const bf16_t* __restrict__ d_o,
                                                               const float* __restrict__ lse,
                                                               float* __restrict__ dsum,
                                                               bf16_t* __restrict__ dqkv, int S, int nl, int dh, float c2f, int BH,
                                                               float* __restrict__ part_kv, float* __restrict__ part_q,
                                                               ChunkLen ch_kv, ChunkLen ch_q, int wgs_kv) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int wg = blockIdx.x;                               // uniform: one kind per workgroup, its own barriers
    if (wg < wgs_kv) attn_dkv_wg<DH, CAUSAL, FLOATW, OWN_D>(smem, qkv, o, d_o, lse, dsum, dqkv, S, nl, dh, c2f, BH, part_kv, ch_kv, wg);
    else attn_dq_wg<DH, CAUSAL, FLOATW, OWN_D>(smem, qkv, o, d_o, lse, dsum, dqkv, S, nl, dh, c2f, BH, part_q, ch_q, wg - wgs_kv);
}

// =================================================================================================
// Head sizes 64 and 128, launches of many workgroups (own_rows): four wavefronts per workgroup, each owning 32 rows (queries, or
// keys in dK/dV) of the block outright, two or more workgroups per compute unit.  The workgroups of a unit share no barrier, so
// one's vector arithmetic and LDS latency run beside another's products, and the scores of dK and dV are worked out once; what
// bounds them still is the sum of a wavefront's LDS reads, vector arithmetic and products (a third of the matrix rate).
//   forward   64 keys at a time: one maximum and one rescale for both halves of a tile, two chains of products
//   backward  (head size 64) the weights of a subtile of 32 rows are worked out between the score products of the next one (7 % at
//             4096 tokens, 16 heads), hence three stages in LDS
// =================================================================================================
constexpr int WTHREADS = 256;

template <int DH, bool CAUSAL>
__global__ __launch_bounds__(WTHREADS, 2) void attn_fwd_rows_kernel(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o, float* __restrict__ lse,
                                                                   int S, int nl, int BH, float* __restrict__ part, ChunkLen ch) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int TB = tile_bytes<DH>(), NF = DH / 16, NT = DH / 32, HALF = 32 * DH * 2;
    constexpr int NCH = NCHUNKS<DH, WTHREADS>;
    const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int bh = blockIdx.x % BH, slot = blockIdx.x / BH;      // head fastest: heaviest chunks of all heads first
    const Chunk ck = find_chunk(CAUSAL, false, S, ch, slot, 0);
    const int b = bh / nl, h = bh % nl;
    const int64_t ld = 3LL * nl * DH;
    const bf16_t* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * DH;
    const bf16_t* kbase = qbase + (int64_t)nl * DH;
    const bf16_t* vbase = kbase + (int64_t)nl * DH;
    const int q0 = ck.blk * BLK + wave * 32, q = q0 + (lane & 31);
    const float c2 = LOG2E / sqrtf((float)DH);

    bf16x8 qf[NF];
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) qf[ks] = frag_k_global(qbase, ld, q, S, DH, ks, lane);
    f32x16 oacc[NT];
#pragma unroll
    for (int dt = 0; dt < NT; ++dt) oacc[dt] = zero16();
    float m = -INFINITY, lsum = 0.0f;

    const int kv_end = CAUSAL ? min(S, q0 + 32) : S;              // keys that any query of this wavefront sees
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    const i32x4 desc_k = head_rsrc(kbase, ld, S, DH), desc_v = head_rsrc(vbase, ld, S, DH);
    unsigned off[NCH];
    dma_offsets<DH, WTHREADS>(off, ld, DH, t);
    auto fetch_tile = [&](int kt, unsigned stage) {
        const unsigned r0 = (unsigned)kt * TILE * (unsigned)(ld * 2);
        tile_dma<DH, WTHREADS>(desc_k, stage, off, r0, wave);
        tile_dma<DH, WTHREADS>(desc_v, stage + TB, off, r0, wave);
    };
    unsigned ka[NF], va[NT][2];
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) { ka[ks] = lds0 + frag_k_off<DH>(0, ks, lane); keep_in_register(ka[ks]); }
#pragma unroll
    for (int dt = 0; dt < NT; ++dt)
#pragma unroll
        for (int g = 0; g < 2; ++g) { va[dt][g] = lds0 + TB + frag_t_off<DH>(dt * 32, 0, g, lane); keep_in_register(va[dt][g]); }
    fetch_tile(ck.t0, lds0);
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) settle(qf[ks]);
    dma_wait();
    __syncthreads();
    auto step = [&](int kt, auto stg) __attribute__((always_inline)) {
        constexpr int SOFF = decltype(stg)::value * 2 * TB;
        if (kt + 1 < ck.t1) fetch_tile(kt + 1, lds0 + (1 - decltype(stg)::value) * 2 * TB);
        const int kv0 = kt * TILE;
        if (kv0 < kv_end) {                                       // wavefront-uniform
            f32x16 s[2] = {zero16(), zero16()};
            bf16x8 fr[2 * NF];                                    // keys 0..31 and 32..63 in turn, two chains of products
#pragma unroll
            for (int ks = 0; ks < NF; ++ks) {
                fr[2 * ks] = lds_frag_k<SOFF>(ka[ks]);
                fr[2 * ks + 1] = lds_frag_k<SOFF + HALF>(ka[ks]);
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int ks = 0; ks < NF; ++ks) {
                s[0] = MFMA(fr[2 * ks], qf[ks], s[0]);
                s[1] = MFMA(fr[2 * ks + 1], qf[ks], s[1]);
            }
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int dt = 0; dt < NT; ++dt) {                     // [16 rows][dt]
                fr[dt] = lds_frag_t<SOFF>(va[dt][0], va[dt][1]);
                fr[NT + dt] = lds_frag_t<SOFF + HALF / 2>(va[dt][0], va[dt][1]);
                fr[2 * NT + dt] = lds_frag_t<SOFF + HALF>(va[dt][0], va[dt][1]);
                fr[3 * NT + dt] = lds_frag_t<SOFF + HALF + HALF / 2>(va[dt][0], va[dt][1]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kv0 + 63 >= S || (CAUSAL && kv0 + 63 > q0)) {
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int kv = kv0 + 32 * g + (v >> 2) * 8 + half * 4 + (v & 3);
                        s[g][v] = kv < S && (!CAUSAL || kv <= q) ? s[g][v] : -INFINITY;
                    }
            }
            float mb = fmaxf(s[0][0], s[1][0]);
#pragma unroll
            for (int v = 1; v < 16; ++v) mb = fmaxf(fmaxf(mb, s[0][v]), s[1][v]);
            mb = cross_half_max(mb) * c2;                         // c2 > 0: scaling commutes with max
            const float mn = (mb - m > RESCALE_LAG) ? mb : m;     // see attn_fwd_kernel
            const float mu = mn == -INFINITY ? 0.0f : mn;
            const float alpha = fast_exp2(m - mu);
            m = mn;
            float ps[2] = {0.0f, 0.0f};
#pragma unroll
            for (int v = 0; v < 16; ++v)
#pragma unroll
                for (int g = 0; g < 2; ++g) { s[g][v] = fast_exp2(fmaf(s[g][v], c2, -mu)); ps[g] += s[g][v]; }
            lsum = lsum * alpha + (ps[0] + ps[1]);
            if (__any(alpha != 1.0f)) {
#pragma unroll
                for (int dt = 0; dt < NT; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
            }
            const bf16x8 pb[4] = {pack_regs(s[0], 0), pack_regs(s[0], 8), pack_regs(s[1], 0), pack_regs(s[1], 8)};
            __builtin_amdgcn_s_setprio(1);
            auto add = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
                for (int r = r0; r < r0 + 2; ++r)
#pragma unroll
                    for (int dt = 0; dt < NT; ++dt) oacc[dt] = MFMA(fr[r * NT + dt], pb[r], oacc[dt]);
            };
            add(0);
            if (!CAUSAL || kv0 + 32 <= q0 + 31) add(2);           // uniform; zero times a later token's infinity is NaN
            __builtin_amdgcn_s_setprio(0);
        }
        dma_wait();
        __syncthreads();
    };
    {
        int kt = ck.t0;
        for (; kt + 1 < ck.t1; kt += 2) {
            step(kt, std::integral_constant<int, 0>{});
            step(kt + 1, std::integral_constant<int, 1>{});
        }
        if (kt < ck.t1) step(kt, std::integral_constant<int, 0>{});
    }
    lsum += __shfl_xor(lsum, 32, 64);
    if (ck.nch > 1) {
        // one chunk of a longer strip: (max, sum, unnormalised O) of this chunk's keys, float, [query][dh]
        float* pp = part + ((int64_t)slot * BH + bh) * (BLK * (DH + 2));
        const int ql = wave * 32 + (lane & 31);
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                store_f4(pp + ql * DH + dt * 32 + 8 * i + 4 * half, oacc[dt][4 * i], oacc[dt][4 * i + 1], oacc[dt][4 * i + 2], oacc[dt][4 * i + 3]);
        if (half == 0) { pp[BLK * DH + ql] = m; pp[BLK * DH + BLK + ql] = lsum; }
    } else if (q < S) {
        const float inv = lsum > 0.0f ? 1.0f / lsum : 0.0f;
        bf16_t* op = o + ((int64_t)b * S + q) * ((int64_t)nl * DH) + (int64_t)h * DH;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                store4(op + dt * 32 + 8 * i + 4 * half, oacc[dt][4 * i] * inv, oacc[dt][4 * i + 1] * inv, oacc[dt][4 * i + 2] * inv, oacc[dt][4 * i + 3] * inv);
        if (half == 0) lse[((int64_t)b * nl + h) * S + q] = strip_lse<false>(m, lsum);
    }
}

// dK and dV of 32 keys per wavefront.  Score tile: lane = key, registers = queries.
template <int DH, bool CAUSAL>
__device__ __forceinline__ void attn_dkv_rows(char* smem, const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ d_o, const float* __restrict__ lse,
                                              const float* __restrict__ dsum, bf16_t* __restrict__ dqkv, int S, int nl, int BH,
                                              float* __restrict__ part, ChunkLen ch, int wg) {
    constexpr int TB = tile_bytes<DH>(), NF = DH / 16, NT = DH / 32, STAGE = 2 * TB + 2 * TILE * 4;   // Q tile, dO tile, LSE*log2e, D
    constexpr int NCH = NCHUNKS<DH, WTHREADS>;
    const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int bh = wg % BH, slot = wg / BH;
    const Chunk ck = find_chunk(CAUSAL, true, S, ch, slot, 0);
    const int b = bh / nl, h = bh % nl;
    const int64_t ld = 3LL * nl * DH, ldo = (int64_t)nl * DH;
    const bf16_t* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * DH;
    const bf16_t* kbase = qbase + (int64_t)nl * DH;
    const bf16_t* vbase = kbase + (int64_t)nl * DH;
    const bf16_t* dobase = d_o + (int64_t)b * S * ldo + (int64_t)h * DH;
    const float* lrow = lse + ((int64_t)b * nl + h) * S;
    const float* drow = dsum + ((int64_t)b * nl + h) * S;
    const int k0 = ck.blk * BLK + wave * 32, kv = k0 + (lane & 31);
    const float scale = 1.0f / sqrtf((float)DH), c2 = LOG2E * scale;

    bf16x8 kf[NF], vf[NF];
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) {
        kf[ks] = frag_k_global(kbase, ld, kv, S, DH, ks, lane);
        vf[ks] = frag_k_global(vbase, ld, kv, S, DH, ks, lane);
    }
    f32x16 dk[NT], dv[NT];
#pragma unroll
    for (int dt = 0; dt < NT; ++dt) dk[dt] = dv[dt] = zero16();
    const int qt0 = ck.t0, ntiles = ck.t1;
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    const i32x4 desc_q = head_rsrc(qbase, ld, S, DH), desc_do = head_rsrc(dobase, ldo, S, DH);
    unsigned off_q[NCH], off_do[NCH];
    dma_offsets<DH, WTHREADS>(off_q, ld, DH, t);
    dma_offsets<DH, WTHREADS>(off_do, ldo, DH, t);
    float rl = 0.0f, rd = 0.0f;
    auto g2r = [&](int qt, unsigned stage) {
        tile_dma<DH, WTHREADS>(desc_q, stage, off_q, (unsigned)qt * TILE * (unsigned)(ld * 2), wave);
        tile_dma<DH, WTHREADS>(desc_do, stage + TB, off_do, (unsigned)qt * TILE * (unsigned)(ldo * 2), wave);
        if (t < TILE) {
            const int qi = qt * TILE + t;
            rl = qi < S ? lrow[qi] * LOG2E : 0.0f;
            rd = qi < S ? drow[qi] : 0.0f;
        }
    };
    auto r2s = [&](char* st) {
        if (t < TILE) {
            reinterpret_cast<float*>(st + 2 * TB)[t] = rl;
            reinterpret_cast<float*>(st + 2 * TB)[TILE + t] = rd;
        }
    };
    if (qt0 < ntiles) { g2r(qt0, lds0); r2s(smem); }
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) { settle(kf[ks]); settle(vf[ks]); }
    dma_wait();
    __syncthreads();
    constexpr int W = 8;
    f32x16 sc[2], dp[2];                                                   // scores and dP of the subtiles, by parity
    unsigned ko[NF], to[NT][2];                                            // this lane's fragment reads in a tile
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) { ko[ks] = frag_k_off<DH>(0, ks, lane); keep_in_register(ko[ks]); }
#pragma unroll
    for (int dt = 0; dt < NT; ++dt)
#pragma unroll
        for (int g = 0; g < 2; ++g) { to[dt][g] = frag_t_off<DH>(dt * 32, 0, g, lane); keep_in_register(to[dt][g]); }
    bool pending = false;
    unsigned prev = 0, prev_ls = 0;                                        // LDS addresses of the pending subtile's Q rows and LSE
    int prev0 = 0;                                                         // its first query
    // P and dS of the pending subtile, element by element, in the shadow of other products
    bf16x8 gp[2], gs[2];
    float lv[16], dd[16];
    auto read_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 l4 = lds_f4(prev_ls + (8 * i + 4 * half) * 4), d4 = lds_f4(prev_ls + TILE * 4 + (8 * i + 4 * half) * 4);
            lv[4 * i] = l4[0]; lv[4 * i + 1] = l4[1]; lv[4 * i + 2] = l4[2]; lv[4 * i + 3] = l4[3];
            dd[4 * i] = d4[0]; dd[4 * i + 1] = d4[1]; dd[4 * i + 2] = d4[2]; dd[4 * i + 3] = d4[3];
        }
    };
    auto mask = [&](f32x16& x) __attribute__((always_inline)) {            // wave-uniform: diagonal, or the end of S
        if (prev0 + 31 >= S || k0 + 31 >= S || (CAUSAL && k0 + 31 > prev0)) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int qi = prev0 + 8 * (v >> 2) + 4 * half + (v & 3);
                x[v] = qi < S && kv < S && (!CAUSAL || kv <= qi) ? x[v] : -INFINITY;   // exp2(-inf) = 0
            }
        }
    };
    auto weigh = [&](f32x16& x, f32x16& y, int v) __attribute__((always_inline)) {
        x[v] = fast_exp2(fmaf(x[v], c2, -lv[v]));
        y[v] = x[v] * (y[v] - dd[v]);
        if ((v & 7) == 7) { gp[v >> 3] = pack_regs(x, v - 7); gs[v >> 3] = pack_regs(y, v - 7); }
    };
    // S and dP of a subtile (two chains of products), and beside them the weights of the pending one
    auto scores = [&](unsigned qsb, f32x16& cs_, f32x16& cd, f32x16& ps_, f32x16& pd, auto pendc) __attribute__((always_inline)) {
        bf16x8 fr[W];
        auto fetch = [&](int i) { return i & 1 ? lds_frag_k<TB>(qsb + ko[i >> 1]) : lds_frag_k<0>(qsb + ko[i >> 1]); };
        if constexpr (decltype(pendc)::value) read_rows();
#pragma unroll
        for (int i = 0; i < W; ++i) fr[i] = fetch(i);
        __builtin_amdgcn_sched_barrier(0);
        cs_ = zero16();
        cd = zero16();
#pragma unroll
        for (int i = 0; i < 2 * NF; ++i) {
            if (i & 1) cd = MFMA(fr[i % W], vf[i >> 1], cd);
            else cs_ = MFMA(fr[i % W], kf[i >> 1], cs_);
            if (i + W < 2 * NF) fr[i % W] = fetch(i + W);
            if constexpr (decltype(pendc)::value) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (v * 2 * NF / 16 == i) weigh(ps_, pd, v);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // dV and dK of the pending subtile
    auto collect = [&]() __attribute__((always_inline)) {
        bf16x8 fr[W];
        auto fetch = [&](int k) {                                          // [dO, Q][16 rows][dt]
            const unsigned a0 = prev + to[k % NT][0], a1 = prev + to[k % NT][1];
            constexpr int R16 = 16 * DH * 2;
            return k < NF ? (k < NT ? lds_frag_t<TB>(a0, a1) : lds_frag_t<TB + R16>(a0, a1))
                          : (k < NF + NT ? lds_frag_t<0>(a0, a1) : lds_frag_t<R16>(a0, a1));
        };
#pragma unroll
        for (int i = 0; i < W; ++i) fr[i] = fetch(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 2 * NF; ++k) {
            if (k < NF) dv[k % NT] = MFMA(fr[k % W], gp[k / NT], dv[k % NT]);
            else dk[k % NT] = MFMA(fr[k % W], gs[(k - NF) / NT], dk[k % NT]);
            if (k + W < 2 * NF) fr[k % W] = fetch(k + W);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto subtile = [&](unsigned st, int qt, auto sbc) __attribute__((always_inline)) {
        constexpr int SB = decltype(sbc)::value;
        const int qs0 = qt * TILE + SB * 32;
        if (qs0 >= S || (CAUSAL && qs0 + 31 < k0)) return;                 // wavefront-uniform; only before the first and after the last
        const unsigned qsb = st + SB * 32 * DH * 2;
        if (pending) {
            mask(sc[SB ^ 1]);
            scores(qsb, sc[SB], dp[SB], sc[SB ^ 1], dp[SB ^ 1], std::true_type{});
            collect();
        } else {
            scores(qsb, sc[SB], dp[SB], sc[SB ^ 1], dp[SB ^ 1], std::false_type{});
        }
        pending = true;
        prev = qsb;
        prev0 = qs0;
        prev_ls = st + 2 * TB + SB * 32 * 4;
    };
    int stage = 0;
    for (int qt = qt0; qt < ntiles; ++qt) {
        const unsigned st = lds0 + stage * STAGE;
        const int nstage = stage == 2 ? 0 : stage + 1;                     // last read before the barrier before last
        const bool more = qt + 1 < ntiles;
        if (more) g2r(qt + 1, lds0 + nstage * STAGE);
        subtile(st, qt, std::integral_constant<int, 0>{});
        subtile(st, qt, std::integral_constant<int, 1>{});
        if (more) r2s(smem + nstage * STAGE);
        dma_wait();
        __syncthreads();
        stage = nstage;
    }
    if (pending) {
        // the last one, by the parity of its place in a tile
        if ((prev0 / 32) & 1) {
            mask(sc[1]);
            read_rows();
#pragma unroll
            for (int v = 0; v < 16; ++v) weigh(sc[1], dp[1], v);
        } else {
            mask(sc[0]);
            read_rows();
#pragma unroll
            for (int v = 0; v < 16; ++v) weigh(sc[0], dp[0], v);
        }
        collect();
    }
#pragma unroll
    for (int which = 0; which < 2; ++which) {                             // dK, dV
        const f32x16 (&acc)[NT] = which ? dv : dk;
        const float f = which ? 1.0f : scale;
        if (ck.nch > 1) {
            // one chunk of a longer strip: unscaled float partial, [dK | dV][key][dh]
            float* pp = part + ((int64_t)slot * BH + bh) * (2 * BLK * DH) + which * BLK * DH + (wave * 32 + (lane & 31)) * DH;
#pragma unroll
            for (int dt = 0; dt < NT; ++dt)
#pragma unroll
                for (int i = 0; i < 4; ++i) store_f4(pp + dt * 32 + 8 * i + 4 * half, acc[dt][4 * i], acc[dt][4 * i + 1], acc[dt][4 * i + 2], acc[dt][4 * i + 3]);
        } else if (kv < S) {
            bf16_t* outp = dqkv + ((int64_t)b * S + kv) * ld + (int64_t)(1 + which) * nl * DH + (int64_t)h * DH;
#pragma unroll
            for (int dt = 0; dt < NT; ++dt)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    store4(outp + dt * 32 + 8 * i + 4 * half, acc[dt][4 * i] * f, acc[dt][4 * i + 1] * f, acc[dt][4 * i + 2] * f, acc[dt][4 * i + 3] * f);
        }
    }
}

// dQ of 32 queries per wavefront.  Transposed score tile: lane = query.
template <int DH, bool CAUSAL>
__device__ __forceinline__ void attn_dq_rows(char* smem, const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ d_o, const float* __restrict__ lse,
                                             const float* __restrict__ dsum, bf16_t* __restrict__ dqkv, int S, int nl, int BH,
                                             float* __restrict__ part, ChunkLen ch, int wg) {
    constexpr int TB = tile_bytes<DH>(), NF = DH / 16, NT = DH / 32;
    constexpr int NCH = NCHUNKS<DH, WTHREADS>;
    const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int bh = wg % BH, slot = wg / BH;
    const Chunk ck = find_chunk(CAUSAL, false, S, ch, slot, 0);
    const int b = bh / nl, h = bh % nl;
    const int64_t ld = 3LL * nl * DH, ldo = (int64_t)nl * DH;
    const bf16_t* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * DH;
    const bf16_t* kbase = qbase + (int64_t)nl * DH;
    const bf16_t* vbase = kbase + (int64_t)nl * DH;
    const bf16_t* dobase = d_o + (int64_t)b * S * ldo + (int64_t)h * DH;
    const int q0 = ck.blk * BLK + wave * 32, q = q0 + (lane & 31);
    const float scale = 1.0f / sqrtf((float)DH), c2 = LOG2E * scale;
    const float l2 = q < S ? lse[((int64_t)b * nl + h) * S + q] * LOG2E : 0.0f;
    const float dq_d = q < S ? dsum[((int64_t)b * nl + h) * S + q] : 0.0f;

    bf16x8 qf[NF], dof[NF];
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) {
        qf[ks] = frag_k_global(qbase, ld, q, S, DH, ks, lane);
        dof[ks] = frag_k_global(dobase, ldo, q, S, DH, ks, lane);
    }
    f32x16 dq[NT];
#pragma unroll
    for (int dt = 0; dt < NT; ++dt) dq[dt] = zero16();
    const int kv_end = CAUSAL ? min(S, q0 + 32) : S;
    const int tile0 = ck.t0, ntiles = ck.t1;
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    const i32x4 desc_k = head_rsrc(kbase, ld, S, DH), desc_v = head_rsrc(vbase, ld, S, DH);
    unsigned off[NCH];
    dma_offsets<DH, WTHREADS>(off, ld, DH, t);
    auto fetch_tile = [&](int kt, unsigned stage) {
        const unsigned r0 = (unsigned)kt * TILE * (unsigned)(ld * 2);
        tile_dma<DH, WTHREADS>(desc_k, stage, off, r0, wave);
        tile_dma<DH, WTHREADS>(desc_v, stage + TB, off, r0, wave);
    };
    fetch_tile(tile0, lds0);
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) { settle(qf[ks]); settle(dof[ks]); }
    settle(l2);
    settle(dq_d);
    dma_wait();
    __syncthreads();
    constexpr int W = 8;
    f32x16 sc[2], dp[2];                                                   // as in attn_dkv_rows
    unsigned ko[NF], to[NT][2];
#pragma unroll
    for (int ks = 0; ks < NF; ++ks) { ko[ks] = frag_k_off<DH>(0, ks, lane); keep_in_register(ko[ks]); }
#pragma unroll
    for (int dt = 0; dt < NT; ++dt)
#pragma unroll
        for (int g = 0; g < 2; ++g) { to[dt][g] = frag_t_off<DH>(dt * 32, 0, g, lane); keep_in_register(to[dt][g]); }
    bool pending = false;
    unsigned prev = 0;
    int prev0 = 0;
    bf16x8 gs[2];
    auto mask = [&](f32x16& x) __attribute__((always_inline)) {
        if (q0 + 31 >= S || prev0 + 31 >= S || (CAUSAL && prev0 + 31 > q0)) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int kv = prev0 + (v >> 2) * 8 + half * 4 + (v & 3);
                x[v] = q < S && kv < S && (!CAUSAL || kv <= q) ? x[v] : -INFINITY;
            }
        }
    };
    auto weigh = [&](f32x16& x, f32x16& y, int v) __attribute__((always_inline)) {
        y[v] = fast_exp2(fmaf(x[v], c2, -l2)) * (y[v] - dq_d);
        if ((v & 7) == 7) gs[v >> 3] = pack_regs(y, v - 7);
    };
    auto scores = [&](unsigned kb, f32x16& cs_, f32x16& cd, f32x16& ps_, f32x16& pd, auto pendc) __attribute__((always_inline)) {
        bf16x8 fr[W];
        auto fetch = [&](int i) { return i & 1 ? lds_frag_k<TB>(kb + ko[i >> 1]) : lds_frag_k<0>(kb + ko[i >> 1]); };
#pragma unroll
        for (int i = 0; i < W; ++i) fr[i] = fetch(i);
        __builtin_amdgcn_sched_barrier(0);
        cs_ = zero16();
        cd = zero16();
#pragma unroll
        for (int i = 0; i < 2 * NF; ++i) {
            if (i & 1) cd = MFMA(fr[i % W], dof[i >> 1], cd);
            else cs_ = MFMA(fr[i % W], qf[i >> 1], cs_);
            if (i + W < 2 * NF) fr[i % W] = fetch(i + W);
            if constexpr (decltype(pendc)::value) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (v * 2 * NF / 16 == i) weigh(ps_, pd, v);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto collect = [&]() __attribute__((always_inline)) {
        bf16x8 fr[NF];
#pragma unroll
        for (int k = 0; k < NF; ++k)
            fr[k] = k < NT ? lds_frag_t<0>(prev + to[k % NT][0], prev + to[k % NT][1]) : lds_frag_t<16 * DH * 2>(prev + to[k % NT][0], prev + to[k % NT][1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < NF; ++k) dq[k % NT] = MFMA(fr[k], gs[k / NT], dq[k % NT]);
    };
    auto subtile = [&](unsigned st, int kt, auto sbc) __attribute__((always_inline)) {
        constexpr int SB = decltype(sbc)::value;
        const int kv0 = kt * TILE + SB * 32;
        if (kv0 >= kv_end) return;                                         // wavefront-uniform; only after the last
        const unsigned kb = st + SB * 32 * DH * 2;
        if (pending) {
            mask(sc[SB ^ 1]);
            scores(kb, sc[SB], dp[SB], sc[SB ^ 1], dp[SB ^ 1], std::true_type{});
            collect();
        } else {
            scores(kb, sc[SB], dp[SB], sc[SB ^ 1], dp[SB ^ 1], std::false_type{});
        }
        pending = true;
        prev = kb;
        prev0 = kv0;
    };
    int stage = 0;
    for (int kt = tile0; kt < ntiles; ++kt) {
        const int nstage = stage == 2 ? 0 : stage + 1;
        if (kt + 1 < ntiles) fetch_tile(kt + 1, lds0 + nstage * 2 * TB);
        subtile(lds0 + stage * 2 * TB, kt, std::integral_constant<int, 0>{});
        subtile(lds0 + stage * 2 * TB, kt, std::integral_constant<int, 1>{});
        dma_wait();
        __syncthreads();
        stage = nstage;
    }
    if (pending) {
        if ((prev0 / 32) & 1) {
            mask(sc[1]);
#pragma unroll
            for (int v = 0; v < 16; ++v) weigh(sc[1], dp[1], v);
        } else {
            mask(sc[0]);
#pragma unroll
            for (int v = 0; v < 16; ++v) weigh(sc[0], dp[0], v);
        }
        collect();
    }
    if (ck.nch > 1) {
        float* pp = part + ((int64_t)slot * BH + bh) * (BLK * DH) + (wave * 32 + (lane & 31)) * DH;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) store_f4(pp + dt * 32 + 8 * i + 4 * half, dq[dt][4 * i], dq[dt][4 * i + 1], dq[dt][4 * i + 2], dq[dt][4 * i + 3]);
    } else if (q < S) {
        bf16_t* dqp = dqkv + ((int64_t)b * S + q) * ld + (int64_t)h * DH;
#pragma unroll
        for (int dt = 0; dt < NT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                store4(dqp + dt * 32 + 8 * i + 4 * half, dq[dt][4 * i] * scale, dq[dt][4 * i + 1] * scale, dq[dt][4 * i + 2] * scale, dq[dt][4 * i + 3] * scale);
    }
}

template <int DH, bool CAUSAL>
__global__ __launch_bounds__(WTHREADS, 2) void attn_bwd_rows_kernel(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ d_o, const float* __restrict__ lse,
                                                                   const float* __restrict__ dsum, bf16_t* __restrict__ dqkv, int S, int nl, int BH,
                                                                   float* __restrict__ part_kv, float* __restrict__ part_q, ChunkLen ch_kv, ChunkLen ch_q,
                                                                   int wgs_kv) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int wg = blockIdx.x;                               // uniform: one kind per workgroup, its own barriers
    if (wg < wgs_kv) attn_dkv_rows<DH, CAUSAL>(smem, qkv, d_o, lse, dsum, dqkv, S, nl, BH, part_kv, ch_kv, wg);
    else attn_dq_rows<DH, CAUSAL>(smem, qkv, d_o, lse, dsum, dqkv, S, nl, BH, part_q, ch_q, wg - wgs_kv);
}

// ---- host side ----------------------------------------------------------------------------------
bool attn_bf16_supported(const AttnArgs& a) {
    // tile loads address a (batch, head) slice with 32-bit byte offsets; where columns may be padded, HEAD_OOB plus the
    // offset of any row of the last tile must not wrap either
    const int64_t rows = a.dh == 64 || a.dh == 128 ? a.S : (int64_t)a.S + TILE;
    // a launch has fewer than 2^32 threads, in backward those of two workgroups per block
    const int64_t threads = (a.S + BLK - 1) / BLK * (int64_t)a.B * a.nl * 2 * FTHREADS;
    return a.dtype == BF16 && a.dh % 8 == 0 && a.dh <= 128 && a.S >= 1 && (int64_t)a.B * a.nl <= 65535 &&
           rows * 3 * a.nl * a.dh * 2 < (1LL << 31) && threads < (1LL << 32);
}

template <typename K>
static hipError_t set_lds(K kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// Chunk length in tile steps.  No workspace: strips are never cut.  The option attn_chunk = n forces n (0: never cut).
// Every workgroup costs a few steps' worth of start-up and merge and every cut strip its partials, so strips are
// cut only where the longest one would otherwise set the duration, and never into chunks of fewer than 8 steps.
constexpr int NEVER_CUT = 1 << 30;
static bool forced_chunk(const AttnArgs& a, int* ch) {
    if (!a.ws) { *ch = NEVER_CUT; return true; }
    if (const int v = options().attn_chunk; v >= 0) {
        *ch = v > 0 && v < (1 << 16) ? v : NEVER_CUT;
        return true;
    }
    // A layer pass leaves its strips whole.  With its GEMMs one by one on two chains attention shares the chip with those of the
    // other chain, and cutting measured 1.2 % slower per step.  Where they go out in groups it has the chip to itself; forward
    // of one sequence, us, whole and cut to the best of 8 to 24 steps: 12 heads of 2048 tokens (12288 / 1536) 734 and 734, 10
    // (5120 / 1280) 308 and 304, 4 of 4096 tokens (4096 / 512) 232 and 213.  A cut would need room in the pass's workspace.
    if (!a.own_chunking) { *ch = NEVER_CUT; return true; }
    return false;
}
static int device_cus() {
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        hipDeviceProp_t pr;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&pr, dev) != hipSuccess) return 0;
        cus = pr.multiProcessorCount;
    }
    return cus;
}
// Forward (a launch of its own): only when there are fewer strips than compute units (with more, the units that
// finish their short strips early pick up the queued ones): the shortest chunk length for which the chunks of all
// heads still run in one round (one workgroup per compute unit, 5 % over allowed).
static int chunk_tiles_fwd(const AttnArgs& a) {
    int ch;
    if (forced_chunk(a, &ch)) return ch;
    const int cus = device_cus();
    const int64_t bh = (int64_t)a.B * a.nl, nblk = (a.S + BLK - 1) / BLK;
    if (!cus || nblk * bh >= cus) return NEVER_CUT;
    const int longest = (a.S + TILE - 1) / TILE;
    for (ch = 8; ch < longest; ++ch)
        if (strip_slots(a.causal, false, a.S, make_chunk_len(ch)) * bh * 100 <= 105LL * cus) return ch;
    return NEVER_CUT;
}
// Backward: dK/dV and dQ workgroups share one launch, so the units that finish short strips of one kind pick up
// strips of the other; with at least as many workgroups as compute units cutting measured no faster (the combine
// kernel costs what the shorter critical path gains).  With fewer, the same rule as forward over both kinds.
static int chunk_tiles_bwd(const AttnArgs& a, bool kv_side) {
    int ch;
    (void)kv_side;                              // one length for both kinds
    if (forced_chunk(a, &ch)) return ch;
    const int cus = device_cus();
    const int64_t bh = (int64_t)a.B * a.nl, nblk = (a.S + BLK - 1) / BLK;
    if (!cus || 2 * nblk * bh >= cus) return NEVER_CUT;
    const int longest = (a.S + TILE - 1) / TILE;
    for (ch = 8; ch < longest; ++ch) {
        const ChunkLen c = make_chunk_len(ch);
        if ((strip_slots(a.causal, false, a.S, c) + strip_slots(a.causal, true, a.S, c)) * bh * 100 <= 105LL * cus) return ch;
    }
    return NEVER_CUT;
}
static bool float_weights(int dh) { return dh != 64 && dh != 128; }
// log2(e) / sqrt(dh), the scale of the scores with FLOATW: rounded once, not once per operation
static float scale_log2(int dh) { return (float)(1.44269504088896340736 / sqrt((double)dh)); }
static int padded_dh(int dh) { return (dh + 31) / 32 * 32; }
static size_t part_bytes_fwd(const AttnArgs& a, ChunkLen ch) {
    return (size_t)strip_slots(a.causal, false, a.S, ch) * a.B * a.nl * BLK * (padded_dh(a.dh) + 2) * sizeof(float);
}
static size_t part_bytes_dq(const AttnArgs& a, ChunkLen ch) {
    return (size_t)strip_slots(a.causal, false, a.S, ch) * a.B * a.nl * BLK * padded_dh(a.dh) * sizeof(float);
}
static size_t part_bytes_dkv(const AttnArgs& a, ChunkLen ch) {
    return (size_t)strip_slots(a.causal, true, a.S, ch) * a.B * a.nl * BLK * 2 * padded_dh(a.dh) * sizeof(float);
}
// Blocks whose strips are cut: a contiguous range (strip length is monotonic in the block index).
static void cut_range(const AttnArgs& a, bool kv_side, ChunkLen ch, int* blk0, int* n) {
    const int nblk = (a.S + BLK - 1) / BLK;
    int lo = nblk, hi = -1;
    for (int blk = 0; blk < nblk; ++blk)
        if (strip_tiles(a.causal, kv_side, a.S, blk) > ch.ch) { lo = blk < lo ? blk : lo; hi = blk; }
    *blk0 = hi < 0 ? 0 : lo;
    *n = hi < 0 ? 0 : hi - lo + 1;
}
static bool cuts(const AttnArgs& a, bool kv_side, ChunkLen ch) {
    return strip_slots(a.causal, kv_side, a.S, ch) != (a.S + BLK - 1) / BLK;
}
// Workspace that lets the strips be cut (0: they would not be cut anyway).  Sized with a stand-in non-null
// workspace pointer so that the same rule decides as at launch.
size_t attn_bf16_workspace_bytes(const AttnArgs& a0, bool bwd) {
    AttnArgs a = a0;
    a.ws = reinterpret_cast<void*>(16);
    if (!bwd) {
        const ChunkLen ch = make_chunk_len(chunk_tiles_fwd(a));
        return cuts(a, false, ch) ? part_bytes_fwd(a, ch) : 0;
    }
    const ChunkLen ch_q = make_chunk_len(chunk_tiles_bwd(a, false)), ch_kv = make_chunk_len(chunk_tiles_bwd(a, true));
    return (cuts(a, false, ch_q) ? part_bytes_dq(a, ch_q) : 0) + (cuts(a, true, ch_kv) ? part_bytes_dkv(a, ch_kv) : 0);
}

// Whether a launch of n workgroups, the longest of `steps` tile steps, goes to the kernels whose wavefronts own their rows outright.  A
// wavefront alone walks a strip in up to 1.3 times the time (without a mask; 1.9 on the diagonal's half strips), so the longest strip of a
// launch that finds its units at once would set the duration; with more workgroups than units two share one and hide each other's waits.
// us with keys (roles) shared by two wavefronts and with own rows:
//   forward, no mask   up to a workgroup per unit: head size 128, 64 workgroups of 256 / 384 / 2048 / 4096 tokens 10.5 and 10.2 / 12.6 and
//                      12.8 / 35 and 41 / 63 and 79; head size 64 of 512 / 768 / 1024 / 4096 tokens 10.0 and 9.7 / 13.1 and 13.2 / 16.3 and
//                      16.5 / 47 and 51.  Beyond: 288 workgroups of 4096 tokens 133 and 102 (64: 75 and 70), 1024 292 and 264 (168 and 158);
//                      768 of 4096 to 8192 tokens at head size 128, three rounds of one form, level (218 and 221, 415 and 427)
//   forward, causal    head size 128: 768 workgroups 297 and 220, 640 of 512 / 8192 tokens 35 and 27 / 203 and 194, 320 39.5 and 48.9;
//                      head size 64: 640 of 512 / 2048 / 4096 / 8192 tokens 20 and 16 / 38.2 and 36.8 / 63.8 and 65.2 / 119.7 and 122.9, 704
//                      of 4096 71.2 and 68.5, 512 59 and 59
//   backward           head size 64: 1024 workgroups 165 and 141 causal, 59.4 and 47.8 without a mask, 512 35 and 38, 256 18 and 21; head
//                      size 128 (a wavefront per SIMD, 420 registers) 845 and 988 when both roles worked the scores out, so not built
static bool own_rows(int dh, bool causal, bool bwd, int64_t n, int steps) {
    const int64_t cus = compute_units();
    if (bwd) return n >= 3 * cus;
    if (causal) return 4 * n >= (dh == 64 && steps > 48 ? 11 : 10) * cus;
    return n > cus || steps <= (dh == 64 ? 12 : 5);
}

// Whether the workgroups (n) of attn_bwd_kernel work D out for themselves, so that the row-dot kernel and its 2 us are not launched.  A dQ
// workgroup does it once, one of dK/dV for every tile, between the barrier that hands the tile over and the first product: 0.1 to 0.2 us a
// tile step at head size 64, 0.3 at 128.  Lines, each with both sides measured, us, kernel of its own and without:
// - up to 16 steps to a unit, 12 above head size 64.  Forward and backward, 40: 25 heads of 810 80.7 and 79.5, 8 of 1467 85.7 and 86.6; 64: 23 of
//   1002 causal 53.4 and 48.6; 8: 18 of 1746 106.4 and 107.5; 128: 5 of 685 47.5 and 45.9, 20 of 1268 108.0 and 109.8; 96: 28 of 805 101.3 and 102.0.
// - up to 4 workgroups to a unit, 6 up to head size 64, 16 up to 32: a workgroup of few tiles is mostly its start, which D makes longer, and many of
//   them share the kernel's launch.  Backward alone, 128: heads of 64 tokens 512 / 1024 / 4096 37.6 and 36.8 / 70.1 and 72.2 / 294 and 320, 192 of
//   256 causal 53.8 and 51.9, 768 of 192 causal 153 and 160; 40: of 64 causal 512 / 1024 / 4096 26.5 and 25.9 / 52.6 and 53.4 / 185 and 195; 32: of 32
//   2048 / 4096 37.6 and 37.0 / 68.4 and 70.1.
// - above head size 64, where strips of 7 tiles and more stay whole, no last round up to a third full, which the lone workgroups' longer steps
//   make longer, and without a mask no third round.  Backward alone, 128: 512 tokens, 32 / 40 / 48 heads 28.0 and 26.4 / 35.9 and 37.4 / 44.0 and
//   42.9, causal 40 / 48 30.0 and 31.8 / 34.1 and 33.3, 576 tokens 48 / 56 48.8 and 48.2 / 64.5 and 65.6.
static bool own_dsum(int DH, bool causal, int S, int BH, ChunkLen ch, int64_t n) {
    const int cus = compute_units(), tiles = (S + TILE - 1) / TILE;
    int64_t steps = 0;
    for (int blk = 0; blk < (S + BLK - 1) / BLK; ++blk) steps += strip_tiles(causal, true, S, blk);
    if (std::max((int64_t)std::min(ch.ch, tiles), steps * BH / cus) > (DH <= 64 ? 16 : 12)) return false;
    if (n > (int64_t)(DH <= 32 ? 16 : DH <= 64 ? 6 : 4) * cus) return false;
    if (DH <= 64 || n <= cus || tiles < 7 || ch.ch < tiles) return true;
    return (n - 1) % cus >= cus / 3 && (causal || n <= 2 * cus);
}

template <int DH, bool CAUSAL, bool FLOATW>
static hipError_t fwd_t(const AttnArgs& a) {
    constexpr int LDS = fwd_lds_bytes<DH>(), LDS_ROWS = 4 * tile_bytes<DH>();
    static bool once = false;
    if (!once) {
        hipError_t e = set_lds(&attn_fwd_kernel<DH, CAUSAL, FLOATW>, LDS);
        if constexpr (!FLOATW) if (e == hipSuccess) e = set_lds(&attn_fwd_rows_kernel<DH, CAUSAL>, LDS_ROWS);
        if (e != hipSuccess) return e;
        once = true;
    }
    const ChunkLen ch = make_chunk_len(chunk_tiles_fwd(a));
    if (a.ws && cuts(a, false, ch) && part_bytes_fwd(a, ch) > a.ws_bytes) return hipErrorInvalidValue;
    const int BH = a.B * a.nl;
    const int64_t wgs = (int64_t)strip_slots(CAUSAL, false, a.S, ch) * BH;
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    float* part = static_cast<float*>(a.ws);
    bool launched = false;
    if constexpr (!FLOATW) {
        if (own_rows(DH, CAUSAL, false, wgs, std::min(ch.ch, (a.S + TILE - 1) / TILE))) {
            hipLaunchKernelGGL((attn_fwd_rows_kernel<DH, CAUSAL>), dim3((unsigned)wgs), dim3(WTHREADS), LDS_ROWS, a.stream,
                               (const bf16_t*)a.qkv, (bf16_t*)a.o, a.lse, a.S, a.nl, BH, part, ch);
            launched = true;
        }
    }
    if (!launched)
        hipLaunchKernelGGL((attn_fwd_kernel<DH, CAUSAL, FLOATW>), dim3((unsigned)wgs), dim3(FTHREADS), LDS, a.stream,
                           (const bf16_t*)a.qkv, (bf16_t*)a.o, a.lse, a.S, a.nl, a.dh, scale_log2(a.dh), BH, part, ch);
    int blk0 = 0, ncut = 0;
    cut_range(a, false, ch, &blk0, &ncut);
    if (ncut)
        hipLaunchKernelGGL((attn_fwd_combine_kernel<DH, CAUSAL, FLOATW>), dim3(ncut * (BLK * combine_tpr<DH>() / 256), BH), dim3(256), 0,
                           a.stream, part, (bf16_t*)a.o, a.lse, a.S, a.nl, a.dh, BH, ch, blk0);
    return hipGetLastError();
}

template <int DH, bool CAUSAL, bool FLOATW>
static hipError_t bwd_t(const AttnArgs& a) {
    constexpr int LDS_KV = dkv_lds_bytes<DH>();
    constexpr int LDS_Q = dq_lds_bytes<DH>();
    constexpr int LDS = LDS_KV > LDS_Q ? LDS_KV : LDS_Q;
    constexpr bool OWN_ROWS = DH == 64 && !FLOATW;
    constexpr int LDS_ROWS = 3 * (2 * tile_bytes<DH>() + 2 * TILE * 4);
    static bool once = false;
    if (!once) {
        hipError_t e = set_lds(&attn_bwd_kernel<DH, CAUSAL, FLOATW, false>, LDS);
        if (e == hipSuccess) e = set_lds(&attn_bwd_kernel<DH, CAUSAL, FLOATW, true>, LDS);
        if constexpr (OWN_ROWS) if (e == hipSuccess) e = set_lds(&attn_bwd_rows_kernel<DH, CAUSAL>, LDS_ROWS);
        if (e != hipSuccess) return e;
        once = true;
    }
    const ChunkLen ch_q = make_chunk_len(chunk_tiles_bwd(a, false)), ch_kv = make_chunk_len(chunk_tiles_bwd(a, true));
    const bool cut_q = cuts(a, false, ch_q), cut_kv = cuts(a, true, ch_kv);
    const size_t bytes_q = cut_q ? part_bytes_dq(a, ch_q) : 0, bytes_kv = cut_kv ? part_bytes_dkv(a, ch_kv) : 0;
    if (a.ws && bytes_q + bytes_kv > a.ws_bytes) return hipErrorInvalidValue;
    const int BH = a.B * a.nl;
    const int64_t wgs_q = (int64_t)strip_slots(CAUSAL, false, a.S, ch_q) * BH;
    const int64_t wgs_kv = (int64_t)strip_slots(CAUSAL, true, a.S, ch_kv) * BH;
    if (wgs_q + wgs_kv > 0x7fffffffLL) return hipErrorInvalidValue;
    float* part_q = static_cast<float*>(a.ws);
    float* part_kv = a.ws ? reinterpret_cast<float*>(static_cast<char*>(a.ws) + bytes_q) : nullptr;
    const bool rows = OWN_ROWS && own_rows(DH, CAUSAL, true, wgs_kv + wgs_q, 0);
    const bool own_d = !rows && own_dsum(DH, CAUSAL, a.S, BH, ch_kv, wgs_kv + wgs_q);
    if (!own_d) {
        const int64_t lanes = (int64_t)a.B * a.S * a.nl * (DH <= 32 ? 4 : DH == 64 ? 8 : 16);
        hipLaunchKernelGGL((attn_dsum_kernel<DH>), dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, a.stream,
                           (const bf16_t*)a.o, (const bf16_t*)a.d_o, a.dsum, a.B, a.S, a.nl, a.dh);
    }
    bool launched = false;
    if constexpr (OWN_ROWS) {
        if (rows) {
            hipLaunchKernelGGL((attn_bwd_rows_kernel<DH, CAUSAL>), dim3((unsigned)(wgs_kv + wgs_q)), dim3(WTHREADS), LDS_ROWS, a.stream,
                               (const bf16_t*)a.qkv, (const bf16_t*)a.d_o, a.lse, a.dsum, (bf16_t*)a.dqkv, a.S, a.nl, BH, part_kv, part_q,
                               ch_kv, ch_q, (int)wgs_kv);
            launched = true;
        }
    }
    const auto kernel = own_d ? &attn_bwd_kernel<DH, CAUSAL, FLOATW, true> : &attn_bwd_kernel<DH, CAUSAL, FLOATW, false>;
    if (!launched)
        hipLaunchKernelGGL(kernel, dim3((unsigned)(wgs_kv + wgs_q)), dim3(FTHREADS), LDS, a.stream,
                           (const bf16_t*)a.qkv, (const bf16_t*)a.o, (const bf16_t*)a.d_o, a.lse, a.dsum, (bf16_t*)a.dqkv, a.S, a.nl, a.dh,
                           scale_log2(a.dh), BH, part_kv, part_q, ch_kv, ch_q, (int)wgs_kv);
    int blk0_q = 0, ncut_q = 0, blk0_kv = 0, ncut_kv = 0;
    cut_range(a, false, ch_q, &blk0_q, &ncut_q);
    cut_range(a, true, ch_kv, &blk0_kv, &ncut_kv);
    if (ncut_q || ncut_kv)
        hipLaunchKernelGGL((attn_bwd_combine_kernel<DH, CAUSAL>),
                           dim3((ncut_q > ncut_kv ? ncut_q : ncut_kv) * (BLK * combine_tpr<DH>() / 256), BH, 3), dim3(256), 0, a.stream,
                           part_q, part_kv, (bf16_t*)a.dqkv, a.S, a.nl, a.dh, BH, ch_q, ch_kv, blk0_q, ncut_q, blk0_kv,
                           ncut_kv);
    return hipGetLastError();
}

template <int DH, bool FLOATW>
static hipError_t run_dh(const AttnArgs& a, bool bwd) {
    if (bwd) return a.causal ? bwd_t<DH, true, FLOATW>(a) : bwd_t<DH, false, FLOATW>(a);
    return a.causal ? fwd_t<DH, true, FLOATW>(a) : fwd_t<DH, false, FLOATW>(a);
}
static hipError_t run_attention(const AttnArgs& a, bool bwd) {
    switch (padded_dh(a.dh)) {
        case 32: return run_dh<32, true>(a, bwd);
        case 64: return float_weights(a.dh) ? run_dh<64, true>(a, bwd) : run_dh<64, false>(a, bwd);
        case 96: return run_dh<96, true>(a, bwd);
        default: return float_weights(a.dh) ? run_dh<128, true>(a, bwd) : run_dh<128, false>(a, bwd);
    }
}
hipError_t attn_bf16_fwd(const AttnArgs& a) { return run_attention(a, false); }
hipError_t attn_bf16_bwd(const AttnArgs& a) { return run_attention(a, true); }

}  // namespace tpl

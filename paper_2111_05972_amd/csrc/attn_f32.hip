// float softmax attention for gfx950 on the matrix cores (MFMA 32x32x2 f32), head sizes up to 128, forward and backward.
//
// What bounds it.  A 32 x 32 tile of scores takes DH / 2 instructions of 64 cycles, its value product as many again, for
// two operand registers per lane each: matrix time dwarfs everything else, including the softmax arithmetic and the
// operand traffic.  So the kernels are arranged for many independent wavefronts rather than for operand reuse: a
// workgroup owns 32 rows (queries in forward and dQ, keys in dK/dV) of one (batch, head), its four wavefronts walk every
// fourth 32-row tile of the other side with LDS tiles of their own (no barrier in the loop), and the four results are
// combined through LDS at the end in wavefront order.
//
// Measured (16 heads x 512 x 64, no mask): forward 19.6 us (1.07 GFLOP), backward 48 us, where one wavefront per row on
// vector arithmetic took 338 and 670 us.
//
// Register layouts.  The accumulator of a 32 x 32 block gives lane l column l % 32 and rows 8 i + 4 (l / 32) + j (register
// 4 i + j).  Forward and dQ compute scores transposed (rows = keys, columns = queries), dK/dV untransposed (rows =
// queries, columns = keys).  The next product sums over those rows two at a time, lanes 0..31 one row and lanes 32..63
// another; instruction 4 i + j takes rows 8 i + j and 8 i + 4 + j, which are register 4 i + j as it stands: probabilities
// are an operand without any movement.  Products over the head dimension take element e of a lane's 16-byte read of its
// row (d = 8 g + 4 (l / 32) + e) the same way.
//
// Staging.  Tiles are copied by buffer_load ... lds; rows past the sequence and head columns past dh (DH is dh rounded up
// to 32) read zero.  A tile is requested as soon as its slot has been read for the last time and is waited for by count.
#include <hip/hip_runtime.h>

#include "attn_rows.h"
#include "device_math.h"
#include "kernels.h"
#include "lds_dma.h"

namespace tpl {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int XT = 32;                         // rows of a tile
constexpr unsigned X_OOB = 0x80000000u;
#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x2f32((a), (b), (c), 0, 0, 0)

// Tile of 32 rows x DH floats in LDS: chunk (16 bytes) c of row r at position c ^ xswz(r) of its row.  Two kinds of read:
// 16 bytes of 16 consecutive rows at one chunk, and single floats of 32 consecutive columns of rows r and r + 4.
template <int DH> __device__ __forceinline__ int xswz(int r) {
    if ((DH / 4) % 16 == 0) return (((r >> 2) & 1) << 3) | (((r >> 3) & 1) << 2) | (r & 3);
    return (r >> 1) & 7;                        // rows of 128 or 384 bytes: neighbours already differ by half a bank line
}
template <int DH> constexpr int xtile_bytes() { return XT * DH * 4; }
template <int DH> constexpr int xloads() { return DH / 8; }           // direct loads per lane and tile (one wavefront)

template <int DH>
__device__ __forceinline__ void xoffsets(unsigned (&off)[xloads<DH>()], int64_t ld, int dh, int lane) {
    constexpr int NC = DH / 4;
#pragma unroll
    for (int i = 0; i < xloads<DH>(); ++i) {
        const int p = lane + 64 * i, r = p / NC, c = (p % NC) ^ xswz<DH>(r);
        off[i] = 4 * c < dh ? (unsigned)r * (unsigned)(ld * 4) + (unsigned)c * 16u : X_OOB;
    }
}
template <int DH>
__device__ __forceinline__ void xfetch(const i32x4& rsrc, unsigned lds, const unsigned (&off)[xloads<DH>()], int row0, int64_t ld) {
    const unsigned r0 = (unsigned)row0 * (unsigned)(ld * 4);
#pragma unroll
    for (int i = 0; i < xloads<DH>(); ++i) buffer_load_lds_b128(rsrc, lds + i * 1024, off[i] + r0);
}
template <int N> __device__ __forceinline__ void xwait() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
// The LDS reads issued so far have delivered: their slot may be overwritten.
__device__ __forceinline__ void xreads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// acc += T[32 rows] R^T over the head dimension: rows of the LDS tile against the lane's register row
template <int DH>
__device__ __forceinline__ f32x16 xscores(const char* tile, const float (&r)[DH / 2], int lane) {
    const int row = lane & 31, half = lane >> 5, x = xswz<DH>(row);
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.0f;
#pragma unroll
    for (int g = 0; g < DH / 8; ++g) {
        const float4 a = *reinterpret_cast<const float4*>(tile + row * (DH * 4) + (((2 * g + half) ^ x) << 4));
        s = MFMA32(a.x, r[4 * g + 0], s);
        s = MFMA32(a.y, r[4 * g + 1], s);
        s = MFMA32(a.z, r[4 * g + 2], s);
        s = MFMA32(a.w, r[4 * g + 3], s);
    }
    return s;
}
// acc[d block][.] += T^T W: sum over the 32 tile rows, weights in accumulator order
template <int DH>
__device__ __forceinline__ void xaccumulate(f32x16 (&acc)[DH / 32], const char* tile, const f32x16& w, int lane) {
    const int half = lane >> 5, col = lane & 31;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = 8 * (v >> 2) + 4 * half + (v & 3);
#pragma unroll
        for (int d = 0; d < DH / 32; ++d) {
            const int c = (d * 32 + col) >> 2;
            const float a = *reinterpret_cast<const float*>(tile + r * (DH * 4) + ((c ^ xswz<DH>(r)) << 4) + (col & 3) * 4);
            acc[d] = MFMA32(a, w[v], acc[d]);
        }
    }
}
// The lane's row (of 32) of a row-major global matrix in operand order; zero past nrows and past dh.
template <int DH>
__device__ __forceinline__ void xrow(float (&r)[DH / 2], const float* base, int64_t ld, int row, int nrows, int dh, int lane) {
    const int half = lane >> 5;
#pragma unroll
    for (int g = 0; g < DH / 8; ++g) {
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const int d = 8 * g + 4 * half;
        if (row < nrows && d < dh) v = *reinterpret_cast<const float4*>(base + (int64_t)row * ld + d);
        r[4 * g] = v.x; r[4 * g + 1] = v.y; r[4 * g + 2] = v.z; r[4 * g + 3] = v.w;
    }
}
__device__ __forceinline__ i32x4 xrsrc(const float* base, int64_t ld, int S, int dh) {
    return make_rsrc(base, (unsigned)(((int64_t)(S - 1) * ld + dh) * 4));
}
__device__ __forceinline__ float xother(float v) { return __shfl_xor(v, 32, 64); }

// Adds the four wavefronts' blocks in wavefront order, each scaled by its f, and hands element (row 8 i + 4 half + j,
// column) to put(d block, i, four rows' values): wavefront w writes accumulator quads w of every block, rows for which
// xmine(row, w).  Returns 0, or NaN if one of the lane's values is not finite.
//
// Infinities and NaN under the causal mask.  The matrix instruction multiplies a masked weight, zero, with its row, and zero
// times infinity is NaN: in the tile that the diagonal crosses, a token would reach tokens before it.  A wavefront that ends
// with a value that is not finite therefore computes what it has written again, row by row, where a masked row is not read
// (attn_rows.h; LDS at xrows).
__device__ __forceinline__ bool xmine(int row, int wave) { return ((row >> 3) & 3) == wave; }
template <int DH, typename Put>
__device__ __forceinline__ float xcombine(char* smem, const f32x16 (&acc)[DH / 32], const float (&f)[4], int wave, int lane, Put put) {
    float* red = reinterpret_cast<float*>(smem);                  // [wavefront][block][register][lane]
    __syncthreads();
#pragma unroll
    for (int d = 0; d < DH / 32; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[((wave * (DH / 32) + d) * 16 + v) * 64 + lane] = acc[d][v];
    __syncthreads();
    float z = 0.0f;
#pragma unroll
    for (int d = 0; d < DH / 32; ++d) {
        float r[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int v = wave * 4 + j;
            float s = red[(d * 16 + v) * 64 + lane] * f[0];
#pragma unroll
            for (int w = 1; w < 4; ++w) s = fmaf(red[((w * (DH / 32) + d) * 16 + v) * 64 + lane], f[w], s);
            r[j] = s;
            z = fmaf(s, 0.0f, z);
        }
        put(d, wave, r);
    }
    return z;
}

// two tiles per wavefront (also the combine area), row terms, two rows per wavefront for attn_rows.h
template <int DH> constexpr int xlds_bytes() { return 4 * 2 * xtile_bytes<DH>() + 4 * 2 * XT * 4 + 4 * 2 * DH * 4; }
template <int DH> __device__ __forceinline__ float* xrows(char* smem, int wave) {
    return reinterpret_cast<float*>(smem + 4 * 2 * xtile_bytes<DH>() + 4 * 2 * XT * 4) + wave * 2 * DH;
}

// ---- forward: workgroup = (32 queries, batch*head) ---------------------------------------------------------------
template <int DH>
__global__ __launch_bounds__(256) void attn_f32_fwd_kernel(int S, int nl, int dh, int causal, int nblk, const float* __restrict__ qkv,
                                                           float* __restrict__ o, float* __restrict__ lse) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int TB = xtile_bytes<DH>(), NL = xloads<DH>();
    const int lane = threadIdx.x & 63, half = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qb = nblk - 1 - (int)blockIdx.x % nblk, bh = blockIdx.x / nblk, b = bh / nl, h = bh % nl;   // long strips first
    const int64_t ld = 3LL * nl * dh;
    const float* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * dh;
    const i32x4 rk = xrsrc(qbase + (int64_t)nl * dh, ld, S, dh), rv = xrsrc(qbase + 2LL * nl * dh, ld, S, dh);
    const int q0 = qb * XT, q = q0 + (lane & 31);
    const float scale = 1.0f / sqrtf((float)dh);
    float qr[DH / 2];
    xrow<DH>(qr, qbase, ld, q, S, dh, lane);
    f32x16 acc[DH / 32];
#pragma unroll
    for (int d = 0; d < DH / 32; ++d)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[d][v] = 0.0f;
    float m = -INFINITY, l = 0.0f;
    const int nt = causal ? qb + 1 : (S + XT - 1) / XT;
    char* kt_ = smem + wave * 2 * TB;
    const unsigned lk = (unsigned)(uintptr_t)(lds_void_ptr)kt_, lv = lk + TB;
    unsigned off[NL];
    xoffsets<DH>(off, ld, dh, lane);
    if (wave < nt) { xfetch<DH>(rk, lk, off, wave * XT, ld); xfetch<DH>(rv, lv, off, wave * XT, ld); }
    for (int t = wave; t < nt; t += 4) {
        const int nx = t + 4;
        xwait<NL>();                                              // K of this tile (V is younger)
        f32x16 s = xscores<DH>(kt_, qr, lane);
        xreads_done();
        // past the last tile this reads rows past the end (zeros), so that the count of loads in flight stays the same
        xfetch<DH>(rk, lk, off, nx < nt ? nx * XT : S, ld);
        const int k0 = t * XT;
        const bool edge = k0 + XT > S || (causal && k0 + XT - 1 > q0);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] *= scale;
            if (edge) {
                const int k = k0 + 8 * (v >> 2) + 4 * half + (v & 3);
                if (k >= S || (causal && k > q)) s[v] = -INFINITY;
            }
        }
        float mt = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mt = fmaxf(mt, s[v]);
        mt = fmaxf(mt, xother(mt));
        const float mn = fmaxf(m, mt), mu = mn == -INFINITY ? 0.0f : mn, alpha = expf(m - mu);
        m = mn;
        float ps = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; ++v) { s[v] = expf(s[v] - mu); ps += s[v]; }
        l = l * alpha + ps;
#pragma unroll
        for (int d = 0; d < DH / 32; ++d)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[d][v] *= alpha;
        xwait<NL>();                                              // V of this tile (the next K is younger)
        xaccumulate<DH>(acc, kt_ + TB, s, lane);
        xreads_done();
        xfetch<DH>(rv, lv, off, nx < nt ? nx * XT : S, ld);
    }
    xwait<0>();
    l += xother(l);
    float* st = reinterpret_cast<float*>(smem + 8 * TB);          // [wavefront][m, l][query]
    if (half == 0) { st[wave * 64 + lane] = m; st[wave * 64 + 32 + lane] = l; }
    __syncthreads();
    float mt = -INFINITY, f[4], lt = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) mt = fmaxf(mt, st[w * 64 + (lane & 31)]);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        f[w] = expf(st[w * 64 + (lane & 31)] - (mt == -INFINITY ? 0.0f : mt));   // all scores -inf: sum 0, LSE -inf
        lt = fmaf(st[w * 64 + 32 + (lane & 31)], f[w], lt);
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) f[w] /= lt;
    float* op = o + ((int64_t)b * S + q) * ((int64_t)nl * dh) + (int64_t)h * dh;
    const float z = xcombine<DH>(smem, acc, f, wave, lane, [&](int d, int i, const float (&r)[4]) {
        const int c = d * 32 + 8 * i + 4 * half;
        if (q < S && c < dh) *reinterpret_cast<float4*>(op + c) = make_float4(r[0], r[1], r[2], r[3]);
    });
    if (wave == 0 && half == 0 && q < S) lse[(int64_t)bh * S + q] = mt + logf(lt);
    if (!causal || !__any(z != 0.0f)) return;
    rows_stored();
    float* q_s = xrows<DH>(smem, wave);
    for (int i = q0; i < q0 + XT && i < S; ++i) {
        load_row(q_s, qbase + (int64_t)i * ld, dh, lane);
        row_loaded();
        float* oi = o + ((int64_t)b * S + i) * ((int64_t)nl * dh) + (int64_t)h * dh;
        float mr, lr;
        attn_row_fwd<(DH + 63) / 64>(q_s, qbase + (int64_t)nl * dh, qbase + 2LL * nl * dh, ld, dh, 0, i + 1, scale, true, lane, mr, lr,
                                     [&](int d, float v) { if (xmine(d, wave)) oi[d] = v; });
        row_loaded();
    }
}

// Where dK/dV gets D = rowsum(dO * O) from: dQ's launch before, attn_f32_dsum_kernel, or itself.
enum { D_OF_DQ, D_GIVEN, D_OWN };

// D: 16 lanes per (token, head)
__global__ __launch_bounds__(256) void attn_f32_dsum_kernel(const float* __restrict__ o, const float* __restrict__ d_o, float* __restrict__ dsum,
                                                            int B, int S, int nl, int dh) {
    const int64_t items = (int64_t)B * S * nl;                                                 // token-major, then head
    const int l = threadIdx.x % 16;
    for (int64_t item = ((int64_t)blockIdx.x * 256 + threadIdx.x) / 16; item < items; item += (int64_t)gridDim.x * 16) {
        float D = 0.0f;
        for (int c = 4 * l; c < dh; c += 64) {
            const float4 x = *reinterpret_cast<const float4*>(o + item * dh + c), g = *reinterpret_cast<const float4*>(d_o + item * dh + c);
            D = fmaf(x.x, g.x, D); D = fmaf(x.y, g.y, D); D = fmaf(x.z, g.z, D); D = fmaf(x.w, g.w, D);
        }
#pragma unroll
        for (int i = 8; i > 0; i >>= 1) D += __shfl_xor(D, i, 64);
        if (l == 0) {
            const int64_t row = item / nl;
            dsum[((row / S) * nl + (item - row * nl)) * S + row % S] = D;
        }
    }
}

// ---- backward: n workgroups of (32 keys, batch*head) for dK and dV, n of (32 queries, batch*head) for dQ ------------------------------
// KIND_BOTH: all of them in one launch, dK/dV first; this launch starts at workgroup wg0 of the 2 n.  dK/dV does not wait for dQ's: D is
// given or worked out for its query tiles as well.  With D given two workgroups share a compute unit (at most 256 registers).  dQ leaves D
// for dK/dV unless it is given; D_OWN: dK/dV stores the same value that dQ's workgroups store.
// Both stand in the kernel itself: as functions called from it they spilled up to 24 scalar registers (2048 tokens, 4 heads of 80 / 128,
// causal 213 / 326 us, so 208 / 298; heads of 32 1 to 5 % faster, of 64 between 2 % slower and 3 % faster).
enum { KIND_DQ, KIND_DKV, KIND_BOTH };
template <int DH, int DK_D, int KIND>
__global__ __launch_bounds__(256, DK_D == D_GIVEN ? 2 : 1) void attn_f32_bwd_kernel(int n, int wg0, int S, int nl, int dh, int causal, int nblk, const float* __restrict__ qkv,
                                                           const float* __restrict__ o, const float* __restrict__ lse,
                                                           const float* __restrict__ d_o, float* __restrict__ dqkv, float* dsum) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int first = blockIdx.x + wg0;                           // uniform: one kind per workgroup
    if (KIND == KIND_DQ || (KIND == KIND_BOTH && first >= n)) {
        const int wg = KIND == KIND_BOTH ? first - n : first;
        constexpr int TB = xtile_bytes<DH>(), NL = xloads<DH>();
        const int lane = threadIdx.x & 63, half = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int qb = nblk - 1 - wg % nblk, bh = wg / nblk, b = bh / nl, h = bh % nl;
        const int64_t ld = 3LL * nl * dh, ldo = (int64_t)nl * dh;
        const float* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * dh;
        const i32x4 rk = xrsrc(qbase + (int64_t)nl * dh, ld, S, dh), rv = xrsrc(qbase + 2LL * nl * dh, ld, S, dh);
        const int q0 = qb * XT, q = q0 + (lane & 31);
        const float scale = 1.0f / sqrtf((float)dh);
        char* kt_ = smem + wave * 2 * TB;
        const unsigned lk = (unsigned)(uintptr_t)(lds_void_ptr)kt_, lv = lk + TB;
        float qr[DH / 2], gr[DH / 2];
        xrow<DH>(qr, qbase, ld, q, S, dh, lane);
        const int64_t orow = (int64_t)b * S * ldo + (int64_t)h * dh;
        xrow<DH>(gr, d_o + orow, ldo, q, S, dh, lane);
        float D = 0.0f;
        {
            float orr[DH / 2];
            xrow<DH>(orr, o + orow, ldo, q, S, dh, lane);
#pragma unroll
            for (int e = 0; e < DH / 2; ++e) D = fmaf(gr[e], orr[e], D);
            D += xother(D);
        }
        const float L = q < S ? lse[(int64_t)bh * S + q] : 0.0f;
        if (DK_D != D_GIVEN && wave == 0 && half == 0 && q < S) dsum[(int64_t)bh * S + q] = D;
        f32x16 acc[DH / 32];
#pragma unroll
        for (int d = 0; d < DH / 32; ++d)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[d][v] = 0.0f;
        const int nt = causal ? qb + 1 : (S + XT - 1) / XT;
        unsigned off[NL];
        xoffsets<DH>(off, ld, dh, lane);
        // V first: it is read first
        if (wave < nt) { xfetch<DH>(rv, lv, off, wave * XT, ld); xfetch<DH>(rk, lk, off, wave * XT, ld); }
        for (int t = wave; t < nt; t += 4) {
            const int nx = t + 4;
            xwait<NL>();
            f32x16 dp = xscores<DH>(kt_ + TB, gr, lane);              // dP^T = V dO^T
            xreads_done();
            xfetch<DH>(rv, lv, off, nx < nt ? nx * XT : S, ld);
            xwait<NL>();
            const f32x16 s = xscores<DH>(kt_, qr, lane);
            const int k0 = t * XT;
            const bool edge = k0 + XT > S || (causal && k0 + XT - 1 > q0);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float p = expf(s[v] * scale - L);
                if (edge) {
                    const int k = k0 + 8 * (v >> 2) + 4 * half + (v & 3);
                    if (k >= S || (causal && k > q)) p = 0.0f;
                }
                dp[v] = p * (dp[v] - D);
            }
            xaccumulate<DH>(acc, kt_, dp, lane);                      // dQ^T += K^T dS
            xreads_done();
            xfetch<DH>(rk, lk, off, nx < nt ? nx * XT : S, ld);
        }
        xwait<0>();
        const float f[4] = {scale, scale, scale, scale};
        float* dqp = dqkv + ((int64_t)b * S + q) * ld + (int64_t)h * dh;
        const float z = xcombine<DH>(smem, acc, f, wave, lane, [&](int d, int i, const float (&r)[4]) {
            const int c = d * 32 + 8 * i + 4 * half;
            if (q < S && c < dh) *reinterpret_cast<float4*>(dqp + c) = make_float4(r[0], r[1], r[2], r[3]);
        });
        if (!causal || !__any(z != 0.0f)) return;
        rows_stored();
        float* q_s = xrows<DH>(smem, wave);
        for (int i = q0; i < q0 + XT && i < S; ++i) {
            load_row(q_s, qbase + (int64_t)i * ld, dh, lane);
            load_row(q_s + DH, d_o + orow + (int64_t)i * ldo, dh, lane);
            row_loaded();
            float* dqi = dqkv + ((int64_t)b * S + i) * ld + (int64_t)h * dh;
            float Di = 0.0f;
            for (int d = lane; d < dh; d += 64) Di = fmaf(q_s[DH + d], o[orow + (int64_t)i * ldo + d], Di);
            attn_row_dq<(DH + 63) / 64>(q_s, q_s + DH, qbase + (int64_t)nl * dh, qbase + 2LL * nl * dh, ld, dh, 0, i + 1, scale,
                                        lse[(int64_t)bh * S + i], row_sum(Di), lane, [&](int d, float v) { if (xmine(d, wave)) dqi[d] = v * scale; });
            row_loaded();
        }
        return;
    }
    if constexpr (KIND != KIND_DQ) {
        const int wg = first;
        constexpr int TB = xtile_bytes<DH>(), NL = xloads<DH>();
        const int lane = threadIdx.x & 63, half = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int kb = wg % nblk, bh = wg / nblk, b = bh / nl, h = bh % nl;   // long strips first
        const int64_t ld = 3LL * nl * dh, ldo = (int64_t)nl * dh;
        const float* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * dh;
        const i32x4 rq = xrsrc(qbase, ld, S, dh), rg = xrsrc(d_o + (int64_t)b * S * ldo + (int64_t)h * dh, ldo, S, dh);
        const int k0 = kb * XT, k = k0 + (lane & 31);
        const float scale = 1.0f / sqrtf((float)dh);
        float kr[DH / 2], vr[DH / 2];
        xrow<DH>(kr, qbase + (int64_t)nl * dh, ld, k, S, dh, lane);
        xrow<DH>(vr, qbase + 2LL * nl * dh, ld, k, S, dh, lane);
        f32x16 dk[DH / 32], dv[DH / 32];
#pragma unroll
        for (int d = 0; d < DH / 32; ++d)
#pragma unroll
            for (int v = 0; v < 16; ++v) { dk[d][v] = 0.0f; dv[d][v] = 0.0f; }
        const float* lrow = lse + (int64_t)bh * S;
        float* drow = dsum + (int64_t)bh * S;
        char* qt_ = smem + wave * 2 * TB;
        const unsigned lq = (unsigned)(uintptr_t)(lds_void_ptr)qt_, lg = lq + TB;
        float* terms = reinterpret_cast<float*>(smem + 8 * TB) + wave * 2 * XT;   // LSE, D of the tile's queries
        const int t0 = causal ? kb : 0, nt = (S + XT - 1) / XT;
        unsigned offq[NL], offg[NL];
        xoffsets<DH>(offq, ld, dh, lane);
        xoffsets<DH>(offg, ldo, dh, lane);
        auto term = [&](int t) {                                      // lanes 0..31: LSE, lanes 32..63: D
            const int i = t * XT + (lane & 31);
            if constexpr (DK_D == D_OWN) {
                float gr[DH / 2], orr[DH / 2], D = 0.0f;
                const int64_t orow = (int64_t)b * S * ldo + (int64_t)h * dh;
                xrow<DH>(gr, d_o + orow, ldo, i, S, dh, lane);
                xrow<DH>(orr, o + orow, ldo, i, S, dh, lane);
#pragma unroll
                for (int e = 0; e < DH / 2; ++e) D = fmaf(gr[e], orr[e], D);
                D += xother(D);
                if (half == 0 && i < S) drow[i] = D;
                return i < S ? (half ? D : lrow[i]) : 0.0f;
            }
            return i < S ? (half ? drow[i] : lrow[i]) : 0.0f;
        };
        float tn = 0.0f;
        if (t0 + wave < nt) {
            tn = term(t0 + wave);
            xfetch<DH>(rq, lq, offq, (t0 + wave) * XT, ld);
            xfetch<DH>(rg, lg, offg, (t0 + wave) * XT, ldo);
        }
        for (int t = t0 + wave; t < nt; t += 4) {
            const int nx = t + 4;
            terms[lane] = tn;
            xwait<0>();
            if (nx < nt) tn = term(nx);
            f32x16 p = xscores<DH>(qt_, kr, lane);
            f32x16 ds = xscores<DH>(qt_ + TB, vr, lane);              // dP = dO V^T
            const int q0 = t * XT;
            const bool edge = q0 + XT > S || k0 + XT > S || (causal && k0 + XT - 1 > q0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 l4 = *reinterpret_cast<const float4*>(terms + 8 * i + 4 * half);
                const float4 d4 = *reinterpret_cast<const float4*>(terms + XT + 8 * i + 4 * half);
                const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dv4[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int v = 4 * i + j;
                    float e = expf(p[v] * scale - lv[j]);
                    if (edge) {
                        const int q = q0 + 8 * i + 4 * half + j;
                        if (q >= S || k >= S || (causal && k > q)) e = 0.0f;
                    }
                    p[v] = e;
                    ds[v] = e * (ds[v] - dv4[j]);
                }
            }
            xaccumulate<DH>(dv, qt_ + TB, p, lane);                   // dV^T += dO^T P
            xreads_done();
            xfetch<DH>(rg, lg, offg, nx < nt ? nx * XT : S, ldo);
            xaccumulate<DH>(dk, qt_, ds, lane);                       // dK^T += Q^T dS
            xreads_done();
            xfetch<DH>(rq, lq, offq, nx < nt ? nx * XT : S, ld);
        }
        xwait<0>();
        float* kp = dqkv + ((int64_t)b * S + k) * ld + (int64_t)nl * dh + (int64_t)h * dh;
        float* vp = kp + (int64_t)nl * dh;
        const float fk[4] = {scale, scale, scale, scale}, fv[4] = {1.0f, 1.0f, 1.0f, 1.0f};
        float z = xcombine<DH>(smem, dk, fk, wave, lane, [&](int d, int i, const float (&r)[4]) {
            const int c = d * 32 + 8 * i + 4 * half;
            if (k < S && c < dh) *reinterpret_cast<float4*>(kp + c) = make_float4(r[0], r[1], r[2], r[3]);
        });
        z += xcombine<DH>(smem, dv, fv, wave, lane, [&](int d, int i, const float (&r)[4]) {
            const int c = d * 32 + 8 * i + 4 * half;
            if (k < S && c < dh) *reinterpret_cast<float4*>(vp + c) = make_float4(r[0], r[1], r[2], r[3]);
        });
        if (!causal || !__any(z != 0.0f)) return;
        rows_stored();
        float* k_s = xrows<DH>(smem, wave);
        for (int j = k0; j < k0 + XT && j < S; ++j) {
            const float* kj = qbase + (int64_t)nl * dh + (int64_t)j * ld;
            load_row(k_s, kj, dh, lane);
            load_row(k_s + DH, kj + (int64_t)nl * dh, dh, lane);
            row_loaded();
            float* dkj = dqkv + ((int64_t)b * S + j) * ld + (int64_t)nl * dh + (int64_t)h * dh;
            float* dvj = dkj + (int64_t)nl * dh;
            attn_row_dkv<(DH + 63) / 64>(k_s, k_s + DH, qbase, ld, d_o + (int64_t)b * S * ldo + (int64_t)h * dh, ldo, lrow, [&](int i) { return drow[i]; }, dh, j, S, scale,
                                         lane, [&](int d, float a, float v) { if (xmine(d, wave)) { dkj[d] = a * scale; dvj[d] = v; } });
            row_loaded();
        }
    }
}

// ---- host ----------------------------------------------------------------------------------------------------------------
bool attn_f32_supported(const AttnArgs& a) {
    // 16-byte chunks of a head's row; 32-bit byte offsets inside a (batch, head) slice, 32 rows past its end included; fewer
    // than 2^32 threads in a launch
    return a.dtype == F32 && a.dh % 4 == 0 && a.dh <= 128 && ((int64_t)a.S + XT) * 3 * a.nl * a.dh * 4 < (1LL << 31) &&
           (int64_t)a.B * a.nl * ((a.S + XT - 1) / XT) * 256 < (1LL << 32);
}
// Head sizes whose two kinds of workgroups share a compute unit, by registers and LDS: D by a kernel of its own, then dQ and dK/dV in
// one launch.  A wavefront alone on its SIMD waits for its tiles and its dependent products; two fill each other's waits.  us, two
// launches one after the other and so: 4 x 512, 4 heads of 64 55.6 and 48.5, 8 heads 95.6 and 82.9; 2048 tokens, 16 heads of 64, causal
// 562 and 436; 300 tokens, 16 heads of 64, causal 41.1 and 29.5; 4 x 512, 8 heads of 32 47.8 and 45.7.  Wider heads need 330 registers.
template <int DH> constexpr bool pairs() { return DH <= 64; }
template <int DH>
static hipError_t set_lds() {
    hipError_t e = hipSuccess;
    auto set = [&](const void* k) { if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, xlds_bytes<DH>()); };
    set(reinterpret_cast<const void*>(&attn_f32_fwd_kernel<DH>));
    set(reinterpret_cast<const void*>(&attn_f32_bwd_kernel<DH, D_OWN, KIND_BOTH>));
    if constexpr (pairs<DH>()) {
        set(reinterpret_cast<const void*>(&attn_f32_bwd_kernel<DH, D_GIVEN, KIND_BOTH>));
    } else {
        set(reinterpret_cast<const void*>(&attn_f32_bwd_kernel<DH, D_OF_DQ, KIND_DQ>));
        set(reinterpret_cast<const void*>(&attn_f32_bwd_kernel<DH, D_OF_DQ, KIND_DKV>));
    }
    return e;
}
// dQ and dK/dV in one launch where all their workgroups find a compute unit at once: neither waits for the other, and a launch is
// saved.  us, two launches and one, n workgroups of each kind: n = 16 (2 x 128 tokens, 2 heads of 64, causal) 21.0 and 13.2, n = 64
// 31.4 and 21.7, n = 128 52 and 37 (heads of 128: 171 and 129); with more of them D, worked out again, costs more than that: n = 256
// 58 and 63, n = 512 96 and 115, where D comes from a kernel of its own (pairs) or from dQ's launch.
static bool one_launch(int64_t n) { return 2 * n <= compute_units(); }
template <int DH>
static hipError_t launch(const AttnArgs& a, bool bwd) {
    static const hipError_t attr = set_lds<DH>();
    if (attr != hipSuccess) return attr;
    const int nblk = (a.S + XT - 1) / XT;
    const dim3 grid((unsigned)(nblk * a.B * a.nl)), wg(256);
    if (!bwd) {
        hipLaunchKernelGGL(attn_f32_fwd_kernel<DH>, grid, wg, xlds_bytes<DH>(), a.stream, a.S, a.nl, a.dh, a.causal, nblk,
                           (const float*)a.qkv, (float*)a.o, a.lse);
        return hipGetLastError();
    }
    if (one_launch((int64_t)nblk * a.B * a.nl)) {
        const dim3 both(2 * grid.x);
        hipLaunchKernelGGL((attn_f32_bwd_kernel<DH, D_OWN, KIND_BOTH>), both, wg, xlds_bytes<DH>(), a.stream, (int)grid.x, 0, a.S, a.nl, a.dh, a.causal, nblk,
                           (const float*)a.qkv, (const float*)a.o, a.lse, (const float*)a.d_o, (float*)a.dqkv, a.dsum);
        return hipGetLastError();
    }
    if constexpr (pairs<DH>()) {
        const int64_t rows16 = ((int64_t)a.B * a.S * a.nl + 15) / 16;
        hipLaunchKernelGGL(attn_f32_dsum_kernel, dim3((unsigned)(rows16 < 1 << 20 ? rows16 : 1 << 20)), wg, 0, a.stream, (const float*)a.o,
                           (const float*)a.d_o, a.dsum, a.B, a.S, a.nl, a.dh);
        const bool fits = 2LL * grid.x * wg.x < 1LL << 32;            // a launch has fewer than 2^32 threads
        for (unsigned wg0 = 0; wg0 < 2 * grid.x; wg0 += fits ? 2 * grid.x : grid.x)
            hipLaunchKernelGGL((attn_f32_bwd_kernel<DH, D_GIVEN, KIND_BOTH>), dim3(fits ? 2 * grid.x : grid.x), wg, xlds_bytes<DH>(), a.stream, (int)grid.x,
                               (int)wg0, a.S, a.nl, a.dh, a.causal, nblk, (const float*)a.qkv, (const float*)a.o, a.lse, (const float*)a.d_o,
                               (float*)a.dqkv, a.dsum);
    } else {
        hipLaunchKernelGGL((attn_f32_bwd_kernel<DH, D_OF_DQ, KIND_DQ>), grid, wg, xlds_bytes<DH>(), a.stream, (int)grid.x, 0, a.S, a.nl, a.dh, a.causal, nblk,
                           (const float*)a.qkv, (const float*)a.o, a.lse, (const float*)a.d_o, (float*)a.dqkv, a.dsum);
        hipLaunchKernelGGL((attn_f32_bwd_kernel<DH, D_OF_DQ, KIND_DKV>), grid, wg, xlds_bytes<DH>(), a.stream, (int)grid.x, 0, a.S, a.nl, a.dh, a.causal, nblk,
                           (const float*)a.qkv, (const float*)a.o, a.lse, (const float*)a.d_o, (float*)a.dqkv, a.dsum);
    }
    return hipGetLastError();
}
static hipError_t attn_f32(const AttnArgs& a, bool bwd) {
    switch ((a.dh + 31) / 32) {
        case 1: return launch<32>(a, bwd);
        case 2: return launch<64>(a, bwd);
        case 3: return launch<96>(a, bwd);
        default: return launch<128>(a, bwd);
    }
}
hipError_t attn_f32_fwd(const AttnArgs& a) { return attn_f32(a, false); }
hipError_t attn_f32_bwd(const AttnArgs& a) { return attn_f32(a, true); }

}  // namespace tpl

// float GEMM for gfx950: C[M,N] = epi(opA(A) opB(B)) on the matrix cores (MFMA 32x32x2 f32: float operands, float
// accumulation, so nothing is rounded that the generic kernel did not round; only the order of the sums differs).
//
// What bounds it.  A 32x32x2 instruction is 64 cycles for two operand registers per lane, so LDS and global bandwidth
// are far from their limits at any tile and the kernel is bound by the matrix pipe where there is work for all of it,
// by latency where there is not.  Hence three tiles that differ only in how much of the output one workgroup takes:
//   128 x 128   2 x 2 wavefronts of 64 x 64                     (many tiles)
//    64 x 64    2 x 2 wavefronts of 32 x 32
//    32 x 32    4 wavefronts on the same block, each a quarter of every k-step, added through LDS in wavefront order
// and K cut into shares (one workgroup per tile and share, float partial sums in the workspace added in share order by
// gemm_f32_sum_kernel) where even those leave compute units idle.
//
// Measured (floor: flops at the 154 TFLOP/s of a large float product): 4096 x 2048 x 2048 262 us (floor 223) on the
// 128-wide tile, 276 and 318 on the narrower ones; 2048 x 1024 x 1024 41 us (28) on the 64-wide, 44 and 47 on the others;
// 256 x 512 x 256 4.2 us, a launch's least, on the 32-wide, where the generic kernel with its 64 x 64 tiles of vector
// arithmetic took 46; 384 x 384 x 16384 55 us (31) in 16 shares of 32-wide tiles.  The estimate in f32_plan is within 5 %
// of the best (tile, shares) on 33 of 34 such shapes.
//
// Pipeline.  K in steps of 32 through an LDS ring filled by buffer_load ... lds (128-byte rows: whole cache lines;
// everything outside the matrix reads zero), one barrier per step, the loads of step kt + STAGES - 1 issued right after
// the barrier of step kt.  Operands stay in the layout they have in memory:
//   K contiguous      rows of 32 k; a lane reads 4 consecutive k of its row (16 bytes)
//   M or N contiguous rows of the tile's width per k; a lane reads one float per k
// A k-group is 8 k: instruction j of a group takes k = j from lanes 0..31 and k = 4 + j from lanes 32..63, which is what
// the 16-byte read of a K-contiguous row delivers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_math.h"
#include "kernels.h"
#include "lds_dma.h"
#include "tile_order.h"

namespace tpl {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int FK = 32;                          // k per stage
constexpr unsigned F_OOB = 0x80000000u;         // past any operand this kernel takes (below 2 GiB)

template <int WM_, int WN_, int TM_, int TN_, int KW_, int STAGES_>
struct F32Tile {
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, KW = KW_, STAGES = STAGES_;
    static_assert(WM * WN * KW == 4, "four wavefronts");
    static constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    static constexpr int LA = BM / 32, LB = BN / 32;                     // direct loads per thread and stage
    static constexpr int A_BYTES = BM * FK * 4, STAGE_BYTES = (BM + BN) * FK * 4;
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES > (KW > 1 ? 16384 : 0) ? STAGES * STAGE_BYTES : 16384;
};

struct GemmF32Params {
    const float* A; const float* B; float* C;
    const float* bias; const float* resid; float* aux;
    int M, N, K, lda, ldb, epi;
    int tiles_m, tiles_n, nk, nk_total;         // nk: k-steps of one share
    float* partial;                             // [share][M][N], or null
    float* colsum;                              // [N]: sum over k of B[k][n] (weight gradients of a group), or null
    float* colsum_part;                         // with K shares: [share][N]
};
constexpr int F_CS_RUN = 16;                    // stages of a run of the column sums
constexpr int F_BAND = 8;                       // tile rows per band of the tile order

// LDS position (in 16-byte chunks) of the stage tile of an operand of R rows.  K contiguous: chunk c of row r at
// 8 r + (c ^ (r / 2 % 8)), so 16 rows read at one k lie on all banks.  M/N contiguous: row k holds R / 4 chunks; the two
// lane halves read rows k and k + 4, which are kept in different halves of the 256-byte bank line.
template <bool KMAJ, int R> __device__ __forceinline__ void f32_chunk_src(int p, int& row, int& chunk) {
    if (KMAJ) {
        row = p >> 3;
        chunk = (p & 7) ^ ((row >> 1) & 7);
    } else {
        constexpr int CPR = R / 4;
        const int pr = p / CPR, c = p % CPR;
        if (CPR >= 16) { row = pr; chunk = c ^ (((pr >> 2) & 1) << 3); }
        else { row = (pr & ~7) | ((pr & 1) << 2) | ((pr >> 1) & 3); chunk = c; }   // physical rows 2 j, 2 j + 1 = k j, j + 4
    }
}
template <bool KMAJ, int R> __device__ __forceinline__ int f32_mn_addr(int k, int mn) {   // byte address, M/N contiguous
    constexpr int CPR = R / 4;
    if (CPR >= 16) return k * (R * 4) + ((((mn >> 2) ^ (((k >> 2) & 1) << 3))) << 4) + (mn & 3) * 4;
    const int pr = (k & ~7) | ((k & 3) << 1) | ((k >> 2) & 1);
    return pr * (R * 4) + mn * 4;
}

// One output tile (and K share): number list_pos of the share-major list of the GEMM's workgroups.
template <typename T, bool A_KMAJ, bool B_KMAJ, bool COLSUM>
__device__ __forceinline__ void gemm_f32_tile(const GemmF32Params& p, int list_pos, char* smem) {
    static_assert(!COLSUM || !B_KMAJ, "column sums ride on the floats a lane reads of an N-contiguous B");
    constexpr int TM = T::TM, TN = T::TN, BM = T::BM, BN = T::BN, LA = T::LA, LB = T::LB, S = T::STAGES;
    const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wk = T::KW > 1 ? wave : 0, wm = T::KW > 1 ? 0 : wave / T::WN, wn = T::KW > 1 ? 0 : wave % T::WN;
    const int ntiles = p.tiles_m * p.tiles_n;
    const int share = list_pos / ntiles;
    int tm, tn;
    tile_coords(list_pos - share * ntiles, p.tiles_m, p.tiles_n, F_BAND, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int kt0 = share * p.nk;
    const int nk = p.nk_total - kt0 < p.nk ? p.nk_total - kt0 : p.nk;

    const i32x4 ra = make_rsrc(p.A, (unsigned)((int64_t)(A_KMAJ ? p.M : p.K) * p.lda * 4));
    const i32x4 rb = make_rsrc(p.B, (unsigned)((int64_t)(B_KMAJ ? p.N : p.K) * p.ldb * 4));
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    unsigned offa[LA], offb[LB];
    int ka[LA], kb[LB];                          // k of the chunk inside a stage (K contiguous), 0 otherwise
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        int r, c;
        f32_chunk_src<A_KMAJ, BM>(t + 256 * i, r, c);
        const bool ok = A_KMAJ ? m0 + r < p.M : m0 + 4 * c < p.M;
        offa[i] = ok ? (unsigned)(A_KMAJ ? ((int64_t)(m0 + r) * p.lda + 4 * c) * 4 : ((int64_t)r * p.lda + m0 + 4 * c) * 4) : F_OOB;
        ka[i] = A_KMAJ ? 4 * c : 0;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        int r, c;
        f32_chunk_src<B_KMAJ, BN>(t + 256 * i, r, c);
        const bool ok = B_KMAJ ? n0 + r < p.N : n0 + 4 * c < p.N;
        offb[i] = ok ? (unsigned)(B_KMAJ ? ((int64_t)(n0 + r) * p.ldb + 4 * c) * 4 : ((int64_t)r * p.ldb + n0 + 4 * c) * 4) : F_OOB;
        kb[i] = B_KMAJ ? 4 * c : 0;
    }
    const unsigned sa = A_KMAJ ? 4u : (unsigned)p.lda * 4u, sb = B_KMAJ ? 4u : (unsigned)p.ldb * 4u;   // bytes per k
    // Stages past the end of the share read through a descriptor of no records, so that the number of loads in flight
    // never changes.  Rows k >= K of an M/N-contiguous operand lie past its buffer; K-contiguous chunks past K are
    // checked (they would be the next row's).
    auto fetch = [&](int s) {
        const unsigned buf = lds0 + (unsigned)(s % S) * T::STAGE_BYTES + (unsigned)wave * 1024u;
        const int k0 = (kt0 + s) * FK;
        i32x4 r = ra;
        r[2] = __builtin_amdgcn_readfirstlane(s < nk ? ra[2] : 0);
#pragma unroll
        for (int i = 0; i < LA; ++i)
            buffer_load_lds_b128(r, buf + i * 4096, k0 + ka[i] < p.K ? offa[i] + (unsigned)k0 * sa : F_OOB);
        r = rb;
        r[2] = __builtin_amdgcn_readfirstlane(s < nk ? rb[2] : 0);
#pragma unroll
        for (int i = 0; i < LB; ++i)
            buffer_load_lds_b128(r, buf + T::A_BYTES + i * 4096, k0 + kb[i] < p.K ? offb[i] + (unsigned)k0 * sb : F_OOB);
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    auto frag = [&](float (&f)[4], const char* st, int mn, int g, auto kmaj, auto rows) {
        constexpr bool KM = decltype(kmaj)::value;
        constexpr int R = decltype(rows)::value;
        const int row = mn + (lane & 31);
        if (KM) {
            const int c = 2 * g + half;
            const float4 v = *reinterpret_cast<const float4*>(st + row * 128 + ((c ^ ((row >> 1) & 7)) << 4));
            f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = *reinterpret_cast<const float*>(st + f32_mn_addr<KM, R>(8 * g + 4 * half + j, row));
        }
    };
    // Column sums of B: the wavefronts of the first row of blocks in the first tile row hold every k of their columns once
    // (one half of each group of 8 per lane half).  A stage is summed by itself, F_CS_RUN stages by themselves, then the
    // runs.  Stage by stage into one sum lost 1.5 times what the column-sum kernels lose (relative error of a bias gradient
    // over 2048 tokens 1.7e-7, now 1.1e-7 as with those kernels; time of the step unchanged).
    const bool cs_on = COLSUM && p.colsum && tm == 0 && wm == 0;   // uniform over the wavefront
    float cs[TN], cs_run[TN], cs_stage[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) cs[j] = cs_run[j] = cs_stage[j] = 0.0f;
    auto group = [&](const char* st, int g) {                     // 8 k: TM TN x 4 matrix instructions
        float fa[TM][4], fb[TN][4];
#pragma unroll
        for (int i = 0; i < TM; ++i)
            frag(fa[i], st, (wm * TM + i) * 32, g, std::integral_constant<bool, A_KMAJ>{}, std::integral_constant<int, BM>{});
#pragma unroll
        for (int j = 0; j < TN; ++j)
            frag(fb[j], st + T::A_BYTES, (wn * TN + j) * 32, g, std::integral_constant<bool, B_KMAJ>{}, std::integral_constant<int, BN>{});
        if (COLSUM && cs_on) {
#pragma unroll
            for (int j = 0; j < TN; ++j) cs_stage[j] += (fb[j][0] + fb[j][1]) + (fb[j][2] + fb[j][3]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
    };

#pragma unroll
    for (int s = 0; s < S - 1; ++s) fetch(s);
    const int run = COLSUM ? F_CS_RUN : nk;
    for (int run0 = 0; run0 < nk; run0 += run) {
        const int run1 = run0 + run < nk ? run0 + run : nk;
        for (int kt = run0; kt < run1; ++kt) {
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"((S - 2) * (LA + LB)) : "memory");   // stage kt has landed (this wavefront's part)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                           // reads of stage kt - 1 are done
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            fetch(kt + S - 1);                                    // into the slot of stage kt - 1
            const char* st = smem + (kt % S) * T::STAGE_BYTES;
            if (T::KW > 1) {
                group(st, wk);
            } else {
#pragma unroll
                for (int g = 0; g < 4; ++g) group(st, g);
            }
            if (COLSUM && cs_on) {
#pragma unroll
                for (int j = 0; j < TN; ++j) { cs_run[j] += cs_stage[j]; cs_stage[j] = 0.0f; }
            }
        }
        if (COLSUM && cs_on) {
#pragma unroll
            for (int j = 0; j < TN; ++j) { cs[j] += cs_run[j]; cs_run[j] = 0.0f; }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // Epilogue straight from the accumulators: register v of a block is row 8 (v / 4) + 4 half + v % 4, column lane % 32,
    // so an access covers two rows of 128 bytes.  All reads of a block (residual, GeLU input) go out before the first is
    // used; rows and columns past the end read element 0 and are not stored.
    const bool split = p.partial != nullptr;
    auto emit = [&](int gn, auto count, auto row, auto value) {
        constexpr int NV = decltype(count)::value;
        const bool col = gn < p.N;
        if (split) {
            float* part = p.partial + (int64_t)share * p.M * p.N;
#pragma unroll
            for (int v = 0; v < NV; ++v)
                if (col && row(v) < p.M) part[(int64_t)row(v) * p.N + gn] = value(v);
            return;
        }
        auto at = [&](int v) { return col && row(v) < p.M ? (int64_t)row(v) * p.N + gn : (int64_t)0; };
        const float bias = p.bias ? p.bias[col ? gn : 0] : 0.0f;
        float r[NV], u[NV];
        if (p.resid) {
#pragma unroll
            for (int v = 0; v < NV; ++v) r[v] = p.resid[at(v)];
        }
        if (p.epi == EPI_DGELU) {
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = p.aux[at(v)];
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            float x = value(v) + bias;
            if (p.resid) x += r[v];
            const bool ok = col && row(v) < p.M;
            if (p.epi == EPI_GELU) {
                if (ok) p.aux[at(v)] = x;
                x = gelu_f(x);
            } else if (p.epi == EPI_DGELU) {
                x *= gelu_grad_f(u[v]);
            }
            if (ok) p.C[at(v)] = x;
        }
    };
    auto emit_colsum = [&](int gn, float s) {
        if (half == 0 && gn < p.N) (split ? p.colsum_part + (int64_t)share * p.N : p.colsum)[gn] = s;
    };
    if (T::KW > 1) {
        // four partial sums of one block: each wavefront adds the four, in wavefront order, for a quarter of the rows
        float* red = reinterpret_cast<float*>(smem);              // [wavefront][register][lane], then [wavefront][column]
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = acc[0][0][v];
        if (COLSUM && cs_on) red[4096 + wave * 64 + lane] = cs[0];
        __syncthreads();
        const int gn = n0 + (lane & 31);
        emit(gn, std::integral_constant<int, 4>{}, [&](int q) { return m0 + 8 * wave + 4 * half + q; }, [&](int q) {
            const int v = wave * 4 + q;
            return ((red[v * 64 + lane] + red[(16 + v) * 64 + lane]) + red[(32 + v) * 64 + lane]) + red[(48 + v) * 64 + lane];
        });
        if (COLSUM && cs_on && wave == 0) {
            float s = 0.0f;
#pragma unroll
            for (int w = 0; w < 4; ++w) s += red[4096 + w * 64 + (lane & 31)] + red[4096 + w * 64 + 32 + (lane & 31)];
            emit_colsum(gn, s);
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int gn = n0 + (wn * TN + j) * 32 + (lane & 31);
#pragma unroll
        for (int i = 0; i < TM; ++i)
            emit(gn, std::integral_constant<int, 16>{},
                 [&](int v) { return m0 + (wm * TM + i) * 32 + 8 * (v >> 2) + 4 * half + (v & 3); },
                 [&](int v) { return acc[i][j][v]; });
        if (COLSUM && cs_on) emit_colsum(gn, cs[j] + __shfl_xor(cs[j], 32, 64));
    }
}
template <typename T, bool A_KMAJ, bool B_KMAJ>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Params p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    gemm_f32_tile<T, A_KMAJ, B_KMAJ, false>(p, share_of_block(blockIdx.x, gridDim.x), smem);
}

// Independent GEMMs of a layer pass as one list of workgroups, as in gemm_bf16.hip: GEMM i is the workgroups
// [first[i], first[i+1]); the three layouts of a layer are three bodies of the kernel, the bias gradients ride in the
// weight gradients.  A launch of one of these GEMMs costs 4 to 6 us whatever it computes, and its last round leaves units
// idle.  Whole training steps, one launch per GEMM and bias gradient -> groups: 256 tokens of 256 / 128 109 -> 61 us, 260 of
// 768 / 384 203 -> 126, 2048 of 1024 / 256 499 -> 414 (floor 272 at 154 TFLOP/s), 4096 of 256 / 256 1219 -> 981, 700 of
// 1920 / 960 1051 -> 1048, 2000 of 2048 / 1024 2934 -> 2863: never behind, so float layers always go this way.
constexpr int F_GROUP_MAX = 4;
struct GroupF32Params {
    GemmF32Params g[F_GROUP_MAX];
    int first[F_GROUP_MAX + 1];
    int layout[F_GROUP_MAX];                    // 0: NN, 1: NT, 2: TN
    int shares[F_GROUP_MAX];
    int n;
};
template <typename T>
__global__ __launch_bounds__(256) void gemm_f32_group_kernel(GroupF32Params gp) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int bid = blockIdx.x;
    int i = 0;
    while (i + 1 < gp.n && bid >= gp.first[i + 1]) ++i;
    const GemmF32Params& p = gp.g[i];
    const int pos = share_of_block(bid - gp.first[i], gp.first[i + 1] - gp.first[i]);
    const int layout = gp.layout[i];
    if (layout == 0) gemm_f32_tile<T, true, false, false>(p, pos, smem);
    else if (layout == 1) gemm_f32_tile<T, true, true, false>(p, pos, smem);
    else gemm_f32_tile<T, false, false, true>(p, pos, smem);
}

// Sum of the K shares in share order, then the epilogue; 4 columns per thread.
__device__ __forceinline__ void f32_sum_shares(const GemmF32Params& p, int shares, int64_t idx) {
    const int64_t mn = (int64_t)p.M * p.N;
    float v[4] = {0, 0, 0, 0};
    auto add4 = [&](const float* q) {
        const float4 x = *reinterpret_cast<const float4*>(q);
        v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
    };
    for (int s = 0; s < shares; ++s) add4(p.partial + s * mn + idx);
    if (p.bias) add4(p.bias + idx % p.N);
    if (p.resid) add4(p.resid + idx);
    if (p.epi == EPI_GELU) {
        *reinterpret_cast<float4*>(p.aux + idx) = make_float4(v[0], v[1], v[2], v[3]);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu_f(v[e]);
    } else if (p.epi == EPI_DGELU) {
        const float4 u = *reinterpret_cast<const float4*>(p.aux + idx);
        v[0] *= gelu_grad_f(u.x); v[1] *= gelu_grad_f(u.y); v[2] *= gelu_grad_f(u.z); v[3] *= gelu_grad_f(u.w);
    }
    *reinterpret_cast<float4*>(p.C + idx) = make_float4(v[0], v[1], v[2], v[3]);
}
__global__ __launch_bounds__(256) void gemm_f32_sum_kernel(GemmF32Params p, int shares) {
    const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (idx < (int64_t)p.M * p.N) f32_sum_shares(p, shares, idx);
}
// The same for the GEMMs of a group that were cut: GEMM i has the workgroups [first[i], first[i+1]), the column sums last.
__global__ __launch_bounds__(256) void gemm_f32_group_sum_kernel(GroupF32Params gp) {
    const int bid = blockIdx.x;
    int i = 0;
    while (i + 1 < gp.n && bid >= gp.first[i + 1]) ++i;
    const GemmF32Params& p = gp.g[i];
    const int64_t idx = ((int64_t)(bid - gp.first[i]) * 256 + threadIdx.x) * 4, mn = (int64_t)p.M * p.N;
    if (idx < mn) { f32_sum_shares(p, gp.shares[i], idx); return; }
    const int64_t col = idx - mn;
    if (!p.colsum || col >= p.N) return;
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int s = 0; s < gp.shares[i]; ++s) {
        const float4 x = *reinterpret_cast<const float4*>(p.colsum_part + (int64_t)s * p.N + col);
        v.x += x.x; v.y += x.y; v.z += x.z; v.w += x.w;
    }
    *reinterpret_cast<float4*>(p.colsum + col) = v;
}

bool gemm_f32_supported(const GemmArgs& a) {
    if (a.dtype != F32 || a.N % 4 || (a.trans_a ? a.M : a.K) % 4 || (a.trans_b && a.K % 4)) return false;
    // 32-bit buffer offsets
    return a.M * a.K * 4 < 0x7FFFFFFFll && a.N * a.K * 4 < 0x7FFFFFFFll && ((a.M + 31) / 32) * ((a.N + 31) / 32) < (1 << 24) &&
           a.K < (1 << 24);
}

// Tile and K shares by a time estimate.  Compute units share a launch's workgroups evenly and the workgroups of one unit
// share its matrix pipes, so a launch takes (workgroups per unit, rounded up) x (matrix cycles of one) at least; one
// workgroup alone cannot run a k-step in less than its load latency over the loads in flight, and every launch has a
// fixed start and end.  Cutting K costs the partial sums' traffic and a second launch.
struct F32Plan { int variant, shares, nk; };
static F32Plan f32_plan(int64_t M, int64_t N, int64_t K) {
    static const int bm[3] = {128, 64, 32};
    static const double step_us[3] = {1.95, 0.49, 0.125};         // matrix cycles of a k-step
    static const double alone_us[3] = {2.2, 0.65, 0.45};          // a k-step of a workgroup that has its unit to itself
    const int cus = compute_units();
    const int nk = (int)((K + FK - 1) / FK);
    F32Plan best{0, 1, nk};
    double best_us = -1;
    for (int v = 0; v < 3; ++v) {
        const int64_t tiles = ((M + bm[v] - 1) / bm[v]) * ((N + bm[v] - 1) / bm[v]);
        for (int want = 1; want <= 16; want *= 2) {
            const int per = (nk + want - 1) / want, shares = (nk + per - 1) / per;
            if (want > 1 && (shares != want || per < 4 || tiles * (want / 2) >= 4 * cus)) continue;
            const int64_t wgs = tiles * shares;
            const double rounds = (double)((wgs + cus - 1) / cus);
            double us = std::max(rounds * step_us[v], alone_us[v]) * per + 3.0;
            if (shares > 1) us += 4.5 + (double)M * N * 8.0 * shares / 3.0e6;
            if (best_us < 0 || us < best_us) { best = F32Plan{v, shares, per}; best_us = us; }
        }
    }
    return best;
}

size_t gemm_f32_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    const F32Plan pl = f32_plan(M, N, K);
    return pl.shares > 1 ? (size_t)pl.shares * (size_t)M * (size_t)N * sizeof(float) : 0;
}

template <typename T, bool AK, bool BK>
static hipError_t launch_f32(GemmF32Params p, int shares, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32_kernel<T, AK, BK>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    p.tiles_m = (p.M + T::BM - 1) / T::BM;
    p.tiles_n = (p.N + T::BN - 1) / T::BN;
    hipLaunchKernelGGL((gemm_f32_kernel<T, AK, BK>), dim3((unsigned)(p.tiles_m * p.tiles_n * shares)), dim3(256), T::LDS_BYTES, s, p);
    return hipGetLastError();
}
template <typename T>
static hipError_t launch_f32_layout(const GemmF32Params& p, const GemmArgs& a, int shares) {
    if (!a.trans_a) return a.trans_b ? launch_f32<T, true, true>(p, shares, a.stream) : launch_f32<T, true, false>(p, shares, a.stream);
    return a.trans_b ? launch_f32<T, false, true>(p, shares, a.stream) : launch_f32<T, false, false>(p, shares, a.stream);
}

static GemmF32Params f32_params(const GemmArgs& a) {
    GemmF32Params p{};
    p.A = (const float*)a.A; p.B = (const float*)a.B; p.C = (float*)a.C;
    p.bias = (const float*)a.bias; p.resid = (const float*)a.resid; p.aux = (float*)a.aux;
    p.M = (int)a.M; p.N = (int)a.N; p.K = (int)a.K; p.epi = a.epi;
    p.lda = a.trans_a ? p.M : p.K;
    p.ldb = a.trans_b ? p.K : p.N;
    p.nk_total = (p.K + FK - 1) / FK;
    return p;
}

hipError_t gemm_f32(const GemmArgs& a) {
    GemmF32Params p = f32_params(a);
    const F32Plan pl = f32_plan(a.M, a.N, a.K);
    p.nk = pl.nk;
    if (pl.shares > 1) {
        if (!a.ws || a.ws_bytes < (size_t)pl.shares * (size_t)a.M * (size_t)a.N * sizeof(float)) return hipErrorInvalidValue;
        p.partial = (float*)a.ws;
    }
    hipError_t e;
    switch (pl.variant) {
        case 0: e = launch_f32_layout<F32Tile<2, 2, 2, 2, 1, 2>>(p, a, pl.shares); break;
        case 1: e = launch_f32_layout<F32Tile<2, 2, 1, 1, 1, 3>>(p, a, pl.shares); break;
        default: e = launch_f32_layout<F32Tile<1, 1, 1, 1, 4, 4>>(p, a, pl.shares); break;
    }
    if (e != hipSuccess || pl.shares == 1) return e;
    hipLaunchKernelGGL(gemm_f32_sum_kernel, dim3((unsigned)((a.M * a.N / 4 + 255) / 256)), dim3(256), 0, a.stream, p, pl.shares);
    return hipGetLastError();
}

// ---- groups ----------------------------------------------------------------------------------------------------------
// One tile for the whole group and K shares per GEMM by a time estimate: the units' work evenly spread, plus half of the
// longest workgroup for the end of the launch, or the longest workgroup by itself, whichever is more.
// On 10 layers (17 to 4096 tokens, 256 to 2048 wide) the tile it takes is the best of the three or within 5 % of it: 32 at
// 256 tokens of 256 / 128 (61 us; 75 and 107 on 64 and 128), 64 at 2048 of 1024 / 256 (414; 446 on 32, 518 on 128).
using F32Tile128 = F32Tile<2, 2, 2, 2, 1, 2>;
using F32Tile64 = F32Tile<2, 2, 1, 1, 1, 3>;
using F32Tile32 = F32Tile<1, 1, 1, 1, 4, 4>;
// The 64-wide tile with two stages instead of three: four workgroups share a unit instead of three (32 KB of LDS instead of 48), so that with
// at least six to a unit one's start, barriers and epilogue have three others beside them.  Whole steps, us, three stages and two: 4115 tokens
// of 1024 / 512 1662 and 1613, 3260 of 768 / 384 725 and 687, 6349 of 512 / 64 266.9 and 262.2, 1136 of 1792 / 1792 2315 and 2242; with fewer
// the last of a unit runs at a lone workgroup's pace on half the loads: 3563 of 448 / 224 (3.1 to 5.5 to a unit) 363 and 368 on two stages.  Launches of
// 6 to 6.5 to a unit: 33 without weight gradients 3 to 9 % faster on two stages; of 53 with them, long beside short, 42 up to 9 % faster and 11 up to
// 3.7 % slower, as the last workgroups of a unit happen to fall (2700 tokens of 1024 / 128 314.6 and 317.1 a step); from 6.5 on, one of 61
// launches 2.9 % slower, the others 0.3 % slower to 9.6 % faster.
using F32Tile64Four = F32Tile<2, 2, 1, 1, 1, 2>;
constexpr int F32_FOUR_MIN = 6;                 // workgroups per unit
namespace {
struct F32GroupTile { int bm; double step_us, wg_us, alone_us; };
constexpr F32GroupTile F32_GROUP_TILES[] = {{128, 1.95, 3.0, 2.2}, {64, 0.50, 1.0, 0.65}, {32, 0.15, 0.5, 0.45}};
struct F32GroupPlan { int tile, nk[F_GROUP_MAX], shares[F_GROUP_MAX]; double us; };

F32GroupPlan plan_f32_group(const GemmArgs* g, int n) {
    const int cus = compute_units(), forced = options().gemm_group >= 256 ? -1 : options().gemm_group;   // 256, 384, 512: bf16 tiles
    F32GroupPlan best{};
    best.us = -1;
    for (int t = 0; t < 3; ++t) {
        const F32GroupTile& gt = F32_GROUP_TILES[t];
        if (forced > 0 && gt.bm != (forced == 192 ? 32 : forced)) continue;
        F32GroupPlan p{};
        p.tile = t;
        int64_t tiles[F_GROUP_MAX];
        int nk[F_GROUP_MAX];
        for (int i = 0; i < n; ++i) {
            tiles[i] = ((g[i].M + gt.bm - 1) / gt.bm) * ((g[i].N + gt.bm - 1) / gt.bm);
            nk[i] = p.nk[i] = (int)((g[i].K + FK - 1) / FK);
            p.shares[i] = 1;
        }
        auto estimate = [&]() {
            double work = 0, longest = 0, bytes = 0;
            for (int i = 0; i < n; ++i) {
                work += (double)tiles[i] * p.shares[i] * (p.nk[i] * gt.step_us + gt.wg_us);
                longest = std::max(longest, (double)p.nk[i]);
                if (p.shares[i] > 1) bytes += (double)g[i].M * g[i].N * (8.0 * p.shares[i] + 4.0);
            }
            return std::max(work / cus + 0.5 * longest * gt.step_us, longest * gt.alone_us) + 4.0 +
                   (bytes > 0 ? 4.5 + bytes / 3.0e6 : 0.0);
        };
        p.us = estimate();
        for (int cuts = 0; cuts < 32; ++cuts) {                   // cut the longest again while that helps
            int l = 0;
            for (int i = 1; i < n; ++i) if (p.nk[i] > p.nk[l]) l = i;
            const int want = p.shares[l] + 1;
            if (want > 16 || nk[l] / want < 4) break;
            const F32GroupPlan before = p;
            p.nk[l] = (nk[l] + want - 1) / want;
            p.shares[l] = (nk[l] + p.nk[l] - 1) / p.nk[l];
            p.us = estimate();
            if (best.us < 0 || before.us < best.us) best = before;
        }
        if (best.us < 0 || p.us < best.us) best = p;
    }
    return best;
}
size_t f32_share_bytes(const GemmArgs& a, int shares) {           // partial sums, column sums included
    return shares > 1 ? (size_t)shares * ((size_t)a.M * a.N + (size_t)a.N) * sizeof(float) : 0;
}
}  // namespace

size_t gemm_f32_group_workspace_bytes(const GemmArgs* g, int n) {
    const F32GroupPlan pl = plan_f32_group(g, n);
    size_t need = 0;
    for (int i = 0; i < n; ++i) need += f32_share_bytes(g[i], pl.shares[i]);
    return need;
}

template <typename T>
static hipError_t launch_f32_group(const GroupF32Params& gp, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32_group_kernel<T>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(gemm_f32_group_kernel<T>, dim3((unsigned)gp.first[gp.n]), dim3(256), T::LDS_BYTES, s, gp);
    return hipGetLastError();
}

hipError_t gemm_f32_group(const GemmArgs* g, int n, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n < 1 || n > F_GROUP_MAX) return hipErrorInvalidValue;
    const F32GroupPlan pl = plan_f32_group(g, n);
    const int bm = F32_GROUP_TILES[pl.tile].bm;
    int order[F_GROUP_MAX] = {0, 1, 2, 3};
    std::stable_sort(order, order + n, [&](int a, int b) { return pl.nk[a] > pl.nk[b]; });
    GroupF32Params gp{}, sp{};                                    // the GEMMs; the sums of those that were cut
    gp.n = n;
    char* part = static_cast<char*>(ws);
    size_t used = 0;
    for (int q = 0; q < n; ++q) {
        const GemmArgs& a = g[order[q]];
        const int shares = pl.shares[order[q]];
        GemmF32Params p = f32_params(a);
        p.nk = pl.nk[order[q]];
        p.tiles_m = (int)((a.M + bm - 1) / bm);
        p.tiles_n = (int)((a.N + bm - 1) / bm);
        p.colsum = a.trans_a ? (float*)a.colsum_b : nullptr;
        if (shares > 1) {
            const size_t bytes = f32_share_bytes(a, shares);
            if (!ws || used + bytes > ws_bytes) return hipErrorInvalidValue;
            p.partial = reinterpret_cast<float*>(part + used);
            p.colsum_part = p.partial + (size_t)shares * a.M * a.N;
            used += bytes;
            sp.g[sp.n] = p;
            sp.shares[sp.n] = shares;
            const int64_t outs = a.M * a.N + (p.colsum ? a.N : 0);
            sp.first[sp.n + 1] = sp.first[sp.n] + (int)((outs + 1023) / 1024);
            ++sp.n;
        }
        gp.g[q] = p;
        gp.shares[q] = shares;
        gp.layout[q] = a.trans_a ? 2 : a.trans_b ? 1 : 0;
        gp.first[q + 1] = gp.first[q] + p.tiles_m * p.tiles_n * shares;
    }
    hipError_t e = pl.tile == 0   ? launch_f32_group<F32Tile128>(gp, stream)
                   : pl.tile == 1 ? (gp.first[n] >= F32_FOUR_MIN * compute_units() ? launch_f32_group<F32Tile64Four>(gp, stream) : launch_f32_group<F32Tile64>(gp, stream))
                                  : launch_f32_group<F32Tile32>(gp, stream);
    if (e != hipSuccess || sp.n == 0) return e;
    hipLaunchKernelGGL(gemm_f32_group_sum_kernel, dim3((unsigned)sp.first[sp.n]), dim3(256), 0, stream, sp);
    return hipGetLastError();
}

}  // namespace tpl

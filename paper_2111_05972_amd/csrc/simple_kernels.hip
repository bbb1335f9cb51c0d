// Generic kernels: any shape, float or bfloat16 storage, float accumulation.
// They cover the shapes the MFMA kernels do not take (head sizes above 128, operands of 2 GiB and more).
#include <hip/hip_runtime.h>

#include <mutex>

#include "attn_rows.h"
#include "device_math.h"
#include "kernels.h"

namespace tpl {

// ------------------------------------------------------------------------------------------------
// GEMM: 64x64 output tile per 256-thread block, 4x4 outputs per thread, operands addressed through
// (row, column) strides so all four transpose combinations share one kernel.
// ------------------------------------------------------------------------------------------------
constexpr int SG_BM = 64, SG_BN = 64, SG_BK = 16;

template <typename T>
__global__ __launch_bounds__(256) void gemm_simple_kernel(
    int64_t M, int64_t N, int64_t K, const T* __restrict__ A, int64_t a_rs, int64_t a_cs,
    const T* __restrict__ B, int64_t b_rs, int64_t b_cs, T* __restrict__ C,
    const T* __restrict__ bias, const T* __restrict__ resid, T* __restrict__ aux, int epi) {
    __shared__ float As[SG_BK][SG_BM + 1];
    __shared__ float Bs[SG_BK][SG_BN + 1];
    const int t = threadIdx.x;
    const int64_t m0 = (int64_t)blockIdx.y * SG_BM, n0 = (int64_t)blockIdx.x * SG_BN;
    const int tm = (t / 16) * 4, tn = (t % 16) * 4;
    float acc[4][4] = {};
    for (int64_t k0 = 0; k0 < K; k0 += SG_BK) {
        for (int i = 0; i < 4; ++i) {
            int mm, kk;
            if (a_cs == 1) { kk = t % SG_BK; mm = t / SG_BK + 16 * i; }
            else           { mm = t % SG_BM; kk = t / SG_BM + 4 * i; }
            int64_t gm = m0 + mm, gk = k0 + kk;
            As[kk][mm] = (gm < M && gk < K) ? to_f32(A[gm * a_rs + gk * a_cs]) : 0.0f;
            int nn, kb;
            if (b_rs == 1) { kb = t % SG_BK; nn = t / SG_BK + 16 * i; }
            else           { nn = t % SG_BN; kb = t / SG_BN + 4 * i; }
            int64_t gn = n0 + nn, gkb = k0 + kb;
            Bs[kb][nn] = (gn < N && gkb < K) ? to_f32(B[gkb * b_rs + gn * b_cs]) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < SG_BK; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = As[kk][tm + i]; b[i] = Bs[kk][tn + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    for (int i = 0; i < 4; ++i) {
        int64_t gm = m0 + tm + i;
        if (gm >= M) continue;
        for (int j = 0; j < 4; ++j) {
            int64_t gn = n0 + tn + j;
            if (gn >= N) continue;
            float v = acc[i][j];
            if (bias) v += to_f32(bias[gn]);
            if (resid) v += to_f32(resid[gm * N + gn]);
            if (epi == EPI_GELU) {
                aux[gm * N + gn] = from_f32<T>(v);
                v = gelu_f(v);
            } else if (epi == EPI_DGELU) {
                v *= gelu_grad_f(to_f32(aux[gm * N + gn]));
            }
            C[gm * N + gn] = from_f32<T>(v);
        }
    }
}

template <typename T>
static hipError_t gemm_simple_t(const GemmArgs& a) {
    dim3 grid((unsigned)((a.N + SG_BN - 1) / SG_BN), (unsigned)((a.M + SG_BM - 1) / SG_BM));
    int64_t a_rs = a.trans_a ? 1 : a.K, a_cs = a.trans_a ? a.M : 1;   // A(m,k)
    int64_t b_rs = a.trans_b ? 1 : a.N, b_cs = a.trans_b ? a.K : 1;   // B(k,n)
    hipLaunchKernelGGL(gemm_simple_kernel<T>, grid, dim3(256), 0, a.stream, a.M, a.N, a.K,
                       (const T*)a.A, a_rs, a_cs, (const T*)a.B, b_rs, b_cs, (T*)a.C,
                       (const T*)a.bias, (const T*)a.resid, (T*)a.aux, a.epi);
    return hipGetLastError();
}

hipError_t gemm_simple(const GemmArgs& a) {
    return a.dtype == F32 ? gemm_simple_t<float>(a) : gemm_simple_t<bf16_t>(a);
}

// ------------------------------------------------------------------------------------------------
// Attention, one wavefront per query row (forward, dQ) or per key row (dK, dV).
// qkv is [B*S, 3*nl*dh] with columns (q|k|v, head, dh); the arithmetic of a row is in attn_rows.h.
// ------------------------------------------------------------------------------------------------
constexpr int AT_WAVES = 4;
constexpr int AT_MAXDH = 256;

template <typename T>
__global__ __launch_bounds__(64 * AT_WAVES) void attn_simple_fwd_kernel(
    int B, int S, int nl, int dh, int causal, const T* __restrict__ qkv, T* __restrict__ o,
    float* __restrict__ lse) {
    __shared__ float q_s[AT_WAVES][AT_MAXDH];
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int i_raw = blockIdx.x * AT_WAVES + w;
    const bool valid = i_raw < S;          // a tail wavefront recomputes the last row and stores nothing
    const int i = valid ? i_raw : S - 1;
    const int b = blockIdx.y / nl, h = blockIdx.y % nl;
    const int64_t ld = 3LL * nl * dh;
    const T* qp = qkv + ((int64_t)b * S + i) * ld + (int64_t)h * dh;
    const T* kbase = qkv + (int64_t)b * S * ld + (int64_t)nl * dh + (int64_t)h * dh;
    const T* vbase = kbase + (int64_t)nl * dh;
    load_row(q_s[w], qp, dh, lane);
    __syncthreads();
    float m, l;
    T* op = o + ((int64_t)b * S + i) * ((int64_t)nl * dh) + (int64_t)h * dh;
    attn_row_fwd<AT_MAXDH / 64>(q_s[w], kbase, vbase, ld, dh, 0, causal ? i + 1 : S, 1.0f / sqrtf((float)dh), true, lane, m, l,
                                [&](int d, float v) { if (valid) op[d] = from_f32<T>(v); });
    if (valid && lane == 0) lse[((int64_t)b * nl + h) * S + i] = m + logf(l);
}

// dQ_i = sum_j dS_ij K_j / sqrt(dh), dS_ij = P_ij (dO_i.V_j - D_i), D_i = dO_i.O_i; also stores D.
template <typename T>
__global__ __launch_bounds__(64 * AT_WAVES) void attn_simple_dq_kernel(
    int B, int S, int nl, int dh, int causal, const T* __restrict__ qkv, const T* __restrict__ o,
    const float* __restrict__ lse, const T* __restrict__ d_o, T* __restrict__ dqkv,
    float* __restrict__ dsum) {
    __shared__ float q_s[AT_WAVES][AT_MAXDH];
    __shared__ float do_s[AT_WAVES][AT_MAXDH];
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int i_raw = blockIdx.x * AT_WAVES + w;
    const bool valid = i_raw < S;
    const int i = valid ? i_raw : S - 1;
    const int b = blockIdx.y / nl, h = blockIdx.y % nl;
    const int64_t ld = 3LL * nl * dh, ldo = (int64_t)nl * dh;
    const T* qp = qkv + ((int64_t)b * S + i) * ld + (int64_t)h * dh;
    const T* kbase = qkv + (int64_t)b * S * ld + (int64_t)nl * dh + (int64_t)h * dh;
    const T* vbase = kbase + (int64_t)nl * dh;
    const T* dop = d_o + ((int64_t)b * S + i) * ldo + (int64_t)h * dh;
    const T* op = o + ((int64_t)b * S + i) * ldo + (int64_t)h * dh;
    float dpart = 0.0f;
    for (int d = lane; d < dh; d += 64) {
        float g = to_f32(dop[d]);
        q_s[w][d] = to_f32(qp[d]);
        do_s[w][d] = g;
        dpart = fmaf(g, to_f32(op[d]), dpart);
    }
    const float Di = row_sum(dpart);
    __syncthreads();
    const float scale = 1.0f / sqrtf((float)dh);
    T* dqp = dqkv + ((int64_t)b * S + i) * ld + (int64_t)h * dh;
    attn_row_dq<AT_MAXDH / 64>(q_s[w], do_s[w], kbase, vbase, ld, dh, 0, causal ? i + 1 : S, scale, lse[((int64_t)b * nl + h) * S + i], Di,
                               lane, [&](int d, float v) { if (valid) dqp[d] = from_f32<T>(v * scale); });
    if (valid && lane == 0) dsum[((int64_t)b * nl + h) * S + i] = Di;
}

// dK_j = sum_i dS_ij Q_i / sqrt(dh), dV_j = sum_i P_ij dO_i.
template <typename T>
__global__ __launch_bounds__(64 * AT_WAVES) void attn_simple_dkv_kernel(
    int B, int S, int nl, int dh, int causal, const T* __restrict__ qkv,
    const float* __restrict__ lse, const T* __restrict__ d_o, T* __restrict__ dqkv,
    const float* __restrict__ dsum) {
    __shared__ float k_s[AT_WAVES][AT_MAXDH];
    __shared__ float v_s[AT_WAVES][AT_MAXDH];
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int j_raw = blockIdx.x * AT_WAVES + w;
    const bool valid = j_raw < S;
    const int j = valid ? j_raw : S - 1;
    const int b = blockIdx.y / nl, h = blockIdx.y % nl;
    const int64_t ld = 3LL * nl * dh, ldo = (int64_t)nl * dh;
    const T* qbase = qkv + (int64_t)b * S * ld + (int64_t)h * dh;
    const T* kp = qbase + (int64_t)j * ld + (int64_t)nl * dh;
    const T* vp = kp + (int64_t)nl * dh;
    const T* dobase = d_o + (int64_t)b * S * ldo + (int64_t)h * dh;
    load_row(k_s[w], kp, dh, lane);
    load_row(v_s[w], vp, dh, lane);
    __syncthreads();
    const float scale = 1.0f / sqrtf((float)dh);
    T* dkp = dqkv + ((int64_t)b * S + j) * ld + (int64_t)nl * dh + (int64_t)h * dh;
    T* dvp = dkp + (int64_t)nl * dh;
    const float* drow = dsum + ((int64_t)b * nl + h) * S;
    attn_row_dkv<AT_MAXDH / 64>(k_s[w], v_s[w], qbase, ld, dobase, ldo, lse + ((int64_t)b * nl + h) * S, [&](int i) { return drow[i]; }, dh,
                                causal ? j : 0, S, scale, lane, [&](int d, float dk, float dv) {
                                    if (valid) { dkp[d] = from_f32<T>(dk * scale); dvp[d] = from_f32<T>(dv); }
                                });
}

template <typename T>
static hipError_t attn_fwd_t(const AttnArgs& a) {
    dim3 grid((a.S + AT_WAVES - 1) / AT_WAVES, a.B * a.nl);
    hipLaunchKernelGGL(attn_simple_fwd_kernel<T>, grid, dim3(64 * AT_WAVES), 0, a.stream, a.B, a.S,
                       a.nl, a.dh, a.causal, (const T*)a.qkv, (T*)a.o, a.lse);
    return hipGetLastError();
}
template <typename T>
static hipError_t attn_bwd_t(const AttnArgs& a) {
    dim3 grid((a.S + AT_WAVES - 1) / AT_WAVES, a.B * a.nl);
    hipLaunchKernelGGL(attn_simple_dq_kernel<T>, grid, dim3(64 * AT_WAVES), 0, a.stream, a.B, a.S,
                       a.nl, a.dh, a.causal, (const T*)a.qkv, (const T*)a.o, a.lse,
                       (const T*)a.d_o, (T*)a.dqkv, a.dsum);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_simple_dkv_kernel<T>, grid, dim3(64 * AT_WAVES), 0, a.stream, a.B, a.S,
                       a.nl, a.dh, a.causal, (const T*)a.qkv, a.lse, (const T*)a.d_o, (T*)a.dqkv,
                       a.dsum);
    return hipGetLastError();
}

hipError_t attn_simple_fwd(const AttnArgs& a) {
    return a.dtype == F32 ? attn_fwd_t<float>(a) : attn_fwd_t<bf16_t>(a);
}
hipError_t attn_simple_bwd(const AttnArgs& a) {
    return a.dtype == F32 ? attn_bwd_t<float>(a) : attn_bwd_t<bf16_t>(a);
}

// ------------------------------------------------------------------------------------------------
// Column sums (bias gradients): out[n] = sum_m X[m,n].  HBM-bound: X is read once with 16-byte loads.
// Two fixed-order stages so results do not depend on scheduling: a block sums a slab of CS_ROWS rows
// for 512 columns (64 column groups of 8 x 4 row lanes, combined through LDS in lane order) into
// scratch[slab][n]; then the slabs of a column are added in a fixed order (four interleaved lanes).
// ------------------------------------------------------------------------------------------------
constexpr int CS_ROWS = 64;

template <typename T>
__global__ __launch_bounds__(256) void colsum_stage1(int64_t M, int64_t N, const T* __restrict__ X,
                                                     float* __restrict__ part) {
    __shared__ float red[4][64][8];
    const int cg = threadIdx.x & 63, rl = threadIdx.x >> 6;
    const int64_t n = ((int64_t)blockIdx.x * 64 + cg) * 8;
    const int64_t m0 = (int64_t)blockIdx.y * CS_ROWS, m1 = m0 + CS_ROWS < M ? m0 + CS_ROWS : M;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int cnt = n + 8 <= N ? 8 : (n < N ? (int)(N - n) : 0);     // columns this thread owns
    if (cnt == 8) {
        int64_t m = m0 + rl;
        for (; m + 12 < m1; m += 16) {                               // four rows in flight, added in row order
            float v[4][8];
#pragma unroll
            for (int r = 0; r < 4; ++r) load8(X + (m + 4 * r) * N + n, v[r]);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] += v[r][e];
        }
        for (; m < m1; m += 4) {
            float v[8];
            load8(X + m * N + n, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += v[e];
        }
    } else if (cnt > 0) {                                            // ragged tail of a float matrix
        for (int64_t m = m0 + rl; m < m1; m += 4)
            for (int e = 0; e < cnt; ++e) acc[e] += to_f32(X[m * N + n + e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[rl][cg][e] = acc[e];
    __syncthreads();
    if (rl == 0) {
        float* dst = part + (int64_t)blockIdx.y * N + n;
        for (int e = 0; e < cnt; ++e) dst[e] = ((red[0][cg][e] + red[1][cg][e]) + red[2][cg][e]) + red[3][cg][e];
    }
}
// 64 columns x 4 slab lanes per workgroup: lane g adds slabs g, g+4, ... in order (four loads in flight), the four
// lanes are combined through LDS in lane order.
template <typename T>
__global__ __launch_bounds__(256) void colsum_stage2(int64_t slabs, int64_t N, const float* __restrict__ part,
                                                     T* __restrict__ out) {
    __shared__ float red[4][64];
    const int cl = threadIdx.x & 63, gl = threadIdx.x >> 6;
    const int64_t n = (int64_t)blockIdx.x * 64 + cl;
    float s = 0.0f;
    if (n < N) {
        const float* src = part + n;
        int64_t i = gl;
        for (; i + 12 < slabs; i += 16) {
            const float a = src[i * N], b = src[(i + 4) * N], c = src[(i + 8) * N],
                        d = src[(i + 12) * N];
            s += a; s += b; s += c; s += d;
        }
        for (; i < slabs; i += 4) s += src[i * N];
    }
    red[gl][cl] = s;
    __syncthreads();
    if (gl == 0 && n < N) out[n] = from_f32<T>(((red[0][cl] + red[1][cl]) + red[2][cl]) + red[3][cl]);
}

// Both stages in one launch where a matrix is small: a workgroup sums 32 columns over all rows, four threads a row, 128 rows at a time; a thread
// adds its rows one after another, with eight of them requested at once only where it has eight (from 897 rows on).  The 128 row lanes are combined
// through LDS in a fixed tree.  What bounds such a launch is its start and end, two to three us whatever it computes, and what a unit reads by
// itself: up to 1024 rows and 8 MB.  Back to back, matrix in cache, us, both stages and this: 100 x 1024 5.2 and 3.3, 512 x 3840 5.5 and 3.8,
// 1024 x 3840 5.6 and 4.0, but 1280 x 8192 (21 MB) 6.1 and 9.1; local compute of a rank with five such sums: 72 tokens of 1024 / 4 147.4 and 139.8, 520 of
// 5120 / 8 383 and 375, 832 of 640 / 2 209.9 and 205.0.  The line is on the safe side: beyond it 1376 of 512 / 8 200.2 and 195.2, 1560 of 1024 / 8 230.7
// and 227.0, 2048 of 1024 / 4 265.5 and 264.4, 2048 of 5120 / 4 1149 and 1152, 3384 of 1024 / 8 283.5 and 287.3, 3912 of 256 / 4 235.0 and 240.3.
constexpr int CO_COLS = 32, CO_ROWS = 128;
template <typename T>
__global__ __launch_bounds__(512) void colsum_once(int64_t M, int64_t N, const T* __restrict__ X, T* __restrict__ out) {
    __shared__ float red[CO_ROWS / 2][CO_COLS + 1];
    const int cg = threadIdx.x & 3, rl = threadIdx.x >> 2;
    const int64_t n = (int64_t)blockIdx.x * CO_COLS + cg * 8;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (n < N) {                                                     // N is a multiple of 8
        int64_t m = rl;
        for (; m + 7 * CO_ROWS < M; m += 8 * CO_ROWS) {
            float v[8][8];
#pragma unroll
            for (int r = 0; r < 8; ++r) load8(X + (m + r * CO_ROWS) * N + n, v[r]);
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] += v[r][e];
        }
        for (; m < M; m += CO_ROWS) {
            float v[8];
            load8(X + m * N + n, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += v[e];
        }
    }
    for (int half = CO_ROWS / 2; half > 0; half >>= 1) {             // lanes [half, 2 half) hand over to [0, half)
        if (rl >= half && rl < 2 * half)
#pragma unroll
            for (int e = 0; e < 8; ++e) red[rl - half][cg * 8 + e] = acc[e];
        __syncthreads();
        if (rl < half)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += red[rl][cg * 8 + e];
        __syncthreads();
    }
    if (rl == 0 && n < N)
#pragma unroll
        for (int e = 0; e < 8; ++e) out[n + e] = from_f32<T>(acc[e]);
}
constexpr int64_t CO_MAX_ROWS = 1024, CO_MAX_BYTES = 8 << 20;

size_t colsum_scratch_bytes(int64_t M, int64_t N) {
    return (size_t)((M + CS_ROWS - 1) / CS_ROWS) * (size_t)N * sizeof(float);
}

// Scratch for the entry points that may not allocate: one array per GPU, held until the process ends.  In host
// code the array's name is only a handle; its device address is looked up once per device (with that device
// current) and that pointer is what every launch and copy uses.
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

hipError_t static_scratch(void** ptr) {
    constexpr int MAX_DEV = 64;
    static void* per_device[MAX_DEV] = {};
    static std::mutex mu;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEV) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!per_device[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        per_device[dev] = p;
    }
    *ptr = per_device[dev];
    return hipSuccess;
}

hipError_t colsum(int dtype, int64_t M, int64_t N, const void* X, void* out, float* scratch,
                  hipStream_t s) {
    if (N % 8 == 0 && M <= CO_MAX_ROWS && M * N * (dtype == F32 ? 4 : 2) <= CO_MAX_BYTES) {
        const dim3 grid((unsigned)((N + CO_COLS - 1) / CO_COLS));
        if (dtype == F32) hipLaunchKernelGGL(colsum_once<float>, grid, dim3(512), 0, s, M, N, (const float*)X, (float*)out);
        else hipLaunchKernelGGL(colsum_once<bf16_t>, grid, dim3(512), 0, s, M, N, (const bf16_t*)X, (bf16_t*)out);
        return hipGetLastError();
    }
    int64_t slabs = (M + CS_ROWS - 1) / CS_ROWS;
    dim3 g1((unsigned)((N + 511) / 512), (unsigned)slabs), g2((unsigned)((N + 63) / 64));
    if (dtype == F32) {
        hipLaunchKernelGGL(colsum_stage1<float>, g1, dim3(256), 0, s, M, N, (const float*)X, scratch);
        hipLaunchKernelGGL(colsum_stage2<float>, g2, dim3(256), 0, s, slabs, N, scratch, (float*)out);
    } else {
        hipLaunchKernelGGL(colsum_stage1<bf16_t>, g1, dim3(256), 0, s, M, N, (const bf16_t*)X, scratch);
        hipLaunchKernelGGL(colsum_stage2<bf16_t>, g2, dim3(256), 0, s, slabs, N, scratch, (bf16_t*)out);
    }
    return hipGetLastError();
}

}  // namespace tpl

// Softmax attention row by row, one wavefront per row on vector arithmetic: any head size up to 64 NA, any range of the other
// side, and a row that the mask leaves out is not read.  The generic kernels are made of these; the matrix-core kernels come
// here for rows whose diagonal tile holds an infinity or a NaN, where a masked weight of zero times that row would be NaN.
//
// The other side is visited 64 rows at a time: lane j owns row j0 + j for the dot products, then lane d owns output column
// d (and d + 64, ...) for the weighted sums, with the weights passed across lanes by shuffles.
#pragma once
#include <hip/hip_runtime.h>

#include "device_math.h"

namespace tpl {

__device__ __forceinline__ float row_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float row_sum(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
template <typename T> __device__ __forceinline__ void load_row(float* dst, const T* src, int dh, int lane) {
    for (int d = lane; d < dh; d += 64) dst[d] = to_f32(src[d]);
}
// What this wavefront has written to LDS may be read by its other lanes.
__device__ __forceinline__ void row_loaded() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// What this wavefront has stored so far is in memory: its next stores to the same places come after it.
__device__ __forceinline__ void rows_stored() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Forward over keys [jbeg, jend): row maximum m and sum l of the scaled scores' exponentials, and store(d, O[d]), divided by
// l if normalise.  q_s: the query in LDS.
template <int NA, typename T, typename Store>
__device__ __forceinline__ void attn_row_fwd(const float* q_s, const T* kbase, const T* vbase, int64_t ld, int dh, int jbeg, int jend,
                                             float scale, bool normalise, int lane, float& m, float& l, Store store) {
    // pass 1: row maximum and sum of exponentials
    float mx = -INFINITY, sum = 0.0f;
    for (int j0 = jbeg; j0 < jend; j0 += 64) {
        int j = j0 + lane;
        if (j < jend) {
            const T* kp = kbase + (int64_t)j * ld;
            float s = 0.0f;
            for (int d = 0; d < dh; ++d) s = fmaf(q_s[d], to_f32(kp[d]), s);
            s *= scale;
            float nm = fmaxf(mx, s), mu = nm == -INFINITY ? 0.0f : nm;      // a NaN score makes the sum NaN, one of -inf adds 0
            sum = sum * expf(mx - mu) + expf(s - mu);
            mx = nm;
        }
    }
    m = row_max(mx);
    const float mu = m == -INFINITY ? 0.0f : m;
    l = row_sum(sum * expf(mx - mu));
    const float inv = normalise ? 1.0f / l : 1.0f;
    // pass 2: O = sum_j p_j V_j
    float acc[NA] = {};
    for (int j0 = jbeg; j0 < jend; j0 += 64) {
        int j = j0 + lane;
        float p = 0.0f;
        if (j < jend) {
            const T* kp = kbase + (int64_t)j * ld;
            float s = 0.0f;
            for (int d = 0; d < dh; ++d) s = fmaf(q_s[d], to_f32(kp[d]), s);
            p = expf(s * scale - mu) * inv;
        }
        int cnt = min(64, jend - j0);
        for (int jj = 0; jj < cnt; ++jj) {
            float pj = __shfl(p, jj, 64);
            const T* vp = vbase + (int64_t)(j0 + jj) * ld;
#pragma unroll
            for (int t = 0; t < NA; ++t) {
                int d = lane + 64 * t;
                if (d < dh) acc[t] = fmaf(pj, to_f32(vp[d]), acc[t]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NA; ++t) {
        int d = lane + 64 * t;
        if (d < dh) store(d, acc[t]);
    }
}

// dQ over keys [jbeg, jend), not scaled: store(d, sum_j dS_j K_j[d]), dS_j = P_j (dO . V_j - D).  q_s, do_s: the rows in LDS;
// L, D: the row's log-sum-exp and dO . O.
template <int NA, typename T, typename Store>
__device__ __forceinline__ void attn_row_dq(const float* q_s, const float* do_s, const T* kbase, const T* vbase, int64_t ld, int dh,
                                            int jbeg, int jend, float scale, float L, float D, int lane, Store store) {
    float acc[NA] = {};
    for (int j0 = jbeg; j0 < jend; j0 += 64) {
        int j = j0 + lane;
        float ds = 0.0f;
        if (j < jend) {
            const T* kp = kbase + (int64_t)j * ld;
            const T* vp = vbase + (int64_t)j * ld;
            float s = 0.0f, dp = 0.0f;
            for (int d = 0; d < dh; ++d) {
                s = fmaf(q_s[d], to_f32(kp[d]), s);
                dp = fmaf(do_s[d], to_f32(vp[d]), dp);
            }
            ds = expf(s * scale - L) * (dp - D);
        }
        int cnt = min(64, jend - j0);
        for (int jj = 0; jj < cnt; ++jj) {
            float dsj = __shfl(ds, jj, 64);
            const T* kp = kbase + (int64_t)(j0 + jj) * ld;
#pragma unroll
            for (int t = 0; t < NA; ++t) {
                int d = lane + 64 * t;
                if (d < dh) acc[t] = fmaf(dsj, to_f32(kp[d]), acc[t]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NA; ++t) {
        int d = lane + 64 * t;
        if (d < dh) store(d, acc[t]);
    }
}

// dK (not scaled) and dV over queries [ibeg, iend): store(d, sum_i dS_i Q_i[d], sum_i P_i dO_i[d]).  k_s, v_s: the rows in
// LDS; lrow, d_of: log-sum-exp and D of the queries.
template <int NA, typename T, typename DOf, typename Store>
__device__ __forceinline__ void attn_row_dkv(const float* k_s, const float* v_s, const T* qbase, int64_t ld, const T* dobase, int64_t ldo,
                                             const float* lrow, DOf d_of, int dh, int ibeg, int iend, float scale, int lane,
                                             Store store) {
    float dk[NA] = {}, dv[NA] = {};
    for (int i0 = ibeg; i0 < iend; i0 += 64) {
        int i = i0 + lane;
        float p = 0.0f, ds = 0.0f;
        if (i < iend) {
            const T* qp = qbase + (int64_t)i * ld;
            const T* dop = dobase + (int64_t)i * ldo;
            float s = 0.0f, dp = 0.0f;
            for (int d = 0; d < dh; ++d) {
                s = fmaf(to_f32(qp[d]), k_s[d], s);
                dp = fmaf(to_f32(dop[d]), v_s[d], dp);
            }
            p = expf(s * scale - lrow[i]);
            ds = p * (dp - d_of(i));
        }
        int cnt = min(64, iend - i0);
        for (int ii = 0; ii < cnt; ++ii) {
            float pi = __shfl(p, ii, 64), dsi = __shfl(ds, ii, 64);
            const T* qp = qbase + (int64_t)(i0 + ii) * ld;
            const T* dop = dobase + (int64_t)(i0 + ii) * ldo;
#pragma unroll
            for (int t = 0; t < NA; ++t) {
                int d = lane + 64 * t;
                if (d < dh) {
                    dk[t] = fmaf(dsi, to_f32(qp[d]), dk[t]);
                    dv[t] = fmaf(pi, to_f32(dop[d]), dv[t]);
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NA; ++t) {
        int d = lane + 64 * t;
        if (d < dh) store(d, dk[t], dv[t]);
    }
}

}  // namespace tpl

// bf16 GEMM for gfx950: C[M,N] = epi(opA(A) opB(B)), float accumulation on the matrix cores.
//
// Kernels (the host picks one per GEMM by an estimate of its time, see make_plan):
//   gemm_bf16_kernel          4 wavefronts that fetch and compute, MFMA 32x32x16; tiles 256x256, 256x192, and
//                             192x192 / 128x128 with two workgroups per compute unit
//   gemm_bf16_spec_kernel     256x192, 4 math + 4 fetch wavefronts, MFMA 32x32x16      (forward GEMMs: NN)
//   gemm_bf16_spec16_kernel   the same roles on MFMA 16x16x32, K-major A               (data gradients: NT)
//   gemm_bf16_x16s_kernel     192x192, two workgroups per compute unit, MFMA 16x16x32  (weight gradients: TN; short-K
//                             forward GEMMs such as the out-projection)
//   gemm_bf16_x16w8_kernel    256x192, 8 wavefronts that fetch and compute, 16x16x32   (short K, one GEMM at a time)
//   gemm_sum_shares_kernel    adds the partial sums of a GEMM whose K was cut into shares, applies the epilogue
//
// Pipeline.  K is walked in stages of 32 through LDS rings filled by buffer_load ... lds: global memory goes
// straight into LDS, no staging registers, and anything outside the matrix is zero filled by the buffer bounds
// check.  Loads run 2 to 4 stages ahead of the math; there is one workgroup barrier per stage.  The loop bodies
// are written as single pieces (one matrix instruction, one fragment read, one direct load) separated by
// scheduling fences, so the instruction order is the one written.
//
// What decides the design (measured on the device):
//  * With random operands these GEMMs run at the board's power limit with the clock pulled down; throughput then
//    follows energy per flop.  MFMA 16x16x32 needs less than 32x32x16 (each instruction carries 32 k, so the float
//    accumulators are read and written half as often per flop): a pure matrix-instruction loop on random data
//    sustains 15 % more with it.
//  * Issuing a 1 KiB memory instruction (fragment read or direct load) holds a wavefront for about 35 cycles.  Under
//    a 32-cycle 32x32x16 instruction that is almost hidden, under a 16-cycle 16x16x32 it is not.  Hence fetch-only
//    wavefronts beside the math wavefronts, or two wavefronts per SIMD.
//  * Two wavefronts per SIMD leave 256 registers each, 144 to 192 of them accumulators: the 16x16x32 kernels
//    single-buffer their fragments and refill each register as soon as its last use of the k-step is issued.
//
// Operand layouts.  Either operand may be stored with K contiguous ("K-major": A as [M,K], B as [N,K]) or with
// its M/N dimension contiguous ("MN-major": A as [K,M], B as [K,N]).  K-major tiles are read from LDS with
// 16-byte reads; MN-major tiles with the transposing ds_read_b64_tr_b16, which hands each lane four
// K-consecutive values of one column, so no operand is ever transposed in HBM or in registers.  LDS chunk
// positions are XOR-swizzled (applied on the global-address side of the direct loads) so that the reads are
// free of bank conflicts; the XOR depends on the fragment shape that reads the tile.
//
// Scheduling over the chip.  One workgroup per (output tile, K share).  Workgroup ids are dealt round-robin to
// the 8 XCDs (each with its own L2), so ids are regrouped to give every XCD a contiguous run of tiles, and tiles
// are ordered column-major inside bands of a few tile rows (the height that minimises what the tiles in flight on
// an XCD fetch together, see choose_band): the tiles in flight on an XCD share operand panels in that XCD's L2.
//
// Epilogue.  Accumulators go through per-wavefront LDS staging so that every global access of the epilogue
// (bias, residual, GeLU input, output) is a 16-byte access and a staged row is contiguous.
#include <hip/hip_runtime.h>
#include <type_traits>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <mutex>

#include "gemm_bf16_common.h"
#include "gemm_bf16_pp.h"
#include "kernels.h"

namespace tpl {

// Tile variant: 2 x 2 wavefronts, each owning TM x TN MFMA 32x32 blocks -> a (64 TM) x (64 TN) tile.
template <int TM_, int TN_, int STAGES_>
struct Tile {
    static constexpr int TM = TM_, TN = TN_, STAGES = STAGES_;
    static constexpr int BM = 64 * TM, BN = 64 * TN;
    static constexpr int A_BYTES = BM * DK * 2, B_BYTES = BN * DK * 2;   // one stage of each operand
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int LOADS = TM + TN;                                // direct loads per lane and stage
    static constexpr int EROW = TN * 32 * 4 + 16;                        // staged epilogue row of a wavefront
    static constexpr int EWAVE = 32 * EROW;
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES > 4 * EWAVE ? STAGES * STAGE_BYTES : 4 * EWAVE;
    static_assert((STAGES - 1) * LOADS <= 63, "vmcnt is a 6-bit counter");
};

// Epilogue of one wavefront: accumulators -> its LDS staging area -> 16-byte row accesses.  The wavefront's
// part of the tile goes through the staging area in slabs of 32 rows; store_slab(I, stage) writes slab I
// (row r, column c of the wavefront's part at stage + r * EROW + 4 c); a pass then takes 64 / LPR staged rows, 8 columns
// per lane.
//
// What bounds it: vector arithmetic (a plain tile of 192 x 192 takes 5 us of it, with GeLU 11 us, as long as 30 k-steps)
// and, where it reads memory, the latency of that.  So each kind of epilogue is a loop of its own without tests inside,
// its slab's reads are requested before the slab is staged, and the loop over slabs is a loop: only one slab's passes are
// spelled out, because code that runs once per tile comes from memory (spelled out over all slabs and kinds it was 50 KB
// per kernel, of the 64 KB that the instruction cache of two compute units holds).  Measured against that form, whole
// training steps: RoBERTa-large TP 2 0.552 -> 0.516 ms, GPT-3 13B TP 4 1.964 -> 1.886, 175B TP 8 2.368 -> 2.324.  With the
// passes rolled too (a third of the code again) the first two gained 2 % and lost 0.5 %, the last lost 2 %.
template <typename TL>
struct EpilogueLane {
    static constexpr int TM = TL::TM, TN = TL::TN;
    static constexpr int LPR = TN * 4;                            // lanes per staged row (8 columns each)
    static constexpr int RPP = 64 / LPR;                          // rows per pass (lanes beyond RPP * LPR idle when TN = 3)
    static constexpr int PASSES = (32 + RPP - 1) / RPP;
    int er, ec, gn, row0;                                         // row in a pass, column in the staged row, output column, first row
    float bias8[8];
    __device__ __forceinline__ void init(const GemmParams& p, int wm, int wn, int lane, int m0, int n0, const float* partial) {
        er = lane / LPR;
        ec = (lane % LPR) * 8;
        gn = n0 + wn * TN * 32 + ec;
        row0 = m0 + wm * TM * 32 + er;
        if (er >= RPP || gn >= p.N) row0 = p.M;                   // this lane has nothing to store
#pragma unroll
        for (int e = 0; e < 8; ++e) bias8[e] = 0.0f;
        if (p.bias && !partial && gn < p.N) unpack8(*reinterpret_cast<const uint4*>(p.bias + gn), bias8);
    }
    __device__ __forceinline__ bool on(const GemmParams& p, int i, int pass) const {
        return row0 + i * 32 + pass * RPP < p.M && (32 % RPP == 0 || pass * RPP + er < 32);
    }
    __device__ __forceinline__ int64_t index(const GemmParams& p, int i, int pass) const {
        return (int64_t)(row0 + i * 32 + pass * RPP) * p.N + gn;
    }
    template <int KIND>
    __device__ __forceinline__ uint4 fetch(const GemmParams& p, int i, int pass) const {   // residual or GeLU input of a pass
        uint4 v = make_uint4(0, 0, 0, 0);
        if ((KIND == KIND_RESID || KIND == KIND_DGELU) && on(p, i, pass))
            v = *reinterpret_cast<const uint4*>((KIND == KIND_RESID ? p.resid : p.aux) + index(p, i, pass));
        return v;
    }
    template <int KIND>
    __device__ __forceinline__ void emit(const GemmParams& p, const char* stage, int i, int pass, const uint4& in, float* partial) const {
        if (!on(p, i, pass)) return;
        const float4* src = reinterpret_cast<const float4*>(stage + (pass * RPP + er) * TL::EROW + ec * 4);
        const float4 x0 = src[0], x1 = src[1];
        const int64_t idx = index(p, i, pass);
        if constexpr (KIND == KIND_PARTIAL) {                     // one K share: the raw float sums; the epilogue is applied
            float4* dst = reinterpret_cast<float4*>(partial + idx);   // when the shares are summed
            dst[0] = x0; dst[1] = x1;
            return;
        }
        float v8[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v8[e] += bias8[e];
        if (KIND == KIND_RESID || (KIND == KIND_ANY && p.resid)) {
            float r8[8];
            unpack8(KIND == KIND_RESID ? in : *reinterpret_cast<const uint4*>(p.resid + idx), r8);
#pragma unroll
            for (int e = 0; e < 8; ++e) v8[e] += r8[e];
        }
        if (KIND == KIND_GELU || (KIND == KIND_ANY && p.epi == EPI_GELU)) {
            *reinterpret_cast<uint4*>(p.aux + idx) = pack8(v8);
#pragma unroll
            for (int e = 0; e < 8; ++e) v8[e] = gelu_f(v8[e]);
        } else if (KIND == KIND_DGELU || (KIND == KIND_ANY && p.epi == EPI_DGELU)) {
            float u8[8];
            unpack8(KIND == KIND_DGELU ? in : *reinterpret_cast<const uint4*>(p.aux + idx), u8);
#pragma unroll
            for (int e = 0; e < 8; ++e) v8[e] *= gelu_grad_f(u8[e]);
        }
        const uint4 out = pack8(v8);
        if (p.nt_store) {
            typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
            u32x4 o4 = {out.x, out.y, out.z, out.w};
            __builtin_nontemporal_store(o4, reinterpret_cast<u32x4*>(p.C + idx));
        } else {
            *reinterpret_cast<uint4*>(p.C + idx) = out;
        }
    }
};
// store_slab for a slab number that is only known at run time
template <int I, int TM, typename StoreSlab>
__device__ __forceinline__ void store_slab_at(int i, char* stage, StoreSlab store_slab) {
    if constexpr (I < TM) {
        if (i == I) {
            // the markers keep the compiler from merging the cases into one that indexes the accumulators (in scratch memory)
            asm volatile("; slab %0" ::"n"(I));
            store_slab(std::integral_constant<int, I>{}, stage);
            asm volatile("; slab %0 end" ::"n"(I));
        } else {
            store_slab_at<I + 1, TM>(i, stage, store_slab);
        }
    }
}
// The slabs of one wavefront, passes FIRST, FIRST + STEP, ...; before(i) returns the staging buffer of slab i and stage(i)
// fills it (or waits for the wavefront that does).
template <typename TL, int KIND, int FIRST, int STEP, typename StageOf, typename Stage>
__device__ __forceinline__ void epilogue_slabs(const GemmParams& p, const EpilogueLane<TL>& el, float* partial, StageOf stage_of,
                                               Stage stage) {
    using EL = EpilogueLane<TL>;
    constexpr int NP = (EL::PASSES - FIRST + STEP - 1) / STEP;
#pragma unroll 1
    for (int i = 0; i < TL::TM; ++i) {
        uint4 in[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) in[q] = el.template fetch<KIND>(p, i, FIRST + q * STEP);
        stage(i);
#pragma unroll
        for (int q = 0; q < NP; ++q) el.template emit<KIND>(p, stage_of(i), i, FIRST + q * STEP, in[q], partial);
    }
}
template <typename TL, int FIRST, int STEP, typename StageOf, typename Stage>
__device__ __forceinline__ void epilogue_kinds(const GemmParams& p, const EpilogueLane<TL>& el, float* partial, StageOf so, Stage st) {
    if (partial) epilogue_slabs<TL, KIND_PARTIAL, FIRST, STEP>(p, el, partial, so, st);
    else if (p.epi == EPI_NONE && !p.resid) epilogue_slabs<TL, KIND_PLAIN, FIRST, STEP>(p, el, partial, so, st);
    else if (p.epi == EPI_NONE) epilogue_slabs<TL, KIND_RESID, FIRST, STEP>(p, el, partial, so, st);
    else if (p.epi == EPI_GELU && !p.resid) epilogue_slabs<TL, KIND_GELU, FIRST, STEP>(p, el, partial, so, st);
    else if (p.epi == EPI_DGELU && !p.resid) epilogue_slabs<TL, KIND_DGELU, FIRST, STEP>(p, el, partial, so, st);
    else epilogue_slabs<TL, KIND_ANY, FIRST, STEP>(p, el, partial, so, st);
}
template <typename TL, typename StoreSlab>
__device__ __forceinline__ void epilogue_rows(const GemmParams& p, char* smem, int wave, int lane, int m0, int n0,
                                              float* partial, StoreSlab store_slab) {
    char* buf = smem + wave * TL::EWAVE;
    EpilogueLane<TL> el;
    el.init(p, wave >> 1, wave & 1, lane, m0, n0, partial);
    epilogue_kinds<TL, 0, 1>(p, el, partial, [&](int) { return buf; },
                             [&](int i) __attribute__((always_inline)) { store_slab_at<0, TL::TM>(i, buf, store_slab); });
}
// The same for kernels whose fetching wavefronts 4..7 have nothing left to do: math wavefront w stages slab i into
// one of two buffers, and after a workgroup barrier it and wavefront w + 4 (helper) take alternate passes over it.
// Two buffers: the math wavefront stages slab i + 1 while its helper may still read slab i; buffer (i & 1) is
// written again only after the barrier of slab i + 1, which the helper reaches after it has finished slab i.
// Every wavefront of the workgroup executes exactly TM barriers here.  The helper takes the even passes (one more when
// their number is odd): the math wavefront also stages.
template <typename TL, bool HELPER, typename StoreSlab>
__device__ __forceinline__ void epilogue_rows_shared(const GemmParams& p, char* smem, int wave, int lane, int m0, int n0,
                                                     float* partial, StoreSlab store_slab) {
    const int w4 = wave & 3;
    char* buf = smem + w4 * 2 * TL::EWAVE;
    EpilogueLane<TL> el;
    el.init(p, w4 >> 1, w4 & 1, lane, m0, n0, partial);
    epilogue_kinds<TL, HELPER ? 0 : 1, 2>(p, el, partial, [&](int i) { return buf + (i & 1) * TL::EWAVE; },
                                          [&](int i) __attribute__((always_inline)) {
                                              if constexpr (!HELPER) store_slab_at<0, TL::TM>(i, buf + (i & 1) * TL::EWAVE, store_slab);
                                              __syncthreads();
                                          });
}

// 32x32x16 accumulators: register v of block (i,j) is row (v/4)*8 + (lane/32)*4 + v%4, column j*32 + lane%32.
template <typename TL>
__device__ __forceinline__ void epilogue(const GemmParams& p, const f32x16 (&acc)[TL::TM][TL::TN], char* smem,
                                         int wave, int lane, int m0, int n0, float* partial) {
    epilogue_rows<TL>(p, smem, wave, lane, m0, n0, partial, [&](auto ic, char* stage) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int j = 0; j < TL::TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int row = (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
                *reinterpret_cast<float*>(stage + row * TL::EROW + (j * 32 + (lane & 31)) * 4) = acc[i][j][v];
            }
    });
}
// 16x16x32 accumulators: register v of block (i,j) is row i*16 + (lane/16)*4 + v, column j*16 + lane%16.
template <typename TL>
__device__ __forceinline__ void epilogue16(const GemmParams& p, const f32x4 (&acc)[2 * TL::TM][2 * TL::TN], char* smem,
                                           int wave, int lane, int m0, int n0, float* partial) {
    epilogue_rows<TL>(p, smem, wave, lane, m0, n0, partial, [&](auto ic, char* stage) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
            for (int j = 0; j < 2 * TL::TN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    int row = ii * 16 + (lane >> 4) * 4 + v;
                    *reinterpret_cast<float*>(stage + row * TL::EROW + (j * 16 + (lane & 15)) * 4) = acc[2 * i + ii][j][v];
                }
    });
}
// Shared forms (see epilogue_rows_shared): the math wavefronts pass their accumulators, the helpers nothing.
template <typename TL>
__device__ __forceinline__ void epilogue_shared(const GemmParams& p, const f32x16 (&acc)[TL::TM][TL::TN], char* smem,
                                                int wave, int lane, int m0, int n0, float* partial) {
    epilogue_rows_shared<TL, false>(p, smem, wave, lane, m0, n0, partial, [&](auto ic, char* stage) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int j = 0; j < TL::TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int row = (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
                *reinterpret_cast<float*>(stage + row * TL::EROW + (j * 32 + (lane & 31)) * 4) = acc[i][j][v];
            }
    });
}
template <typename TL>
__device__ __forceinline__ void epilogue16_shared(const GemmParams& p, const f32x4 (&acc)[2 * TL::TM][2 * TL::TN],
                                                  char* smem, int wave, int lane, int m0, int n0, float* partial) {
    epilogue_rows_shared<TL, false>(p, smem, wave, lane, m0, n0, partial, [&](auto ic, char* stage) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
            for (int j = 0; j < 2 * TL::TN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    int row = ii * 16 + (lane >> 4) * 4 + v;
                    *reinterpret_cast<float*>(stage + row * TL::EROW + (j * 16 + (lane & 15)) * 4) = acc[2 * i + ii][j][v];
                }
    });
}
template <typename TL>
__device__ __forceinline__ void epilogue_helper(const GemmParams& p, char* smem, int wave, int lane, int m0, int n0,
                                                float* partial) {
    epilogue_rows_shared<TL, true>(p, smem, wave, lane, m0, n0, partial, [](auto, char*) {});
}

// COLSUM: with p.colsum set, the wavefronts that hold the first rows of tile row 0 also add up the columns of B over k
// (the bias gradient that goes with a weight gradient) from the fragments they multiply: four two-element dot products
// with ones per fragment, in float, in their own copy of the loop.
template <typename TL, bool A_KMAJ, bool B_KMAJ, bool COLSUM>
__device__ __forceinline__ void gemm_tile_32(const GemmParams& p, int list_pos, char* smem) {
    constexpr int TM = TL::TM, TN = TL::TN, BM = TL::BM, BN = TL::BN, DSTAGES = TL::STAGES;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const KShare sh = k_share(p, list_pos);

    const i32x4 ra = make_rsrc(p.A, (unsigned)((int64_t)(A_KMAJ ? p.M : p.K) * p.lda * 2));
    const i32x4 rb = make_rsrc(p.B, (unsigned)((int64_t)(B_KMAJ ? p.N : p.K) * p.ldb * 2));
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    constexpr int NM = TM * TN;                                   // matrix instructions per half stage

    int tm, tn;
    tile_coords(sh.tile, p.tiles_m, p.tiles_n, p.band, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    unsigned offa[TM], offb[TN];
    bool oka[TM], okb[TN];
    int kca, kcb;
    dma_offsets<A_KMAJ, TM>(offa, oka, kca, p.lda, m0, p.M, wave, lane);
    dma_offsets<B_KMAJ, TN>(offb, okb, kcb, p.ldb, n0, p.N, wave, lane);

    // Ring slot of stage s (counted from the start of this workgroup's K share) is s % STAGES.  Stages past
    // the end of the share are issued too (all chunks out of
    // bounds: zero fill, no memory traffic) so the number of loads in flight never changes.  The loads
    // of a stage are numbered 0..LOADS-1 (A chunks, then B chunks); every piece of the loop body below
    // is fenced so that the instruction order is the one written: one fragment read or one direct
    // load between matrix instructions, never a burst that fills the memory queue and holds up the
    // wavefront's next matrix instruction.
    constexpr int L = TL::LOADS, L1 = L / 2;                     // part 1: loads [0,L1), part 2: [L1,L)
    auto dma_one = [&](int s, int d) {
        const unsigned buf = lds0 + (s % DSTAGES) * TL::STAGE_BYTES;
        const int k0 = (sh.kt0 + s) * DK;
        if (d < TM) {
            bool ok = A_KMAJ ? (k0 + kca < sh.kend) : (oka[d] && k0 < sh.kend);
            unsigned step = A_KMAJ ? (unsigned)k0 * 2u : (unsigned)((int64_t)k0 * p.lda * 2);
            buffer_load_lds_b128(ra, buf + (wave_u * TM + d) * 1024, ok ? offa[d] + step : OOB_OFFSET);
        } else {
            const int e = d - TM;
            bool ok = B_KMAJ ? (k0 + kcb < sh.kend) : (okb[e] && k0 < sh.kend);
            unsigned step = B_KMAJ ? (unsigned)k0 * 2u : (unsigned)((int64_t)k0 * p.ldb * 2);
            buffer_load_lds_b128(rb, buf + TL::A_BYTES + (wave_u * TN + e) * 1024, ok ? offb[e] + step : OOB_OFFSET);
        }
    };
    auto read_one = [&](bf16x8 (&fa)[TM], bf16x8 (&fb)[TN], int s, int ks, int r) {
        const char* buf = smem + (s % DSTAGES) * TL::STAGE_BYTES;
        if (r < TM) fa[r] = dma_frag<A_KMAJ, BM>(buf, (wm * TM + r) * 32, ks, lane);
        else fb[r - TM] = dma_frag<B_KMAJ, BN>(buf + TL::A_BYTES, (wn * TN + r - TM) * 32, ks, lane);
    };
    float cs[TN], cs_lost[TN], cs_run[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) cs[j] = cs_lost[j] = cs_run[j] = 0.0f;
    // one half stage: NM matrix instructions on (fa, fb); after instruction m, fragment m of the
    // next set is read, and the direct loads d0..d1-1 of stage ds are spread evenly over the half
    auto half = [&](const bf16x8 (&fa)[TM], const bf16x8 (&fb)[TN], bf16x8 (&na)[TM], bf16x8 (&nb)[TN],
                    int rs, int rks, int ds, auto d0c, auto d1c, auto csc) {
        constexpr int D0 = decltype(d0c)::value, D1 = decltype(d1c)::value, NL = D1 - D0;
        if constexpr (decltype(csc)::value) {
#pragma unroll
            for (int j = 0; j < TN; ++j) cs_run[j] = add_elements(fb[j], cs_run[j]);
        }
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            acc[m / TN][m % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[m / TN], fb[m % TN], acc[m / TN][m % TN], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (m < TM + TN) {
                read_one(na, nb, rs, rks, m);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int d = 0; d < NL; ++d)
                if (m == ((2 * d + 1) * NM) / (2 * NL)) {
                    dma_one(ds, D0 + d);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
#pragma unroll
        for (int m = NM; m < TM + TN; ++m) read_one(na, nb, rs, rks, m);   // the smallest tile: more fragments than instructions
    };
    using IC0 = std::integral_constant<int, 0>;
    using ICL1 = std::integral_constant<int, L1>;
    using ICL = std::integral_constant<int, L>;

#pragma unroll
    for (int s0 = 0; s0 < DSTAGES - 1; ++s0)
#pragma unroll
        for (int d = 0; d < L; ++d) dma_one(s0, d);
#pragma unroll
    for (int d = 0; d < L1; ++d) dma_one(DSTAGES - 1, d);
    wait_vmcnt<(DSTAGES - 2) * L + L1>();                        // first stage has landed
    __builtin_amdgcn_s_barrier();
    bf16x8 fa0[TM], fb0[TN], fa1[TM], fb1[TN];
#pragma unroll
    for (int r = 0; r < TM + TN; ++r) read_one(fa0, fb0, 0, 0, r);
    __builtin_amdgcn_sched_barrier(0);

    auto step = [&](int kt, auto csc) __attribute__((always_inline)) {
        // first half: math on k-substep 0, fragments of substep 1 are read, rest of stage kt+STAGES-1 is fetched
        half(fa0, fb0, fa1, fb1, kt, 1, kt + DSTAGES - 1, ICL1{}, ICL{}, csc);
        // stage kt+1 has landed for this wavefront once only the newer stages are in flight; after the
        // barrier it has landed for all, and nobody reads stage kt's slot any more.
        wait_vmcnt<(DSTAGES - 2) * L>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        half(fa1, fb1, fa0, fb0, kt + 1, 0, kt + DSTAGES, IC0{}, ICL1{}, csc);
    };
    const bool cs_on = COLSUM && p.colsum && tm == 0 && __builtin_amdgcn_readfirstlane(wm) == 0;   // uniform over the wavefront
    if constexpr (COLSUM) {
        if (cs_on) {                                             // both copies have one barrier per k-step
            for (int k0 = 0; k0 < sh.nk; k0 += CS_RUN) {
                const int k1 = k0 + CS_RUN < sh.nk ? k0 + CS_RUN : sh.nk;
                for (int kt = k0; kt < k1; ++kt) step(kt, std::true_type{});
#pragma unroll
                for (int j = 0; j < TN; ++j) { add_carrying(cs[j], cs_lost[j], cs_run[j]); cs_run[j] = 0.0f; }
            }
        } else {
            for (int kt = 0; kt < sh.nk; ++kt) step(kt, std::false_type{});
        }
    } else {
        for (int kt = 0; kt < sh.nk; ++kt) step(kt, std::false_type{});
    }
    if (cs_on) {                                                 // lanes l and l + 32 hold the two k halves of column l
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const float v = cs[j] + __shfl_xor(cs[j], 32, 64);
            if (lane < 32) store_colsum(p, sh, n0 + (wn * TN + j) * 32 + lane, v);
        }
    }
    wait_vmcnt<0>();                                             // drain the ring before LDS is reused
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    epilogue<TL>(p, acc, smem, wave, lane, m0, n0, sh.partial);
}

template <typename TL, bool A_KMAJ, bool B_KMAJ>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    gemm_tile_32<TL, A_KMAJ, B_KMAJ, false>(p, share_of_block(blockIdx.x, gridDim.x), smem);
}

// =================================================================================================
// Eight wavefronts on the 16x16x32 matrix instruction: 4 x 2 wavefronts, two per SIMD, each owning
// (2 TM) x (2 TN) blocks of 16 x 16 (64 x 96 of a 256 x 192 tile).
// Why this instruction.  For random operands the chip runs these GEMMs at its power limit, and the 16x16x32
// form needs less energy per flop than 32x32x16 (a pure matrix-instruction loop on random data sustains about
// 15 % more with it: each instruction carries 32 k, so the float accumulators are read and written half as
// often per flop).  What it costs is twice the fragment registers per k and matrix instructions of only 16
// cycles: issuing a 1 KiB memory instruction (fragment read or direct load) holds a wavefront for about 34
// cycles (measured), so a single wavefront per SIMD that also feeds itself leaves the matrix pipe idle; with
// two per SIMD one issues matrix instructions while the other is held.
// Pipeline.  A stage of 32 k is one k-substep; one barrier per stage at its start makes stage kt+1 visible
// (its fragments are read during the matrix instructions of stage kt) and frees the slot of stage kt (read
// during stage kt-1) for stage kt+STAGES.  Wavefronts 0..3 fetch the A stage (2 TM blocks of 1 KiB each),
// wavefronts 4..7 the B stage (TN blocks each); the lane's offset is loop invariant and the k position is
// the scalar offset of the load, checked against the end of the K share only in the last few stages.
// Where it is used.  Its fixed cost per tile is lower than that of the kernel with fetch-only wavefronts
// and its time per k-step higher (K-major operands arrive as half cache lines in 32-k stages), so the host
// picks it for short K.
// =================================================================================================
// acc += a b, the accumulator tied to one AGPR quad.  Written as assembly because the compiler otherwise
// moves the four-register accumulators between registers around every matrix instruction.  No other
// matrix or vector instruction touches an accumulator within a stage, so no wait states are needed between
// these; the reader after the loop inserts them itself (mfma16_drain).
__device__ __forceinline__ void mfma16_inplace(f32x4& acc, const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

template <int TM_, int TN_, int STAGES_>
struct Tile8 {
    static constexpr int TM = TM_, TN = TN_, STAGES = STAGES_;          // 32-row / 32-column units per wavefront
    static constexpr int BM = 4 * 32 * TM, BN = 2 * 32 * TN;
    static constexpr int A_BYTES = BM * DK * 2, B_BYTES = BN * DK * 2;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int LA = 2 * TM, LB = TN;                          // direct loads per stage of an A / B fetcher
    static constexpr int LMAX = LA > LB ? LA : LB;
    static constexpr int EROW = TN * 32 * 4 + 16, EWAVE = 32 * EROW;
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES > 8 * EWAVE ? STAGES * STAGE_BYTES : 8 * EWAVE;
    static_assert(STAGES * LMAX <= 63, "vmcnt is a 6-bit counter");
};

template <typename TL, bool A_KMAJ, bool B_KMAJ>
__global__ __launch_bounds__(512) void gemm_bf16_x16w8_kernel(GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int TM = TL::TM, TN = TL::TN, BM = TL::BM, BN = TL::BN, DSTAGES = TL::STAGES;
    constexpr int FM = 2 * TM, FN = 2 * TN, NM = FM * FN;
    constexpr int LA = TL::LA, LB = TL::LB, LMAX = TL::LMAX;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const bool is_a = wave_u < 4;                                 // which operand this wavefront fetches
    const int wq = wave_u & 3;
    const KShare sh = k_share(p, share_of_block(blockIdx.x, gridDim.x));
    int tm, tn;
    tile_coords(sh.tile, p.tiles_m, p.tiles_n, p.band, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    // fetch state of this wavefront: descriptor, LDS position of its first block inside a stage, bytes per k,
    // per-lane offsets (rows / columns outside the matrix folded in) and the lane's k column (K-major only)
    const i32x4 ra = make_rsrc(p.A, (unsigned)((int64_t)(A_KMAJ ? p.M : p.K) * p.lda * 2));
    const i32x4 rb = make_rsrc(p.B, (unsigned)((int64_t)(B_KMAJ ? p.N : p.K) * p.ldb * 2));
    i32x4 rs;
#pragma unroll
    for (int q = 0; q < 4; ++q) rs[q] = is_a ? ra[q] : rb[q];
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    const unsigned lds_first = lds0 + (is_a ? wq * LA * 1024 : TL::A_BYTES + wq * LB * 1024);
    const unsigned kbytes = is_a ? (A_KMAJ ? 2u : (unsigned)p.lda * 2u) : (B_KMAJ ? 2u : (unsigned)p.ldb * 2u);
    const int nload = is_a ? LA : LB;
    unsigned vo[LMAX];
    int kc = 0;
    if (is_a) {
        unsigned off[LA]; bool ok[LA];
        dma_offsets<A_KMAJ, LA, false, true>(off, ok, kc, p.lda, m0, p.M, wq, lane);
#pragma unroll
        for (int d = 0; d < LMAX; ++d) vo[d] = d < LA ? ((A_KMAJ || ok[d < LA ? d : 0]) ? off[d < LA ? d : 0] : OOB_HALF) : OOB_HALF;
        if (!A_KMAJ) kc = 0;
    } else {
        unsigned off[LB]; bool ok[LB];
        dma_offsets<B_KMAJ, LB, false, true>(off, ok, kc, p.ldb, n0, p.N, wq, lane);
#pragma unroll
        for (int d = 0; d < LMAX; ++d) vo[d] = d < LB ? ((B_KMAJ || ok[d < LB ? d : 0]) ? off[d < LB ? d : 0] : OOB_HALF) : OOB_HALF;
        if (!B_KMAJ) kc = 0;
    }
    // load d of stage s (of this K share); CHECKED: the stage may reach past the end of the share
    auto dma_one = [&](int s, int d, auto checkedc) {
        if (d >= LA && is_a) return;
        if (d >= LB && !is_a) return;
        const unsigned k0 = (unsigned)(sh.kt0 + s) * DK;
        unsigned v = vo[d];
        if (decltype(checkedc)::value) v = (int)k0 + kc < sh.kend ? v : OOB_HALF;
        buffer_load_lds_b128_s(rs, lds_first + (s % DSTAGES) * TL::STAGE_BYTES + d * 1024, v, k0 * kbytes);
    };
    auto read_one = [&](bf16x8 (&fa)[FM], bf16x8 (&fb)[FN], int s, int r) {
        const char* buf = smem + (s % DSTAGES) * TL::STAGE_BYTES;
        if (r < FM) fa[r] = dma_frag16<A_KMAJ, BM>(buf, (wm * FM + r) * 16, lane);
        else fb[r - FM] = dma_frag16<B_KMAJ, BN>(buf + TL::A_BYTES, (wn * FN + r - FM) * 16, lane);
    };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;

    auto stage = [&](const bf16x8 (&fa)[FM], const bf16x8 (&fb)[FN], bf16x8 (&na)[FM], bf16x8 (&nb)[FN], int kt, auto checkedc) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int m = i * FN + j;
                mfma16_inplace(acc[i][j], fa[i], fb[j]);
                __builtin_amdgcn_sched_barrier(0);
                if (m < FM + FN) {
                    read_one(na, nb, kt + 1, m);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int d = 0; d < LMAX; ++d)
                    if (m == ((2 * d + 1) * NM) / (2 * LMAX)) {
                        dma_one(kt + DSTAGES, d, checkedc);
                        __builtin_amdgcn_sched_barrier(0);
                    }
            }
    };
    using Fast = std::integral_constant<bool, false>;
    using Checked = std::integral_constant<bool, true>;
    // loads this wavefront may leave in flight with stage s+1 landed: those of the D-2 newer stages
    auto wait_stage = [&]() {
        if (LA == LB) wait_vmcnt<(DSTAGES - 2) * LA>();
        else if (is_a) wait_vmcnt<(DSTAGES - 2) * LA>();
        else wait_vmcnt<(DSTAGES - 2) * LB>();
    };

#pragma unroll
    for (int s0 = 0; s0 < DSTAGES; ++s0)
#pragma unroll
        for (int d = 0; d < LMAX; ++d) dma_one(s0, d, Checked{});
    if (LA == LB) wait_vmcnt<(DSTAGES - 1) * LA>();              // stage 0 has landed
    else if (is_a) wait_vmcnt<(DSTAGES - 1) * LA>();
    else wait_vmcnt<(DSTAGES - 1) * LB>();
    __builtin_amdgcn_s_barrier();
    bf16x8 fa0[FM], fb0[FN], fa1[FM], fb1[FN];
#pragma unroll
    for (int r = 0; r < FM + FN; ++r) read_one(fa0, fb0, 0, r);
    __builtin_amdgcn_sched_barrier(0);

    auto sync = [&]() {
        wait_stage();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    const int nfast = (sh.kend - sh.kt0 * DK) / DK - DSTAGES;
    int kt = 0;
    for (; kt + 1 < nfast; kt += 2) {
        sync();
        stage(fa0, fb0, fa1, fb1, kt, Fast{});
        sync();
        stage(fa1, fb1, fa0, fb0, kt + 1, Fast{});
    }
    for (; kt + 1 < sh.nk; kt += 2) {
        sync();
        stage(fa0, fb0, fa1, fb1, kt, Checked{});
        sync();
        stage(fa1, fb1, fa0, fb0, kt + 1, Checked{});
    }
    if (kt < sh.nk) {
        sync();
        stage(fa0, fb0, fa1, fb1, kt, Checked{});
    }
    mfma16_drain();
    wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    epilogue16<TL>(p, acc, smem, wave, lane, m0, n0, sh.partial);
}

// =================================================================================================
// Variant with specialised wavefronts: 512 threads, wavefronts 0..3 only compute (2 x 2, each
// TM x TN blocks), wavefronts 4..7 only fetch.  Both roles meet at the same barriers: one before the
// loop, one per k-step of 32, one after.
//
// LDS rings.  B lives in a ring of NB slots of 32 k.  A K-major A lives in a ring of 3 slots of 64 k
// (rows of 128 bytes): a direct load then covers 8 whole 128-byte lines instead of 16 half lines,
// which the vector memory path serves about 1.4 times faster (measured), and global->LDS
// throughput is what bounds this kernel once the loads no longer hold up matrix instructions.
// (B stays at 32 k: three 64-k slots of both operands do not fit in 160 KiB.)  An MN-major A uses
// a ring of NB slots of 32 k like B.  Slot of k-step kt: B kt % NB; wide A (kt / 2) % 3.
//
// Fetch order.  After the barrier of k-step kt the B slot of kt is free and is refilled with k-step
// kt + NB.  A wide A slot (unit u = k-steps 2u, 2u+1) is free after the barrier of k-step 2u+1; unit
// u+3 is fetched in two halves, after that barrier and after the next one, so every k-step issues
// TM + TN loads per fetching wavefront.
// =================================================================================================
template <int TM_, int TN_>
struct SpecTile {
    static constexpr int TM = TM_, TN = TN_, BM = 64 * TM, BN = 64 * TN;
    static constexpr int NB = 5, NA_WIDE = 3;
    static constexpr int B_SLOT = BN * DK * 2;                           // 32 k of B
    static constexpr int A_SLOT32 = BM * DK * 2, A_SLOT64 = BM * 64 * 2;
    static constexpr int EROW = TN * 32 * 4 + 16, EWAVE = 32 * EROW;     // epilogue staging, as in Tile
    template <bool A_KMAJ> static constexpr int a_bytes() { return A_KMAJ ? NA_WIDE * A_SLOT64 : NB * A_SLOT32; }
    template <bool A_KMAJ> static constexpr int lds_bytes() {
        return a_bytes<A_KMAJ>() + NB * B_SLOT > 8 * EWAVE ? a_bytes<A_KMAJ>() + NB * B_SLOT : 8 * EWAVE;   // 8: two staging buffers per math wavefront
    }
};

// One operand's loads of one k range [k0, k0 + KSPAN) by a fetching wavefront: NL loads, load i to LDS block
// lds_first + 1024 i.  off[i] is the lane's loop-invariant byte offset (k = 0; rows or columns outside the matrix
// already point past the buffer), kin[i] the lane's k position inside the range (K-major: its chunk's first k;
// MN-major: its row), kstep_bytes the bytes per unit of k (2 for K-major, 2 ld for MN-major).
//  * range inside the K share: the k position is the load's SCALAR offset, the lane offset is used as it is;
//  * range past the end of the share: a descriptor of zero records (nothing is read, zeros land in LDS);
//  * range that straddles the end (K not a multiple of the range): per-lane check, the only case with vector
//    instructions.  A vector instruction issued by a fetching wavefront takes an issue slot from the matrix
//    instructions of the math wavefront on the same SIMD (measured: about 2 cycles of matrix-pipe time each), which
//    is why the steady state has none.
template <int NL, int KSPAN>
__device__ __forceinline__ void fetch_range(const i32x4& rsrc, unsigned lds_first, const unsigned (&off)[NL],
                                            const int (&kin)[NL], int k0, int kend, unsigned kstep_bytes) {
    if (k0 >= kend) {
        i32x4 r = rsrc;
        r[2] = 0;
#pragma unroll
        for (int i = 0; i < NL; ++i) buffer_load_lds_b128_s(r, lds_first + i * 1024, off[i], 0u);
    } else if (k0 + KSPAN <= kend) {
        // (the compiler does not always see that the product is wave-uniform)
        const unsigned so = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)k0 * kstep_bytes));
#pragma unroll
        for (int i = 0; i < NL; ++i) buffer_load_lds_b128_s(rsrc, lds_first + i * 1024, off[i], so);
    } else {
#pragma unroll
        for (int i = 0; i < NL; ++i)
            buffer_load_lds_b128(rsrc, lds_first + i * 1024,
                                 k0 + kin[i] < kend ? off[i] + (unsigned)k0 * kstep_bytes : OOB_OFFSET);
    }
}

__device__ __forceinline__ bf16x8 wide_frag(const char* tile, int mn_base, int k16, int lane) {
    int row = mn_base + (lane & 31);
    int c = 2 * k16 + (lane >> 5);
    return *reinterpret_cast<const bf16x8*>(tile + row * 128 + ((c ^ swz_k64(row)) << 4));
}

template <typename ST, bool A_KMAJ, bool B_KMAJ>
__global__ __launch_bounds__(512) void gemm_bf16_spec_kernel(GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int TM = ST::TM, TN = ST::TN, BM = ST::BM, BN = ST::BN, NB = ST::NB, NAW = ST::NA_WIDE;
    constexpr bool WIDE = A_KMAJ;
    constexpr int A_BYTES = ST::template a_bytes<A_KMAJ>();
    constexpr int LPS = TM + TN;                                  // loads per k-step and fetching wavefront
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const KShare sh = k_share(p, share_of_block(blockIdx.x, gridDim.x));   // sh.kt0 is even (host)
    int tm, tn;
    tile_coords(sh.tile, p.tiles_m, p.tiles_n, p.band, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    if (wave >= 4) {
        // ---------------- fetching wavefronts ----------------
        const int w = __builtin_amdgcn_readfirstlane(wave) & 3;
        const i32x4 ra = make_rsrc(p.A, (unsigned)((int64_t)(A_KMAJ ? p.M : p.K) * p.lda * 2));
        const i32x4 rb = make_rsrc(p.B, (unsigned)((int64_t)(B_KMAJ ? p.N : p.K) * p.ldb * 2));
        const unsigned lds_a = (unsigned)(uintptr_t)(lds_void_ptr)smem, lds_b = lds_a + A_BYTES;
        // Lane offsets of this wavefront's loads (see fetch_range): B and a narrow A as in the kernel above; a wide A
        // unit is 2 TM loads, load q covering rows 8 (2 TM w + q) .. + 7, lane l the chunk at LDS position l % 8 of
        // row l / 8.
        unsigned offb[TN], offa[TM], offw0[TM], offw1[TM];
        int kinb[TN], kina[TM], kinw0[TM], kinw1[TM];
        {
            bool okb[TN];
            int kc;
            dma_offsets<B_KMAJ, TN>(offb, okb, kc, p.ldb, n0, p.N, w, lane);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (!B_KMAJ) offb[j] = okb[j] ? offb[j] : OOB_HALF;
                kinb[j] = B_KMAJ ? kc : mn_krow<TN>(w, j, lane);
            }
        }
        if (WIDE) {
#pragma unroll
            for (int q = 0; q < 2 * TM; ++q) {
                const int row = (w * 2 * TM + q) * 8 + (lane >> 3);
                const int c = (lane & 7) ^ swz_k64(row);
                const unsigned o = m0 + row < p.M ? (unsigned)(((int64_t)(m0 + row) * p.lda + c * 8) * 2) : OOB_HALF;
                if (q < TM) { offw0[q] = o; kinw0[q] = c * 8; }
                else { offw1[q - TM] = o; kinw1[q - TM] = c * 8; }
            }
        } else {
            bool oka[TM];
            int kc;
            dma_offsets<A_KMAJ, TM>(offa, oka, kc, p.lda, m0, p.M, w, lane);
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                if (!A_KMAJ) offa[j] = oka[j] ? offa[j] : OOB_HALF;
                kina[j] = A_KMAJ ? kc : mn_krow<TM>(w, j, lane);
            }
        }
        const unsigned kb_bytes = B_KMAJ ? 2u : (unsigned)p.ldb * 2u, ka_bytes = A_KMAJ ? 2u : (unsigned)p.lda * 2u;
        // k-steps kt and wide units u below count from the start of this workgroup's K share
        auto load_b = [&](int kt) {                               // k-step kt of B into its slot
            fetch_range<TN, DK>(rb, lds_b + (kt % NB) * ST::B_SLOT + w * TN * 1024, offb, kinb, (sh.kt0 + kt) * DK, sh.kend,
                                kb_bytes);
        };
        auto load_a32 = [&](int kt) {
            fetch_range<TM, DK>(ra, lds_a + (kt % NB) * ST::A_SLOT32 + w * TM * 1024, offa, kina, (sh.kt0 + kt) * DK, sh.kend,
                                ka_bytes);
        };
        auto load_a64 = [&](int u, int half) {                    // half 0/1 of unit u (k = 64 u ..)
            const unsigned buf = lds_a + (u % NAW) * ST::A_SLOT64 + (w * 2 * TM + half * TM) * 1024;
            const int k0 = 64 * ((sh.kt0 >> 1) + u);
            if (half == 0) fetch_range<TM, 64>(ra, buf, offw0, kinw0, k0, sh.kend, 2u);
            else fetch_range<TM, 64>(ra, buf, offw1, kinw1, k0, sh.kend, 2u);
        };
        // prologue: everything the rings hold, except the second half of the last wide unit
        if (WIDE) {
            load_a64(0, 0); load_a64(0, 1); load_b(0);
            load_a64(1, 0); load_a64(1, 1); load_a64(2, 0);
#pragma unroll
            for (int s0 = 1; s0 < NB; ++s0) load_b(s0);
            wait_vmcnt<3 * TM + (NB - 1) * TN>();                 // unit 0 and B step 0 have landed
        } else {
            load_a32(0); load_b(0);
#pragma unroll
            for (int s0 = 1; s0 < NB; ++s0) { load_a32(s0); load_b(s0); }
            wait_vmcnt<(NB - 1) * LPS>();
        }
        __builtin_amdgcn_s_barrier();
        // Loads in flight allowed at the barrier of k-step kt (k-step kt+1 must have landed).  B step
        // kt+1 went out as the last loads of k-step kt+1-NB; the second half of a wide unit that starts
        // at kt+1 went out as the first loads of k-step kt-3.
        constexpr int W_B = (NB - 2) * LPS;
        constexpr int W_A = WIDE ? TN + 2 * LPS : TN + (NB - 2) * LPS;
        constexpr int W = W_A < W_B ? W_A : W_B;
        for (int kt = 0; kt < sh.nk; ++kt) {
            // The first two k-steps of a wide A come straight after the prologue, which ends with the
            // B steps: fewer loads follow the ones needed than in the steady state.
            if (WIDE && kt == 0) wait_vmcnt<(NB - 2) * TN>();                  // B step 1
            else if (WIDE && kt == 1) wait_vmcnt<(NB - 3) * TN + LPS>();       // unit 1, B step 2
            else wait_vmcnt<W>();
            __builtin_amdgcn_s_barrier();                         // k-step kt has been read by everyone
            if (WIDE) {
                // odd kt = 2u+1 frees unit u: first half of unit u+3; even kt = 2u+2: its second half
                if (kt & 1) load_a64((kt >> 1) + 3, 0);
                else load_a64((kt >> 1) + 2, 1);
            } else {
                load_a32(kt + NB);
            }
            load_b(kt + NB);
        }
        wait_vmcnt<0>();                                          // nothing lands in LDS during the epilogue
        __builtin_amdgcn_s_barrier();
        epilogue_helper<ST>(p, smem, wave, lane, m0, n0, sh.partial);   // shares the rows of math wavefront wave - 4
        return;
    }

    // ---------------- math wavefronts ----------------
    const int wm = wave >> 1, wn = wave & 1;
    constexpr int NM = TM * TN;
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    // Registers: the accumulators take 3/4 of a wavefront's budget (two wavefronts per SIMD), so only
    // the B fragments and the last A fragment are double buffered; A fragment i < TM-1 of the next
    // k-substep is read into the registers of the current one once row i's matrix instructions are issued.
    bf16x8 fa[TM - 1], fal[2], fb[2][TN];
    auto rd_a = [&](bf16x8& dst, int kt, int ks, int i) {         // k-substep ks (16 k) of k-step kt
        if (WIDE) dst = wide_frag(smem + ((kt >> 1) % NAW) * ST::A_SLOT64, (wm * TM + i) * 32, (kt & 1) * 2 + ks, lane);
        else dst = dma_frag<A_KMAJ, BM>(smem + (kt % NB) * ST::A_SLOT32, (wm * TM + i) * 32, ks, lane);
    };
    auto rd_b = [&](bf16x8& dst, int kt, int ks, int j) {
        dst = dma_frag<B_KMAJ, BN>(smem + A_BYTES + (kt % NB) * ST::B_SLOT, (wn * TN + j) * 32, ks, lane);
    };
    auto mhalf = [&](auto curc, int rkt, int rks) {
        constexpr int CUR = decltype(curc)::value, NXT = CUR ^ 1;
        int free_rd = 0;                                          // next of: B fragments 0..TN-1, last A fragment
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int i = m / TN, j = m % TN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(i < TM - 1 ? fa[i] : fal[CUR], fb[CUR][j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (j == TN - 1 && i < TM - 1) {
                rd_a(fa[i], rkt, rks, i);                         // row i is done: refill in place
                __builtin_amdgcn_sched_barrier(0);
            } else if (free_rd <= TN) {
                if (free_rd < TN) rd_b(fb[NXT][free_rd], rkt, rks, free_rd);
                else rd_a(fal[NXT], rkt, rks, TM - 1);
                ++free_rd;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < TM - 1; ++i) rd_a(fa[i], 0, 0, i);
    rd_a(fal[0], 0, 0, TM - 1);
#pragma unroll
    for (int j = 0; j < TN; ++j) rd_b(fb[0][j], 0, 0, j);
    __builtin_amdgcn_sched_barrier(0);
    for (int kt = 0; kt < sh.nk; ++kt) {
        mhalf(C0{}, kt, 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        mhalf(C1{}, kt + 1, 0);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    epilogue_shared<ST>(p, acc, smem, wave, lane, m0, n0, sh.partial);
}

// Sum of the K shares in share order, then the epilogue; 8 columns per thread, every access 16 or 32 bytes.
__device__ __forceinline__ void sum_shares(const GemmParams& p, int shares, int64_t chunk) {
    const int64_t idx = chunk * 8;
    const int64_t mn = (int64_t)p.M * p.N;
    if (idx >= mn) return;
    float v8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int s = 0; s < shares; ++s) {
        const float4* src = reinterpret_cast<const float4*>(p.partial + s * mn + idx);
        const float4 x0 = src[0], x1 = src[1];
        v8[0] += x0.x; v8[1] += x0.y; v8[2] += x0.z; v8[3] += x0.w;
        v8[4] += x1.x; v8[5] += x1.y; v8[6] += x1.z; v8[7] += x1.w;
    }
    if (p.bias) {
        float b8[8];
        unpack8(*reinterpret_cast<const uint4*>(p.bias + idx % p.N), b8);
#pragma unroll
        for (int e = 0; e < 8; ++e) v8[e] += b8[e];
    }
    if (p.resid) {
        float r8[8];
        unpack8(*reinterpret_cast<const uint4*>(p.resid + idx), r8);
#pragma unroll
        for (int e = 0; e < 8; ++e) v8[e] += r8[e];
    }
    if (p.epi == EPI_GELU) {
        *reinterpret_cast<uint4*>(p.aux + idx) = pack8(v8);
#pragma unroll
        for (int e = 0; e < 8; ++e) v8[e] = gelu_f(v8[e]);
    } else if (p.epi == EPI_DGELU) {
        float u8[8];
        unpack8(*reinterpret_cast<const uint4*>(p.aux + idx), u8);
#pragma unroll
        for (int e = 0; e < 8; ++e) v8[e] *= gelu_grad_f(u8[e]);
    }
    *reinterpret_cast<uint4*>(p.C + idx) = pack8(v8);
}
__global__ __launch_bounds__(256) void gemm_sum_shares_kernel(GemmParams p, int shares) {
    sum_shares(p, shares, (int64_t)blockIdx.x * 256 + threadIdx.x);
}

// =================================================================================================
// Fetch and math wavefronts on the 16x16x32 matrix instruction (K-major A only): the tile, the rings and the
// fetching wavefronts of the kernel above, the matrix instruction of the 8-wavefront kernel.  A math wavefront
// owns 128 x 96 = 8 x 6 blocks: 192 accumulator registers of the 256 a wavefront has at two per SIMD, so
// fragments cannot be double buffered.  The 6 B fragments of a k-step stay in registers; the 8 A fragments
// (one per row of blocks, used for 6 consecutive instructions) rotate through four register sets, each refilled
// two rows ahead of its use.  A B fragment is refilled with the next k-step's as soon as it is dead: the last
// two rows are walked column by column, so B fragment j is dead after two instructions, and the next k-step
// starts with two rows walked the same way, which gives every B fragment ten instructions (160 cycles) to
// arrive.  Because the last fragment reads of k-step kt+1 are still in flight when k-step kt ends, the slot of
// k-step kt is handed back to the fetching wavefronts one barrier later than above (at barrier kt+1), and the
// fetch schedule is one k-step shorter: after barrier j, B k-step j+4 and (j even) the whole A unit j/2+2.
// =================================================================================================
__device__ __forceinline__ bf16x8 wide_frag16(const char* tile, int mn_base, int k32, int lane) {
    int row = mn_base + (lane & 15);
    int c = 4 * k32 + (lane >> 4);
    return *reinterpret_cast<const bf16x8*>(tile + row * 128 + ((c ^ swz_k64(row)) << 4));
}
__device__ __forceinline__ void mfma16_v(f32x4& acc, const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}

template <typename ST, bool B_KMAJ>
__global__ __launch_bounds__(512) void gemm_bf16_spec16_kernel(GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int TM = ST::TM, TN = ST::TN, BM = ST::BM, BN = ST::BN, NB = ST::NB, NAW = ST::NA_WIDE;
    constexpr int A_BYTES = ST::template a_bytes<true>();
    constexpr int LA = 2 * TM, LBW = TN;                          // loads per fetching wavefront: A unit, B k-step
    static_assert(NB == 5 && NAW == 3, "the fetch schedule below is written for these ring depths");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const KShare sh = k_share(p, share_of_block(blockIdx.x, gridDim.x));   // sh.kt0 is even (host)
    int tm, tn;
    tile_coords(sh.tile, p.tiles_m, p.tiles_n, p.band, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    if (wave >= 4) {
        // ---------------- fetching wavefronts ----------------
        const int w = __builtin_amdgcn_readfirstlane(wave) & 3;
        const i32x4 ra = make_rsrc(p.A, (unsigned)((int64_t)p.M * p.lda * 2));
        const i32x4 rb = make_rsrc(p.B, (unsigned)((int64_t)(B_KMAJ ? p.N : p.K) * p.ldb * 2));
        const unsigned lds_a = (unsigned)(uintptr_t)(lds_void_ptr)smem, lds_b = lds_a + A_BYTES;
        // lane offsets of this wavefront's loads (see fetch_range)
        unsigned offb[TN], offw[LA];
        int kinb[TN], kinw[LA];
        {
            bool okb[TN];
            int kc;
            dma_offsets<B_KMAJ, TN, true, true>(offb, okb, kc, p.ldb, n0, p.N, w, lane);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (!B_KMAJ) offb[j] = okb[j] ? offb[j] : OOB_HALF;
                kinb[j] = B_KMAJ ? kc : mn_krow<TN>(w, j, lane);
            }
        }
#pragma unroll
        for (int q = 0; q < LA; ++q) {
            const int row = (w * LA + q) * 8 + (lane >> 3);
            const int c = (lane & 7) ^ swz_k64(row);
            kinw[q] = c * 8;
            offw[q] = m0 + row < p.M ? (unsigned)(((int64_t)(m0 + row) * p.lda + c * 8) * 2) : OOB_HALF;
        }
        const unsigned kb_bytes = B_KMAJ ? 2u : (unsigned)p.ldb * 2u;
        auto load_b = [&](int kt) {                               // k-step kt (of this K share) of B into its slot
            fetch_range<TN, DK>(rb, lds_b + (kt % NB) * ST::B_SLOT + w * TN * 1024, offb, kinb, (sh.kt0 + kt) * DK, sh.kend,
                                kb_bytes);
        };
        auto load_a = [&](int u) {                                // unit u (k-steps 2u, 2u+1 of this K share) of A
            fetch_range<LA, 64>(ra, lds_a + (u % NAW) * ST::A_SLOT64 + w * LA * 1024, offw, kinw, 64 * ((sh.kt0 >> 1) + u),
                                sh.kend, 2u);
        };
        load_a(0); load_b(0); load_b(1); load_a(1); load_b(2); load_b(3);
        wait_vmcnt<LA + 3 * LBW>();                               // unit 0 and B k-step 0 have landed
        __builtin_amdgcn_s_barrier();
        // At barrier kt k-step kt+1 must have landed.  Loads go out in batches after each barrier (the A unit,
        // then the B k-step); the two newest batches, LA + 2 LBW loads, may still be in flight.
        for (int kt = 0; kt < sh.nk; ++kt) {
            wait_vmcnt<LA + 2 * LBW>();
            __builtin_amdgcn_s_barrier();                         // k-step kt-1 has been read by everyone
            if ((kt & 1) == 0) load_a((kt >> 1) + 2);
            load_b(kt + NB - 1);
        }
        wait_vmcnt<0>();                                          // nothing lands in LDS during the epilogue
        __builtin_amdgcn_s_barrier();
        epilogue_helper<ST>(p, smem, wave, lane, m0, n0, sh.partial);   // shares the rows of math wavefront wave - 4
        return;
    }

    // ---------------- math wavefronts ----------------
    const int wm = wave >> 1, wn = wave & 1;
    constexpr int FM = 2 * TM, FN = 2 * TN;
    static_assert(FM >= 4, "head and tail pairs need four rows of blocks");
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;
    static_assert(FM == 8, "the row schedule below is written for 8 rows of blocks");
    bf16x8 fa[4], fb[FN];                                         // A fragments rotate through four registers sets
    auto rd_a = [&](int kt, int row, int r) {                     // row `row` of k-step kt into set r
        fa[r] = wide_frag16(smem + ((kt >> 1) % NAW) * ST::A_SLOT64, (wm * FM + row) * 16, kt & 1, lane);
        __builtin_amdgcn_sched_barrier(0);
    };
    // MN-major B (rows of BN values per k, chunk c of row k at position c ^ xor16(k)): fragment f = wn FN + j of
    // the tile is chunks 2f, 2f+1; a lane reads rows k = 8 (lane/16) + 4 h + (lane%16)/4, h = 0, 1, whose xor16
    // does not depend on h, so fragment f sits at bpos[(f ^ x) & 3] + 128 (f / 4) + 1536 h with x fixed per lane:
    // four base registers, everything else immediates and scalars.
    unsigned bpos[4];
    int bq[FN], bs[FN];                                           // per fragment: which base, scalar byte offset
    if (!B_KMAJ) {
        const int k0 = 8 * (lane >> 4) + ((lane & 15) >> 2);
        const int x = ((lane >> 3) & 1) | (((lane >> 4) & 1) << 1);
        const unsigned base = (unsigned)(k0 * (BN * 2) + 8 * (lane & 1) + 16 * ((lane & 3) >> 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) bpos[q] = base + 32u * (unsigned)((q + 2 * wn) & 3 ^ x);
#pragma unroll
        for (int j = 0; j < FN; ++j) { bq[j] = j & 3; bs[j] = 128 * ((wn * FN + j) >> 2); }
    }
    auto rd_b = [&](int kt, int j) {
        const char* slot = smem + A_BYTES + (kt % NB) * ST::B_SLOT;
        if (B_KMAJ) {
            fb[j] = dma_frag16<true, BN>(slot, (wn * FN + j) * 16, lane);
        } else {
            const char* src = slot + __builtin_amdgcn_readfirstlane(bs[j]) + bpos[bq[j]];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(src + h * 4 * (BN * 2)));
                bf16x4 b4 = __builtin_bit_cast(bf16x4, v);
                fb[j][4 * h + 0] = b4[0]; fb[j][4 * h + 1] = b4[1]; fb[j][4 * h + 2] = b4[2]; fb[j][4 * h + 3] = b4[3];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mm = [&](int i, int r, int j) {                          // block (i, j) with the A fragment in set r
        mfma16_v(acc[i][j], fa[r], fb[j]);
        __builtin_amdgcn_sched_barrier(0);
    };
    // reads still in flight at the end of a k-step: the FN B fragments and 2 A fragments of its last lines
    constexpr int TAIL_READS = (B_KMAJ ? FN : 2 * FN) + 2;
    static_assert(TAIL_READS <= 15, "lgkmcnt is a 4-bit counter");
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r) rd_a(0, r, r);
#pragma unroll
    for (int j = 0; j < FN; ++j) rd_b(0, j);
    // Row schedule of a k-step (sets 0..3 hold rows 0..3 at its start):
    //   rows 0,1 column by column | read rows 4,5 -> sets 0,1 | row 2, read row 6 -> set 2 | row 3, read row 7 -> set 3
    //   | row 4, read next row 0 -> set 0 | row 5, read next row 1 -> set 1
    //   | rows 6,7 column by column, each B fragment refilled once both have used it | read next rows 2,3 -> sets 2,3
    for (int kt = 0; kt < sh.nk; ++kt) {
        asm volatile("s_waitcnt lgkmcnt(%0)" :: "n"(TAIL_READS) : "memory");   // every read of k-step kt-1's slots is done
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < FN; ++j) { mm(0, 0, j); mm(1, 1, j); }
        rd_a(kt, 4, 0);
        rd_a(kt, 5, 1);
#pragma unroll
        for (int j = 0; j < FN; ++j) mm(2, 2, j);
        rd_a(kt, 6, 2);
#pragma unroll
        for (int j = 0; j < FN; ++j) mm(3, 3, j);
        rd_a(kt, 7, 3);
#pragma unroll
        for (int j = 0; j < FN; ++j) mm(4, 0, j);
        rd_a(kt + 1, 0, 0);
#pragma unroll
        for (int j = 0; j < FN; ++j) mm(5, 1, j);
        rd_a(kt + 1, 1, 1);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            mm(6, 2, j); mm(7, 3, j);
            rd_b(kt + 1, j);
        }
        rd_a(kt + 1, 2, 2);
        rd_a(kt + 1, 3, 3);
    }
    mfma16_drain();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    epilogue16_shared<ST>(p, acc, smem, wave, lane, m0, n0, sh.partial);
}

// =================================================================================================
// 192 x 192, two workgroups per compute unit, on the 16x16x32 matrix instruction: the tile of the weight
// gradients (short K, where co-resident workgroups hide each other's start and end) at the lower energy per flop
// of this instruction.  Four wavefronts that fetch and compute; each owns 96 x 96 = 6 x 6 blocks, 144
// accumulator registers, and since two workgroups share a SIMD's registers fragments are single buffered as in
// the kernel above: six B fragments refilled in a column-wise tail, A fragments rotating through four register
// sets.  The sets hold rows 0..3 at the start of a k-step and rows 2,3,0,1 of the next at its end, so two k-steps
// (ROT = 0, 2) are unrolled.  One barrier per k-step, placed after the third row: by then every read of the
// current stage has been issued (rows 4, 5 are fetched right after the first two rows), so the barrier frees this
// stage's slot for stage kt+3 and makes stage kt+1 visible for the reads that follow it.
// =================================================================================================
template <typename TL, bool A_KMAJ, bool B_KMAJ, bool COLSUM>
__device__ __forceinline__ void gemm_tile_x16s(const GemmParams& p, int list_pos, char* smem) {
    constexpr int TM = TL::TM, TN = TL::TN, BM = TL::BM, BN = TL::BN, DSTAGES = TL::STAGES;
    constexpr int FM = 2 * TM, FN = 2 * TN, L = TL::LOADS, LH = L / 2;
    static_assert(FM == 6 && DSTAGES == 3 && L % 2 == 0, "row schedule and ring accounting are written for this tile");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const KShare sh = k_share(p, list_pos);
    const i32x4 ra = make_rsrc(p.A, (unsigned)((int64_t)(A_KMAJ ? p.M : p.K) * p.lda * 2));
    const i32x4 rb = make_rsrc(p.B, (unsigned)((int64_t)(B_KMAJ ? p.N : p.K) * p.ldb * 2));
    const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem;
    int tm, tn;
    tile_coords(sh.tile, p.tiles_m, p.tiles_n, p.band, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;

    unsigned offa[TM], offb[TN];
    bool oka[TM], okb[TN];
    int kca, kcb;
    dma_offsets<A_KMAJ, TM, true, true>(offa, oka, kca, p.lda, m0, p.M, wave, lane);
    dma_offsets<B_KMAJ, TN, true, true>(offb, okb, kcb, p.ldb, n0, p.N, wave, lane);
    // MN-major operands: the lane's offset is loop invariant (columns outside the matrix folded in), the k position
    // is the load's scalar offset, and a stage past the end of the K share reads through a descriptor of zero
    // records (everything out of bounds), so such a load costs no vector arithmetic at all.
#pragma unroll
    for (int d = 0; d < TM; ++d) if (!A_KMAJ) offa[d] = oka[d] ? offa[d] : OOB_HALF;
#pragma unroll
    for (int e = 0; e < TN; ++e) if (!B_KMAJ) offb[e] = okb[e] ? offb[e] : OOB_HALF;
    auto dma_one = [&](int slot_off, int s, int d) {              // load d of stage s (of this K share) into its slot
        const unsigned buf = lds0 + (unsigned)slot_off;
        const int k0 = (sh.kt0 + s) * DK;
        if (d < TM) {
            const unsigned dst = buf + (wave_u * TM + d) * 1024;
            if (A_KMAJ) {
                buffer_load_lds_b128(ra, dst, k0 + kca < sh.kend ? offa[d] + (unsigned)k0 * 2u : OOB_OFFSET);
            } else {
                i32x4 r = ra;
                r[2] = k0 < sh.kend ? ra[2] : 0;
                buffer_load_lds_b128_s(r, dst, offa[d], (unsigned)k0 * (unsigned)p.lda * 2u);
            }
        } else {
            const int e = d - TM;
            const unsigned dst = buf + TL::A_BYTES + (wave_u * TN + e) * 1024;
            if (B_KMAJ) {
                buffer_load_lds_b128(rb, dst, k0 + kcb < sh.kend ? offb[e] + (unsigned)k0 * 2u : OOB_OFFSET);
            } else {
                i32x4 r = rb;
                r[2] = k0 < sh.kend ? rb[2] : 0;
                buffer_load_lds_b128_s(r, dst, offb[e], (unsigned)k0 * (unsigned)p.ldb * 2u);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    bf16x8 fa[4], fb[FN];
    // MN-major operands use the xor16 chunk positions and four per-lane base registers (see the kernel above)
    unsigned apos[4], bpos[4];
    {
        const int k0 = 8 * (lane >> 4) + ((lane & 15) >> 2);
        const int x = ((lane >> 3) & 1) | (((lane >> 4) & 1) << 1);
        const unsigned lane_off = (unsigned)(8 * (lane & 1) + 16 * ((lane & 3) >> 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            apos[q] = (unsigned)(k0 * (BM * 2)) + lane_off + 32u * (unsigned)(((q + 2 * wm) & 3) ^ x);
            bpos[q] = (unsigned)(k0 * (BN * 2)) + lane_off + 32u * (unsigned)(((q + 2 * wn) & 3) ^ x);
        }
    }
    auto rd_mn = [&](bf16x8& dst, const char* tile, const unsigned (&pos)[4], int w, int f, int R) {
        const char* src = tile + __builtin_amdgcn_readfirstlane(128 * ((w * 6 + f) >> 2)) + pos[f & 3];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(src + h * 4 * (R * 2)));
            bf16x4 b4 = __builtin_bit_cast(bf16x4, v);
            dst[4 * h + 0] = b4[0]; dst[4 * h + 1] = b4[1]; dst[4 * h + 2] = b4[2]; dst[4 * h + 3] = b4[3];
        }
    };
    auto rd_a = [&](int slot_off, int row, int r) {
        const char* tile = smem + slot_off;
        if (A_KMAJ) fa[r] = dma_frag16<true, BM>(tile, (wm * FM + row) * 16, lane);
        else rd_mn(fa[r], tile, apos, wm, row, BM);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto rd_b = [&](int slot_off, int j) {
        const char* tile = smem + slot_off + TL::A_BYTES;
        if (B_KMAJ) fb[j] = dma_frag16<true, BN>(tile, (wn * FN + j) * 16, lane);
        else rd_mn(fb[j], tile, bpos, wn, j, BN);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mm = [&](int i, int r, int j) {
        mfma16_v(acc[i][j], fa[r], fb[j]);
        __builtin_amdgcn_sched_barrier(0);
    };
    // k-step kt with the A sets rotated by ROT (0 or 2): logical set q is register set (q + ROT) & 3.
    // o0, o1, o2: byte offsets of the ring slots of stages kt, kt+1, kt+2 (stage kt+3 reuses o0).
    // COLSUM: the column sums of B over k (a bias gradient: B = dY, k = tokens) ride along as one more output row.
    // A fragment of ones in place of A makes every row of a 16 x 16 block the sum over the k-step of B's columns, in
    // float on the matrix cores and in k order, a run (CS_RUN) at a time; only the wavefronts that hold the first rows of tile row 0 do it
    // (six more matrix instructions per k-step for them), and they run their own copy of the loop, so the others
    // pay nothing.
    f32x4 cs[COLSUM ? FN : 1];                                    // of the present run
    float cs_runs[COLSUM ? FN : 1], cs_lost[COLSUM ? FN : 1];     // of the runs before
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (bf16_t)1.0f;
#pragma unroll
    for (int j = 0; j < (COLSUM ? FN : 1); ++j) {
        cs_runs[j] = cs_lost[j] = 0.0f;
#pragma unroll
        for (int v = 0; v < 4; ++v) cs[j][v] = 0.0f;
    }
    auto end_run = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < (COLSUM ? FN : 1); ++j) {
            add_carrying(cs_runs[j], cs_lost[j], cs[j][0]);
#pragma unroll
            for (int v = 0; v < 4; ++v) cs[j][v] = 0.0f;
        }
    };
    auto stage = [&](int kt, int o0, int o1, int o2, auto rotc, auto csc) __attribute__((always_inline)) {
        constexpr int ROT = decltype(rotc)::value;
        constexpr bool CS = decltype(csc)::value;
        constexpr int S0 = ROT & 3, S1 = (1 + ROT) & 3, S2 = (2 + ROT) & 3, S3 = (3 + ROT) & 3;
#pragma unroll
        for (int j = 0; j < FN; ++j) {                            // rows 0, 1 column by column
            mm(0, S0, j); mm(1, S1, j);
            // the builtin, not the assembly form: its operands may be set right before it, and then the compiler has to
            // keep the wait states between a vector write and a matrix instruction (a one-step K showed it)
            if constexpr (CS) { cs[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, fb[j], cs[j], 0, 0, 0); __builtin_amdgcn_sched_barrier(0); }
            if (j == 1) dma_one(o2, kt + 2, LH);                  // second half of stage kt+2's loads
            if (j == 3) dma_one(o2, kt + 2, LH + 1);
        }
        rd_a(o0, 4, S0);
        rd_a(o0, 5, S1);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            mm(2, S2, j);
            if (j == 1) dma_one(o2, kt + 2, LH + 2);
        }
        // every read of stage kt has been issued; stage kt+1 has landed once only stage kt+2's loads are in flight
        wait_vmcnt<L>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        rd_a(o1, 0, S2);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            mm(3, S3, j);
            if (j == 2) dma_one(o0, kt + 3, 0);                   // first half of stage kt+3's loads: slot of stage kt
        }
        rd_a(o1, 1, S3);
#pragma unroll
        for (int j = 0; j < FN; ++j) {                            // rows 4, 5 column by column; B refilled when dead
            mm(4, S0, j); mm(5, S1, j);
            rd_b(o1, j);
            if (j == 1) dma_one(o0, kt + 3, 1);
            if (j == 4) dma_one(o0, kt + 3, 2);
        }
        rd_a(o1, 2, S0);
        rd_a(o1, 3, S1);
    };
    static_assert(LH == 3, "three loads before and three after the barrier of a k-step");
    using R0 = std::integral_constant<int, 0>;
    using R2 = std::integral_constant<int, 2>;
    constexpr int SB = TL::STAGE_BYTES;

#pragma unroll
    for (int d = 0; d < L; ++d) dma_one(0, 0, d);
#pragma unroll
    for (int d = 0; d < L; ++d) dma_one(SB, 1, d);
#pragma unroll
    for (int d = 0; d < LH; ++d) dma_one(2 * SB, 2, d);
    wait_vmcnt<L + LH>();                                        // stage 0 has landed
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r) rd_a(0, r, r);
#pragma unroll
    for (int j = 0; j < FN; ++j) rd_b(0, j);
    auto run = [&](auto csc) __attribute__((always_inline)) {
        int kt = 0, o0 = 0, o1 = SB, o2 = 2 * SB;                 // slots of stages kt, kt+1, kt+2 (scalars)
        for (; kt + 1 < sh.nk; kt += 2) {
            stage(kt, o0, o1, o2, R0{}, csc);
            stage(kt + 1, o1, o2, o0, R2{}, csc);
            const int t0 = o0; o0 = o2; o2 = o1; o1 = t0;         // two stages on: (o2, o0, o1)
            if (decltype(csc)::value && kt % CS_RUN == CS_RUN - 2) end_run();
        }
        if (kt < sh.nk) stage(kt, o0, o1, o2, R0{}, csc);
    };
    const bool cs_on = COLSUM && p.colsum && tm == 0 && __builtin_amdgcn_readfirstlane(wm) == 0;    // uniform over the wavefront
    if constexpr (COLSUM) {
        if (cs_on) run(std::true_type{});                         // both copies have one barrier per k-step
        else run(std::false_type{});
    } else {
        run(std::false_type{});
    }
    mfma16_drain();
    if (cs_on && lane < 16) {                                     // lanes 0..15 hold row 0 of each block: columns 0..15
#pragma unroll
        for (int j = 0; j < (COLSUM ? FN : 1); ++j) store_colsum(p, sh, n0 + (wn * FN + j) * 16 + lane, cs_runs[j] + (cs[j][0] - cs_lost[j]));
    }
    wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    epilogue16<TL>(p, acc, smem, wave, lane, m0, n0, sh.partial);
}
template <typename TL, bool A_KMAJ, bool B_KMAJ, bool COLSUM = false>
__global__ __launch_bounds__(256, 2) void gemm_bf16_x16s_kernel(GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    gemm_tile_x16s<TL, A_KMAJ, B_KMAJ, COLSUM>(p, share_of_block(blockIdx.x, gridDim.x), smem);
}

// =================================================================================================
// Several GEMMs in one launch.  The GEMMs of a narrow layer have 10 to 500 tiles of 10 to 60 k-steps each: launched one by
// one, each leaves compute units idle, fills its LDS ring and drains its epilogue with nothing beside it, and costs a
// launch.  The GEMMs of a pass that do not depend on each other (weight gradients, data gradients, both blocks) go out as
// one list of workgroups instead, longest K first.  All use one tile; the layouts of a layer's GEMMs (NN forward, NT data
// gradient, TN weight gradient with the column sums of its B) are three bodies of the same kernel.
// Measured, whole training steps against one launch per GEMM and bias gradient (on two or three chains where the caller
// allows): 198 tokens x 2 of an 832 / 104 shard 156 -> 60 us, BERT-large TP 4 256 -> 166 us, RoBERTa-large TP 2 516 -> 472,
// 3003 tokens of 2560 / 640 548 -> 466, 610 tokens of 10752 / 1344 934 -> 792.  Which tile (the four launches of a step on
// 64 / 128 / 192): 832 / 104 45 / 56 / 81 us, BERT-large 206 / 148 / 179, RoBERTa-large TP 2 669 / 411 / 412, 2560 / 640
// 734 / 452 / 407, the 10B encoder TP 4 2365 / 1393 / 1155.
// =================================================================================================
constexpr int GROUP_MAX = 4;
struct GroupParams {
    GemmParams g[GROUP_MAX];
    int first[GROUP_MAX + 1];      // workgroups [first[i], first[i+1]) compute GEMM i
    int layout[GROUP_MAX];         // 0: NN, 1: NT, 2: TN
    int shares[GROUP_MAX];
    int n;
};
template <typename TL, bool A_KMAJ, bool B_KMAJ, bool COLSUM>
__device__ __forceinline__ void group_tile(const GemmParams& p, int list_pos, char* smem) {
    if constexpr (TL::TM == 3) gemm_tile_x16s<TL, A_KMAJ, B_KMAJ, COLSUM>(p, list_pos, smem);
    else gemm_tile_32<TL, A_KMAJ, B_KMAJ, COLSUM>(p, list_pos, smem);
}
template <typename TL>
__global__ __launch_bounds__(256, 2) void gemm_bf16_group_kernel(GroupParams gp) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int bid = blockIdx.x;
    int i = 0;
    while (i + 1 < gp.n && bid >= gp.first[i + 1]) ++i;
    const GemmParams& p = gp.g[i];
    const int pos = share_of_block(bid - gp.first[i], gp.first[i + 1] - gp.first[i]);
    const int layout = gp.layout[i];
    if (layout == 0) group_tile<TL, true, false, false>(p, pos, smem);
    else if (layout == 1) group_tile<TL, true, true, false>(p, pos, smem);
    else group_tile<TL, false, false, true>(p, pos, smem);
}
// The same on the tiles of gemm_bf16_pp.h, one epilogue behind the three layouts.  Jobs are runs of a GEMM's tiles:
// [first[j], first[j+1]) are the workgroups of job j.
constexpr int JOB_MAX = 2 * GROUP_MAX;
struct PPGroupParams {
    GemmParams g[JOB_MAX];
    PPRun run[JOB_MAX];
    int layout[JOB_MAX], shares[JOB_MAX], first[JOB_MAX + 1];
    int n;
};
template <typename TL>
__global__ __launch_bounds__(512, 2) void gemm_bf16_group_pp_kernel(PPGroupParams gp) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int bid = blockIdx.x;
    int i = 0;
    while (i + 1 < gp.n && bid >= gp.first[i + 1]) ++i;
    const GemmParams& p = gp.g[i];
    const PPWork w = pp_work<TL>(p, gp.run[i], share_of_block(bid - gp.first[i], gp.first[i + 1] - gp.first[i]));
    const int layout = gp.layout[i];
    PPAcc<TL> acc;
    if (layout == 0) pp_products<TL, true, false, false>(p, w, smem, acc);
    else if (layout == 1) pp_products<TL, true, true, false>(p, w, smem, acc);
    else pp_products<TL, false, false, true>(p, w, smem, acc);
    pp_epilogue<TL>(p, acc, w.m0, w.n0, w.partial);
}
// The tiles whose K was cut: a workgroup per 16 rows of a wavefront; [first[j], first[j+1]) are those of job j.
template <typename TL>
__global__ __launch_bounds__(512) void gemm_group_pp_sum_kernel(PPGroupParams gp) {
    const int bid = blockIdx.x;
    int i = 0;
    while (i + 1 < gp.n && bid >= gp.first[i + 1]) ++i;
    const int pos = bid - gp.first[i];
    pp_sum_rows<TL>(gp.g[i], gp.run[i], gp.shares[i], pos / (4 * TL::UA), pos % (4 * TL::UA));
}
// The sums over K shares of all GEMMs of a group that were cut (and of their column sums): GEMM i has the workgroups
// [first[i], first[i+1]) of this launch, 256 chunks of 8 outputs each, the N / 8 chunks of the column sums last.
__global__ __launch_bounds__(256) void gemm_group_sum_kernel(GroupParams gp) {
    const int bid = blockIdx.x;
    int i = 0;
    while (i + 1 < gp.n && bid >= gp.first[i + 1]) ++i;
    const GemmParams& p = gp.g[i];
    const int shares = gp.shares[i];
    const int64_t chunk = (int64_t)(bid - gp.first[i]) * 256 + threadIdx.x, chunks = (int64_t)p.M * p.N / 8;
    if (chunk < chunks) { sum_shares(p, shares, chunk); return; }
    const int64_t col = (chunk - chunks) * 8;
    if (!p.colsum || col >= p.N) return;
    float v8[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int s = 0; s < shares; ++s) {
        float x8[8];
        load8(p.colsum_part + (int64_t)s * p.N + col, x8);
#pragma unroll
        for (int e = 0; e < 8; ++e) v8[e] += x8[e];
    }
    store8(p.colsum + col, v8);
}


bool gemm_bf16_supported(const GemmArgs& a) {
    if (a.dtype != BF16) return false;
    // Only a dimension that is contiguous in memory has to come in whole 16-byte chunks: N (C, bias, an MN-major B), and
    // M or K where an operand is stored with it contiguous.  The rows of an operand may be any number: direct loads of
    // rows past the end read zero, the epilogue checks every row.  So a token count that divides by nothing (M of the
    // forward and data-gradient GEMMs, K of the weight gradients) stays on the matrix cores (against the generic
    // kernel: 100 tokens through the forward of a 12288 / 1536 shard 6.62 -> 0.170 ms; a training step of 3003 tokens at
    // 2560 / 640, attention included, 9.60 -> 3.52 ms).
    if (a.N % 8 || (a.trans_a ? a.M : a.K) % 8 || (a.trans_b && a.K % 8)) return false;
    // 32-bit buffer offsets: operands below 2 GiB
    if (a.M * a.K * 2 >= 0x7FFFFFFFll || a.N * a.K * 2 >= 0x7FFFFFFFll) return false;
    int64_t tiles = ((a.M + 127) / 128) * ((a.N + 127) / 128);
    return tiles < (1 << 24) && a.K < (1 << 24);
}

// Band height of the tile order.  An XCD's L2 (4 MiB) holds no operand panel for long: what it saves is the reuse
// among the tiles in flight on the XCD at one time, which walk K together: `inflight` consecutive tiles of the list =
// h rows x inflight / h columns of the tile grid, needing h A slices and inflight / h B slices per k-step.  The band
// height minimises h * bm + (inflight / h) * bn.  The option gemm_band = h forces a height.
static int choose_band(int R, int bm, int bn, int lds_bytes) {
    if (const int v = options().gemm_band; v > 0) return v;
    // 32 compute units per XCD; the kernels with two workgroups per unit were also measured fastest with the band of
    // 32 tiles in flight (4 rows, 0.6 % of the step ahead of 8), so the count is not doubled for them
    (void)lds_bytes;
    const int inflight = 32;
    int best = 1;
    double best_cost = 1e300;
    for (int h = 1; h <= inflight; h *= 2) {
        const int hh = h < R ? h : R;
        const double cost = (double)hh * bm + (double)inflight / hh * bn;
        if (cost < best_cost) { best_cost = cost; best = hh; }
        if (h >= R) break;
    }
    return best;
}

template <typename TL, bool AK, bool BK_>
static hipError_t launch(GemmParams p, const GemmArgs& a, int shares) {
    static bool attr_set = false;   // raising the dynamic LDS limit is a per-function, one-off call
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_kernel<TL, AK, BK_>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    p.tiles_m = (int)((a.M + TL::BM - 1) / TL::BM);
    p.tiles_n = (int)((a.N + TL::BN - 1) / TL::BN);
    p.band = choose_band(p.tiles_m, TL::BM, TL::BN, TL::LDS_BYTES);
    hipLaunchKernelGGL((gemm_bf16_kernel<TL, AK, BK_>), dim3(p.tiles_m * p.tiles_n * shares), dim3(256),
                       TL::LDS_BYTES, a.stream, p);
    return hipGetLastError();
}

template <typename TL>
static hipError_t launch_layout(const GemmParams& p, const GemmArgs& a, int shares) {
    const bool a_kmaj = !a.trans_a, b_kmaj = a.trans_b;
    if (a_kmaj && b_kmaj) return launch<TL, true, true>(p, a, shares);
    if (a_kmaj && !b_kmaj) return launch<TL, true, false>(p, a, shares);
    if (!a_kmaj && b_kmaj) return launch<TL, false, true>(p, a, shares);
    return launch<TL, false, false>(p, a, shares);
}

template <typename TL, bool AK, bool BK_, bool CS = false>
static hipError_t launch_x16s(GemmParams p, const GemmArgs& a, int shares) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_x16s_kernel<TL, AK, BK_, CS>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    p.tiles_m = (int)((a.M + TL::BM - 1) / TL::BM);
    p.tiles_n = (int)((a.N + TL::BN - 1) / TL::BN);
    p.band = choose_band(p.tiles_m, TL::BM, TL::BN, TL::LDS_BYTES);
    hipLaunchKernelGGL((gemm_bf16_x16s_kernel<TL, AK, BK_, CS>), dim3(p.tiles_m * p.tiles_n * shares), dim3(256),
                       TL::LDS_BYTES, a.stream, p);
    return hipGetLastError();
}
template <typename TL>
static hipError_t launch_x16s_layout(const GemmParams& p, const GemmArgs& a, int shares) {
    const bool a_kmaj = !a.trans_a, b_kmaj = a.trans_b;
    if (a_kmaj && b_kmaj) return launch_x16s<TL, true, true>(p, a, shares);
    if (a_kmaj && !b_kmaj) return launch_x16s<TL, true, false>(p, a, shares);
    if (!a_kmaj && b_kmaj) return launch_x16s<TL, false, true>(p, a, shares);
    if (p.colsum) return launch_x16s<TL, false, false, true>(p, a, shares);
    return launch_x16s<TL, false, false>(p, a, shares);
}

template <typename TL, bool AK, bool BK_>
static hipError_t launch_w8(GemmParams p, const GemmArgs& a, int shares) {
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_x16w8_kernel<TL, AK, BK_>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    p.tiles_m = (int)((a.M + TL::BM - 1) / TL::BM);
    p.tiles_n = (int)((a.N + TL::BN - 1) / TL::BN);
    p.band = choose_band(p.tiles_m, TL::BM, TL::BN, TL::LDS_BYTES);
    hipLaunchKernelGGL((gemm_bf16_x16w8_kernel<TL, AK, BK_>), dim3(p.tiles_m * p.tiles_n * shares), dim3(512),
                       TL::LDS_BYTES, a.stream, p);
    return hipGetLastError();
}
template <typename TL>
static hipError_t launch_w8_layout(const GemmParams& p, const GemmArgs& a, int shares) {
    const bool a_kmaj = !a.trans_a, b_kmaj = a.trans_b;
    if (a_kmaj && b_kmaj) return launch_w8<TL, true, true>(p, a, shares);
    if (a_kmaj && !b_kmaj) return launch_w8<TL, true, false>(p, a, shares);
    if (!a_kmaj && b_kmaj) return launch_w8<TL, false, true>(p, a, shares);
    return launch_w8<TL, false, false>(p, a, shares);
}

template <typename ST, bool AK, bool BK_>
static hipError_t launch_spec(GemmParams p, const GemmArgs& a, int shares) {
    constexpr int LDS = ST::template lds_bytes<AK>();
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_spec_kernel<ST, AK, BK_>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    p.tiles_m = (int)((a.M + ST::BM - 1) / ST::BM);
    p.tiles_n = (int)((a.N + ST::BN - 1) / ST::BN);
    p.band = choose_band(p.tiles_m, ST::BM, ST::BN, LDS);
    hipLaunchKernelGGL((gemm_bf16_spec_kernel<ST, AK, BK_>), dim3(p.tiles_m * p.tiles_n * shares), dim3(512), LDS, a.stream, p);
    return hipGetLastError();
}
template <typename ST, bool BK_>
static hipError_t launch_spec16(GemmParams p, const GemmArgs& a, int shares) {
    constexpr int LDS = ST::template lds_bytes<true>();
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_spec16_kernel<ST, BK_>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    p.tiles_m = (int)((a.M + ST::BM - 1) / ST::BM);
    p.tiles_n = (int)((a.N + ST::BN - 1) / ST::BN);
    p.band = choose_band(p.tiles_m, ST::BM, ST::BN, LDS);
    hipLaunchKernelGGL((gemm_bf16_spec16_kernel<ST, BK_>), dim3(p.tiles_m * p.tiles_n * shares), dim3(512), LDS, a.stream, p);
    return hipGetLastError();
}
template <typename ST>
static hipError_t launch_spec_layout(const GemmParams& p, const GemmArgs& a, int shares) {
    const bool a_kmaj = !a.trans_a, b_kmaj = a.trans_b;
    if (a_kmaj && b_kmaj) return launch_spec<ST, true, true>(p, a, shares);
    if (a_kmaj && !b_kmaj) return launch_spec<ST, true, false>(p, a, shares);
    if (!a_kmaj && b_kmaj) return launch_spec<ST, false, true>(p, a, shares);
    return launch_spec<ST, false, false>(p, a, shares);
}

// Tile variants.  The host launches the one with the least estimated time
//   (tiles per compute unit, rounded up) x (k-stages) x (time per stage) + (per-tile fixed cost),
// with per-stage times measured on 8192^3 GEMMs.  The fixed cost (pipeline fill, and an epilogue that
// is bandwidth-bound because a round's workgroups all reach it together) is paid per round by the
// variants that fit one workgroup per compute unit and once by those that fit two (192 x 192 and
// 128 x 128), whose co-resident workgroups overlap each other's fill and epilogue.  So long-K GEMMs
// with few tiles prefer the big tiles, short-K weight gradients the co-resident ones, and a GEMM
// whose 256 x 256 tile count fills the last round badly a shape that divides better.
int compute_units() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        cus = (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
                  ? prop.multiProcessorCount : 256;
    }
    return cus;
}

constexpr int NVARIANTS = 8;
constexpr int MAX_SHARES = 16;
struct Plan { int variant, shares, nk_share; double us; };

// Splitting K.  A GEMM with few output tiles and a long K (the data gradient of a narrow projection: N = 1536,
// K = 12288 ... 49152) leaves compute units idle or gives each a very long serial K walk.  Its K range is then
// cut into `shares` equal runs of k-steps, one workgroup per (tile, share); every workgroup writes its float
// partial sums to the workspace and a second kernel adds the shares in share order and applies the epilogue,
// so the result does not depend on scheduling.  The estimate charges that second pass with its memory traffic.
static Plan make_plan(int64_t M, int64_t N, int64_t K, bool a_kmaj, bool b_kmaj) {
    // variant 5: 256 x 192 on 8 wavefronts and the 16x16x32 instruction; 6: fetch and math wavefronts on 16x16x32;
    // 7: 192 x 192, two workgroups per compute unit, on 16x16x32
    static const int bm[NVARIANTS] = {256, 256, 128, 192, 256, 256, 256, 192};
    static const int bn[NVARIANTS] = {256, 192, 128, 192, 192, 192, 192, 192};
    static const int wgs_per_cu[NVARIANTS] = {1, 1, 2, 2, 1, 1, 1, 2};
    static const double us_per_stage[NVARIANTS] = {0.92, 0.758, 0.348, 0.5576, 0.658, 0.70, 0.602, 0.509};
    static const double fixed_us[NVARIANTS] = {12.0, 12.0, 12.0, 12.0, 18.0, 12.5, 18.0, 12.0};
    // tuning / test overrides (Options): one variant for every GEMM, a K split, or plans of single shapes
    const Options& opt = options();
    int forced_v = (opt.gemm_tile >= 0 && opt.gemm_tile < NVARIANTS) ? opt.gemm_tile : -1;
    int forced_s = opt.gemm_shares;
    // gemm_force = "MxNxK@ab=v[:shares];..." (a, b = 1 if A, B is K-major) overrides the plan of single shapes (tuning inside a whole step)
    int forced_shape_v = -1;
    if (opt.gemm_force[0]) {
        const char* q = opt.gemm_force;
        while (*q) {
            long long m = 0, n = 0, k = 0; int ak = 0, bk = 0, v = -1, sh = 0, used = 0;
            if (sscanf(q, "%lldx%lldx%lld@%1d%1d=%d%n", &m, &n, &k, &ak, &bk, &v, &used) >= 6) {   // @ab: A, B K-major
                const char* r = q + used;
                if (*r == ':') sh = atoi(r + 1);
                if (m == M && n == N && k == K && (ak != 0) == a_kmaj && (bk != 0) == b_kmaj && v >= 0 && v < NVARIANTS) {
                    forced_shape_v = v;
                    if (sh > 0) forced_s = sh;
                }
            }
            while (*q && *q != ';') ++q;
            if (*q == ';') ++q;
        }
    }
    if (forced_shape_v >= 0) forced_v = forced_shape_v;
    const int cus = compute_units();
    const int nk = (int)((K + DK - 1) / DK);
    Plan best{0, 1, nk, 0.0};
    double best_c = -1;
    for (int v = 0; v < NVARIANTS; ++v) {
        if (forced_v >= 0 && v != forced_v) continue;
        // the variant with fetch-only wavefronts is built for a K-major A (its MN-major A path spills)
        if (forced_v < 0 && v == 4 && !a_kmaj) continue;
        if (v == 6 && !a_kmaj) continue;              // written for a K-major A only
        // the two-per-CU 16x16x32 tile is the weight-gradient kernel (MN-major A); with a K-major A it pays when K is
        // short (co-resident workgroups hide each other's start and end: the out-projection, K = 1536, -30 us per
        // forward pass against the 8-wavefront variant) or when many rounds of tiles amortise its cold starts; on the
        // long-K forward and data-gradient GEMMs it is 2-5 % slower per step (all measured inside the layer step by
        // forcing single shapes with TPL_GEMM_FORCE, not in isolated loops); the same holds for its 32x32x16 sibling,
        // variant 3 (config 4's out-projection data gradient: -1.2 % of the step without it)
        if (forced_v < 0 && (v == 7 || v == 3) && a_kmaj && nk > 64 &&
            ((M + bm[v] - 1) / bm[v]) * ((N + bn[v] - 1) / bn[v]) < 4 * compute_units()) continue;
        // with an MN-major B its 20 fragment reads per k-step hold up the matrix instructions: no gain there
        if (forced_v < 0 && v == 6 && !b_kmaj) continue;
        // the 8-wavefront variant was measured against the others on K-major A only (forward, data gradients)
        if (forced_v < 0 && v == 5 && !a_kmaj) continue;
        const int64_t tiles = ((M + bm[v] - 1) / bm[v]) * ((N + bn[v] - 1) / bn[v]);
        for (int want = 1; want <= MAX_SHARES; ++want) {
            if (forced_s > 0 && want != (forced_s < MAX_SHARES ? forced_s : MAX_SHARES)) continue;
            if (forced_s <= 0 && want > 1 && (tiles * (want - 1) >= cus || nk / want < 48 || v == 5)) break;
            int per = (nk + want - 1) / want;
            if (v == 4 || v == 6) per = (per + 1) & ~1;          // its wide A slots hold two k-steps: shares start on even steps
            const int shares = (nk + per - 1) / per;
            if (forced_s <= 0 && shares != want) continue;   // the same plan as a smaller `want`
            const double per_cu = (double)((tiles * shares + cus - 1) / cus);
            double c = per_cu * per * us_per_stage[v] + fixed_us[v] * (wgs_per_cu[v] == 1 ? per_cu : 1.0);
            if (shares > 1) c += 6.0 + (double)M * N * (8.0 * shares + 2.0) / 3.0e6;   // second pass at ~3 TB/s
            // single GEMMs of a pass run on two chains, and one that takes (nearly) every compute unit leaves none to the kernels
            // of the other: inside such a step the out-projection data gradient is fastest with 3 shares (192 workgroups), 0.8 %
            // of the step ahead of 4 (256 workgroups)
            if (shares > 1 && tiles * shares * 4 > (int64_t)cus * 3) c *= 1.10;
            if (best_c < 0 || c < best_c) { best = Plan{v, shares, per, c}; best_c = c; }
        }
    }
    return best;
}

// Plans that were made, by a key of whole numbers, so that a call looks its plans up and does not run the planner.  A table of
// SETS x 4 entries, the oldest of a set replaced; shared by all threads.
template <typename Plan, int KEY, int SETS>
class PlanCache {
public:
    template <typename Make>
    Plan get(const int64_t (&key)[KEY], Make make) {
        uint64_t h = 0;
        for (const int64_t k : key) h = (h ^ (uint64_t)k) * 0x9E3779B97F4A7C15ull, h ^= h >> 29;
        Set& set = sets[h % SETS];
        {
            std::lock_guard<std::mutex> lock(mu);
            for (int i = 0; i < set.used; ++i)
                if (std::equal(key, key + KEY, set.entry[i].key)) return set.entry[i].plan;
        }
        const Plan plan = make();                                // outside the lock: another thread's plan is the same
        std::lock_guard<std::mutex> lock(mu);
        Entry& e = set.entry[set.used < WAYS ? set.used++ : set.next++ % WAYS];
        std::copy(key, key + KEY, e.key);
        e.plan = plan;
        return plan;
    }

private:
    static constexpr int WAYS = 4;
    struct Entry { int64_t key[KEY]; Plan plan; };
    struct Set { Entry entry[WAYS]; int used; unsigned next; };
    std::mutex mu;
    Set sets[SETS] = {};
};

// Entries carry the generation of the options they were planned under.
static Plan plan_for(int64_t M, int64_t N, int64_t K, bool a_kmaj, bool b_kmaj) {
    static PlanCache<Plan, 5, 256> cache;
    const int64_t key[5] = {M, N, K, (a_kmaj ? 1 : 0) | (b_kmaj ? 2 : 0), (int64_t)options().generation};
    return cache.get(key, [&] { return make_plan(M, N, K, a_kmaj, b_kmaj); });
}

static GemmParams gemm_params(const GemmArgs& a) {
    GemmParams p{};
    p.A = (const bf16_t*)a.A; p.B = (const bf16_t*)a.B; p.C = (bf16_t*)a.C;
    p.bias = (const bf16_t*)a.bias; p.resid = (const bf16_t*)a.resid; p.aux = (bf16_t*)a.aux;
    p.M = (int)a.M; p.N = (int)a.N; p.K = (int)a.K;
    p.nt_store = a.c_streaming ? 1 : 0;
    p.lda = a.trans_a ? (int)a.M : (int)a.K;
    p.ldb = a.trans_b ? (int)a.K : (int)a.N;
    p.epi = a.epi;
    p.tiles_m = p.tiles_n = 0;
    p.band = 8;
    p.nk_total = (int)((a.K + DK - 1) / DK);
    return p;
}

// ---- groups ------------------------------------------------------------------------------------------------------------
// One tile for the whole group and K shares per GEMM, by a time estimate.  A launch takes as long as its units have work
// (k-steps of all workgroups, a start and an epilogue per workgroup) or as its longest workgroup runs by itself, whichever
// is more; K shares shorten the longest ones and cost the partial sums' traffic and a launch.  Against the measured times of
// 24 groups of 6 layers on each tile the estimate is off by 15 % root mean square: up to 28 % too long for the widest layers
// (10B encoder, GPT-3 13B), up to 28 % too short for the narrowest (832 / 104), the three tiles of a group mostly alike: the
// tile with the least estimate is the fastest of the three on 23 of the 24 and 6 % behind on one.
// The tiles of gemm_bf16_pp.h take a compute unit each, so a launch is its list dealt out to the units (list_time); 8 to 12 %
// root mean square off over 56 groups of 14 layers.  Whole steps on 256 x 256 / 256 x 128 / the best of the smaller tiles, us:
// RoBERTa-large TP 2 437 / 486 / 482, 2560 / 640 at 3003 tokens 450 / 488 / 481, the 10B encoder TP 4 1300 / 1480 / 1490, GPT-3
// 13B TP 4 1740 / 1990 / 1930, 175B TP 8 2240 / 2625 / 2615; few tiles: BERT-large TP 4 183 / 159 / 162, 3072 / 768 at 1500 tokens
// 326 / 313 / 320, 4096 tokens of 768 / 768 329 / 315 / 316 (each launch on its own tile: 308).
namespace {
struct GroupTile { int option, bm, bn; bool turns; double step_us, wg_us, base_us, alone_us, alone_base_us, gelu_us; };
constexpr GroupTile GROUP_TILES[] = {{256, 256, 256, true, 0.72, 8.0, 0, 0, 0, 4.5}, {384, 256, 128, true, 0.42, 7.5, 0, 0, 0, 2.5},
                                     {512, 128, 256, true, 0.55, 7.5, 0, 0, 0, 2.5},
                                     {192, 192, 192, false, 0.60, 2.6, 13.0, 0.77, 4.5, 0}, {128, 128, 128, false, 0.355, 1.0, 7.5, 0.38, 4.5, 0}, {64, 64, 64, false, 0.143, 0.92, 4.5, 0.35, 2.1, 0}};
// 128 x 256 by turns is for groups of at most 128 rows and no weight gradient (the forward of few tokens): no row of tiles is multiplied that
// does not exist, and twice the weights of 256 x 128 are in flight per unit; on more rows it is the slower half tile (860 tokens of 3456 / 1728
// recomputed 512 -> 551, 572 of 5120 / 1280 374 -> 386).  It takes the place of the tile that is chosen otherwise where it leads it, see takes_wide_tile.
constexpr int WIDE_TILE = 2, FEW_TOKENS = 128;
static_assert(GROUP_TILES[WIDE_TILE].turns && GROUP_TILES[WIDE_TILE].bm == FEW_TOKENS && GROUP_TILES[WIDE_TILE].bn == 256, "the tile of few rows");
constexpr int GROUP_TILE_COUNT = sizeof(GROUP_TILES) / sizeof(GROUP_TILES[0]);
// Operands and results of a launch of few rows, streamed: 100 tokens through the forward of a 12288 / 1536 shard (453 MB) take
// 150 us on 128 x 128 tiles, 137 on 256 x 256, which have twice the loads in flight.
constexpr double MEM_BYTES_PER_US = 4.2e6, MEM_BYTES_PER_US_SMALL = 3.5e6;
// Up to FEW_ROWS rows there is one row of tiles on any tile, and every column of tiles reads A again beside the weights that stream; that
// ranks the small tiles, not their K shares.  By the k-steps alone narrow tiles were chosen at 33 to 64 rows: forward with weights from
// memory, us, 4096 / 1024 33 / 48 / 64 tokens 51.8 / 56.4 / 61.1, now 46.3 / 49.0 / 48.1; 4992 / 1248 56 / 59 / 63 and 54.5 / 56.3 / 58.8; 8192 /
// 1024 70 / 71 / 77 and 60 / 62 / 69.  The rate is the highest with which the choice at 33 tokens of 4096 / 1024 is right.
constexpr double AGAIN_BYTES_PER_US = 4.7e6;
constexpr int FEW_ROWS = 64;
// Groups with weight gradients go to the tiles by turns where these are estimated this much faster, unless the list goes out uncut, one
// workgroup to a unit.  Few tokens make tiles of few k-steps that are all start and epilogue, and small groups many K shares; where a
// workgroup has its unit to itself nothing covers those: the estimate of 256 x 256 is 3 to 9 % short there, those of 128 and 192 3 to 14 %
// long (forward: level).  Over 480 launches of 240 layers (16 to 8192 tokens, weights in cache and from memory) the chosen tile took 3.5 %
// longer than the fastest, and 5 % or more longer than the fastest small tile on 102; with this 1.4 %, and on 36.  Backward of 273 tokens of
// 2688 / 672 85 us, now 73; 476 of 1632 / 1632 133 and 126.
constexpr double TURNS_LEAD = 1.12;
constexpr int PP_MIN_STEPS = 12;               // k-steps of a K share
struct PPJob { int gemm, tile0, count, nk, shares; };
struct GroupPlan { int tile, nk[GROUP_MAX], shares[GROUP_MAX]; double us; int njobs; PPJob job[JOB_MAX]; };   // jobs: tiles by turns only

int64_t group_tiles(const GemmArgs& a, const GroupTile& t) { return ((a.M + t.bm - 1) / t.bm) * ((a.N + t.bn - 1) / t.bn); }

// How long `units` machines take for a list of jobs dealt out in order, count[i] of length len[i] each (longest first); at least
// `limit`, not to the end, where it is not below that.
double list_time(int units, int n, const int64_t* count, const double* len, double limit) {
    struct Free { double t; int64_t c; } old[64], now[64];         // units by the time at which they are free, earliest first
    int m = 1;
    old[0] = {0.0, units};
    double end = 0.0;
    for (int i = 0; i < n; ++i) {
        int64_t left = count[i];
        const int64_t rounds = left / units;                      // whole rounds move every unit alike
        if (rounds > 2) {
            for (int q = 0; q < m; ++q) old[q].t += (double)(rounds - 2) * len[i];
            left -= (rounds - 2) * units;
        }
        // Units that take one are free len[i] later, in the order in which they took it: a queue beside that of the others.
        int o = 0, h = 0, r = 0;                                  // heads of `old` and `now` (a ring), entries of `now`
        while (left > 0) {
            Free& f = r == 0 || (o < m && old[o].t <= now[h & 63].t) ? old[o] : now[h & 63];
            const bool from_old = &f >= old && &f < old + 64;
            const int64_t c = std::min(left, f.c);
            const double t = f.t + len[i];
            if (t >= limit) return t;
            end = std::max(end, t);
            left -= c;
            if (c < f.c && m - o + r < 64) f.c -= c;
            else if (from_old) ++o;
            else { ++h; --r; }
            now[(h + r++) & 63] = {t, c};
        }
        if (i + 1 == n) break;
        Free both[64];
        int k = 0;
        while (o < m || r > 0) {
            if (r == 0 || (o < m && old[o].t <= now[h & 63].t)) both[k++] = old[o++];
            else { both[k++] = now[h++ & 63]; --r; }
        }
        std::copy(both, both + k, old);
        m = k;
    }
    return end;
}

// Tiles of gemm_bf16_pp.h, one workgroup per compute unit: the last round of a list that does not fill it is cut.  Of each GEMM `cut`
// tiles, its last ones, go out in `shares` K shares each; the plan is the best found by changing one GEMM at a time.  Not searched for
// (us infinite) where the work of the uncut list alone, which no cut takes down, is not below `limit`.
GroupPlan make_pp_plan(const GemmArgs* g, int n, const GroupTile& gt, double limit) {
    const int cus = compute_units();
    struct Cut { int64_t cut; int shares, nk; };
    int64_t tiles[GROUP_MAX];
    int nk[GROUP_MAX];
    double tile_bytes[GROUP_MAX], floor_us = 0;
    for (int i = 0; i < n; ++i) {
        tiles[i] = group_tiles(g[i], gt);
        nk[i] = (int)((g[i].K + DK - 1) / DK);
        tile_bytes[i] = (double)g[i].M * g[i].N / (double)tiles[i];
        floor_us += 2.0 * ((double)g[i].M * g[i].K + (double)g[i].N * g[i].K + (double)g[i].M * g[i].N) / MEM_BYTES_PER_US;
    }
    auto with_shares = [&](int i, int64_t cut, int want) {
        Cut c{cut, 1, nk[i]};
        if (want > 1) {
            c.nk = ((nk[i] + want - 1) / want + 1) & ~1;              // two k-steps at a time
            c.shares = (nk[i] + c.nk - 1) / c.nk;
        }
        if (c.shares == 1) c.cut = 0;
        return c;
    };
    auto jobs = [&](const Cut* c, PPJob* job) {                       // longest first, else in order
        int m = 0;
        auto add = [&](const PPJob& j) {
            int q = m++;
            for (; q > 0 && job[q - 1].nk < j.nk; --q) job[q] = job[q - 1];
            job[q] = j;
        };
        for (int i = 0; i < n; ++i) {
            if (tiles[i] > c[i].cut) add(PPJob{i, 0, (int)(tiles[i] - c[i].cut), nk[i], 1});
            if (c[i].cut) add(PPJob{i, (int)(tiles[i] - c[i].cut), (int)c[i].cut, c[i].nk, c[i].shares});
        }
        return m;
    };
    auto length = [&](int i, int steps, bool whole) { return steps * gt.step_us + gt.wg_us + (whole && g[i].epi != EPI_NONE ? gt.gelu_us : 0.0); };
    // What a plan cannot take less than, GEMM by GEMM: its longest job and its work over all units, unless list_time takes whole rounds of a
    // job at once behind longer ones (it may come out below the work then), and the sums of the shares.
    struct Bound {
        double work = 0, longest = 0, bytes = 0, many = INFINITY;
        void add(int64_t count, double len, int units) {
            work += (double)count * len;
            longest = std::max(longest, len);
            if (count >= 3 * units) many = std::min(many, len);
        }
    };
    auto add_gemm = [&](Bound& b, int i, const Cut& c) {
        if (tiles[i] > c.cut) b.add(tiles[i] - c.cut, length(i, nk[i], true), cus);
        if (!c.cut) return;
        b.add(c.cut * c.shares, length(i, c.nk, false), cus);
        b.bytes += (double)c.cut * tile_bytes[i] * (8.0 * c.shares + 2.0);
    };
    auto sums = [&](const Bound& b) { return b.bytes > 0 ? 4.2 + b.bytes / 8.0e6 : 0.0; };
    auto least = [&](const Bound& b) {
        return (std::max(std::max(b.many < b.longest ? 0.0 : b.work / cus, b.longest), floor_us) + sums(b)) * (1 - 1e-12);
    };
    // The list dealt out; where that is not below `limit`, anything that is not either.
    auto estimate = [&](const Cut* c, double limit) {
        Bound b;
        for (int i = 0; i < n; ++i) add_gemm(b, i, c[i]);
        PPJob job[JOB_MAX];
        int64_t count[JOB_MAX];
        double len[JOB_MAX];
        const int m = jobs(c, job);
        for (int q = 0; q < m; ++q) {
            count[q] = (int64_t)job[q].count * job[q].shares;
            len[q] = length(job[q].gemm, job[q].nk, job[q].shares == 1);
        }
        return std::max(list_time(cus, m, count, len, limit - sums(b) + 1e-6), floor_us) + sums(b);
    };
    Cut best[GROUP_MAX], now[GROUP_MAX];
    Bound uncut;
    for (int i = 0; i < n; ++i) {
        best[i] = now[i] = with_shares(i, 0, 1);
        add_gemm(uncut, i, best[i]);
    }
    // list_time may come out a little below the work, and far below where long jobs are followed by rounds of much shorter ones
    if (std::max(uncut.many < 0.4 * uncut.longest ? 0.0 : 0.98 * uncut.work / cus, floor_us) >= limit) {
        GroupPlan none{};
        none.us = INFINITY;
        return none;
    }
    double best_us = estimate(best, INFINITY);
    const int longest = *std::max_element(nk, nk + n);
    for (int parts = 2; parts <= MAX_SHARES && longest / parts >= PP_MIN_STEPS; ++parts) {   // everything long cut to one length
        for (int i = 0; i < n; ++i) now[i] = with_shares(i, tiles[i], std::max(1, (nk[i] * parts + longest - 1) / longest));
        const double us = estimate(now, best_us);
        if (us < best_us) { best_us = us; std::copy(now, now + n, best); }
    }
    struct Try { int gemm; Cut c; double least; };
    Try tries[GROUP_MAX * MAX_SHARES * 9];
    for (int round = 0; round < 2 * n; ++round) {                 // the best change of one GEMM, the first of equals
        int m = 0, first = 0, chosen = -1;
        for (int i = 0; i < n; ++i) {
            int64_t others = 0;
            Bound rest;
            for (int q = 0; q < n; ++q) {
                others += q == i ? tiles[q] : tiles[q] - best[q].cut;
                if (q != i) add_gemm(rest, q, best[q]);
            }
            int last_nk = 0;
            for (int want = 1; want <= MAX_SHARES && (want == 1 || nk[i] / want >= PP_MIN_STEPS); ++want) {
                Cut c = with_shares(i, tiles[i], want);
                if (c.nk == last_nk) continue;                    // no other plan than with fewer wanted
                last_nk = c.nk;
                int64_t last_cut = -1;
                // the tiles past whole rounds, or so many eighths; all of one GEMM, and of 128 x 256, whose lists go out in one round
                for (int eighth = n == 1 || gt.bm == FEW_TOKENS ? 8 : 0; eighth <= 8; ++eighth) {
                    const int64_t cut = eighth ? (tiles[i] * eighth + 7) / 8 : std::min(tiles[i], others % cus);
                    if (cut == last_cut) continue;
                    last_cut = cut;
                    c.cut = c.shares > 1 ? cut : 0;
                    Bound b = rest;
                    add_gemm(b, i, c);
                    tries[m] = Try{i, c, least(b)};
                    if (tries[m].least < best_us) {
                        if (tries[m].least < tries[first].least) first = m;
                        ++m;
                    }
                    if (want == 1) break;
                }
            }
        }
        std::copy(best, best + n, now);
        double us = best_us;
        auto consider = [&](int t) {
            if (tries[t].least > us) return;
            now[tries[t].gemm] = tries[t].c;
            const double it = estimate(now, us * (1 + 1e-12));
            if (it < us || (it == us && t < chosen)) { us = it; chosen = t; }
            now[tries[t].gemm] = best[tries[t].gemm];
        };
        if (m) consider(first);                                   // most of the others can then be left out
        for (int t = 0; t < m; ++t) if (t != first) consider(t);
        if (chosen < 0) break;
        best_us = us;
        best[tries[chosen].gemm] = tries[chosen].c;
    }
    GroupPlan p{};
    p.us = best_us;
    p.njobs = jobs(best, p.job);
    return p;
}

// The best of the tiles of this file that `forced` allows (us < 0: none): *beside is what it is put at beside the tiles by turns.  Where
// all workgroups of a launch run at once, one to a unit, or two on 128 x 128 uncut, the estimate that ranks these tiles among
// each other is up to 6 us too long (no round has to end before the next begins), and groups went to tiles by turns that were slower.
// There they are compared by the workgroups of the fullest unit.  us, 256 x 128 by turns and 128 x 128: 160 tokens of 2048 / 1024
// {up, qkv} 23.8 and 19.7, 200 and 300 of 3072 / 768 27 and 22.7, 31.6 and 26.7, {down, out} of 400 tokens of 2560 / 640 25.7 and 20.9,
// of 2048 of 1024 / 512 25.6 and 21.2.  Of 1650 groups of 18 layers (1 to 8192 tokens) it changes 2 %: 0.4 % less time over all of
// them, 27 more than 8 % faster, 3 more than 8 % slower.
GroupPlan make_small_plan(const GemmArgs* g, int n, int forced, double* beside) {
    const int cus = compute_units();
    double operands = 0;
    for (int i = 0; i < n; ++i) operands += 2.0 * ((double)g[i].M * g[i].K + (double)g[i].N * g[i].K + (double)g[i].M * g[i].N);
    GroupPlan best{};
    best.us = -1;
    double best_rank = 0;
    for (int t = 0; t < GROUP_TILE_COUNT; ++t) {
        const GroupTile& gt = GROUP_TILES[t];
        if (gt.turns || (forced > 0 && forced != gt.option)) continue;
        GroupPlan p{};
        p.tile = t;
        int64_t tiles[GROUP_MAX];
        int nk[GROUP_MAX];
        for (int i = 0; i < n; ++i) {
            tiles[i] = group_tiles(g[i], gt);
            nk[i] = p.nk[i] = (int)((g[i].K + DK - 1) / DK);
            p.shares[i] = 1;
        }
        double again_us = 0;
        for (int i = 0; i < n; ++i) again_us = g[i].M <= FEW_ROWS ? again_us + 2.0 * g[i].M * g[i].K * (tiles[i] - 1) / AGAIN_BYTES_PER_US : -INFINITY;
        double at_once = 0;                                       // estimate of a launch whose workgroups all run at once, see below
        auto estimate = [&]() {
            double work = 0, wgs = 0, longest = 0, bytes = 0;
            for (int i = 0; i < n; ++i) {
                wgs += (double)tiles[i] * p.shares[i];
                work += (double)tiles[i] * p.shares[i] * p.nk[i];
                longest = std::max(longest, (double)p.nk[i]);
                if (p.shares[i] > 1) bytes += (double)g[i].M * g[i].N * (8.0 * p.shares[i] + 2.0);
            }
            const double sums = bytes > 0 ? 4.2 : 0.0;
            const double us = std::max(operands / MEM_BYTES_PER_US_SMALL, std::max((work * gt.step_us + wgs * gt.wg_us) / cus + gt.base_us,
                                                                                   longest * gt.alone_us + gt.alone_base_us));
            at_once = 0;
            if (gt.bm >= 128 && wgs <= (gt.bm == 128 && bytes == 0 ? 2 * cus : cus)) {
                int second = 0;                                   // longest first: the k-steps of the workgroup that shares a unit with the longest
                for (int i = 0; i < n; ++i) {
                    double before = 0;                            // workgroups not shorter than those of GEMM i
                    for (int q = 0; q < n; ++q) if (p.nk[q] >= p.nk[i]) before += (double)tiles[q] * p.shares[q];
                    if (before > cus) second = std::max(second, p.nk[i]);
                }
                at_once = std::max(longest * gt.alone_us + 2.5, operands / 4.8e6);
                if (second) at_once = std::max(at_once, (longest + second) * gt.step_us + 2 * gt.wg_us + 2.0);
                at_once += sums + bytes / 1.0e7;
            }
            return us + sums + bytes / 1.6e7;
        };
        GroupPlan mine{};                                         // the best on this tile
        mine.us = -1;
        double mine_beside = 0;
        auto keep = [&]() {
            if (mine.us >= 0 && p.us >= mine.us) return;
            mine = p;
            mine_beside = at_once > 0 ? std::min(at_once, p.us) : p.us;
        };
        p.us = estimate();
        for (int cuts = 0; cuts < 16; ++cuts) {                   // cut the longest again while that helps
            int l = 0;
            for (int i = 1; i < n; ++i) if (p.nk[i] > p.nk[l]) l = i;
            const int want = p.shares[l] + 1;
            if (want > MAX_SHARES || nk[l] / want < 12) break;
            keep();              // one cut alone may not pay while the next does (two GEMMs of the same length): the best seen
            p.nk[l] = (nk[l] + want - 1) / want;
            p.shares[l] = (nk[l] + p.nk[l] - 1) / p.nk[l];
            p.us = estimate();
        }
        keep();
        const double rank = std::max(mine.us, operands / MEM_BYTES_PER_US_SMALL + again_us);
        if (best.us >= 0 && rank >= best_rank) continue;
        best = mine;
        best_rank = rank;
        *beside = mine_beside;
    }
    return best;
}

// Time of a group of few rows on a plan of a tile by turns, weights from memory.  A k-step is as long as its rows take and as its bytes do:
// {us of a k-step without rows, what 128 rows add, bytes per us of the chip}; the two do not quite hide each other, hence the fourth powers.  The
// sums read share after share.  Fitted to 847 launches of 280 groups (8 to 128 rows, 256 / 32 to 12288 / 12288): 4.5 % root mean square off,
// where the estimate of make_pp_plan, which ranks the plans of a tile, is 9 to 11.
double few_rows_us(const GemmArgs* g, int n, const GroupPlan& p) {
    struct Rate { double step_us, rows_us, bytes_per_us; };
    constexpr Rate RATES[] = {{0.37, 0.19, 6.0e6}, {0.23, 0.11, 5.5e6}, {0.235, 0.175, 5.9e6}};
    static_assert(sizeof(RATES) / sizeof(RATES[0]) == WIDE_TILE + 1, "in the order of GROUP_TILES");
    constexpr double WG_US = 11.2, START_US = 6.6, SHARE_US = 0.25, SUM_BYTES_PER_US = 3.6e6;
    const Rate& r = RATES[p.tile];
    double mem_us = START_US, sums_us = 0, len[JOB_MAX];
    int64_t count[JOB_MAX];
    int shares = 0;
    for (int i = 0; i < n; ++i) mem_us += 2.0 * ((double)g[i].M * g[i].K + (double)g[i].N * g[i].K + (double)g[i].M * g[i].N) / r.bytes_per_us;
    for (int j = 0; j < p.njobs; ++j) {
        const PPJob& job = p.job[j];
        const int64_t rows = g[job.gemm].M;
        count[j] = (int64_t)job.count * job.shares;
        len[j] = job.nk * (r.step_us + r.rows_us * (double)rows / FEW_TOKENS) + WG_US;
        if (job.shares == 1) continue;
        shares = std::max(shares, job.shares);
        sums_us += (double)count[j] * (4.0 * ((rows + 15) / 16 * 16) * GROUP_TILES[p.tile].bn) / SUM_BYTES_PER_US;
    }
    const double list_us = list_time(compute_units(), p.njobs, count, len, INFINITY);
    return std::sqrt(std::sqrt(std::pow(list_us, 4) + std::pow(mem_us, 4))) + sums_us + shares * SHARE_US;
}
// Whether a group goes out on `wide` (128 x 256) instead of `other`, put at `other_us` by the estimates that chose it.  Only in one round: the
// few workgroups of a second one request little of what memory could give (8 rows of {up, qkv} of 11840 / 11840, 324 workgroups, 349 us on 256 x 256
// and 380); and of at least nine sixteenths of the units, for the same reason (80 rows of {up, qkv} of 4816 / 4816, 133 workgroups, 91.0 and 99.6, 32 of
// 10304 / 5152, 142, 151 and 161).  Only where the rows of B of the largest GEMM are whole cache lines: where a unit's loads straddle lines this tile
// loses far more than 256 x 256 (64 rows of {down, out} of 8944 / 8944 on 256 x 256 and this 152 and 180 us, of 8960 / 8960 145 and 148; 48 of 6432 / 6432
// 86 and 100).  Against tiles by turns a lead of 3.5 %; the small tiles, put at up to 25 % more than they take where rows are few, need one of 25 %.
// Of 547 groups, weights from memory, 74 go out on it; they take 10 % less time than without the tile, up to 43 %, two of them more than 2 % more (2.2
// and 2.6).  By make_pp_plan's estimates alone, in place of 256 x 128, 29 of 262 did (8 rows of {down, out} of 3136 / 3136 26.9 and 30.2 us, forward of 2
// tokens of 3648 / 1824 52 and 58).  100 tokens of 12288 / 1536, {up, qkv} and {down, out} without the sums of their shares: 256 x 128 69 and 68 us,
// 256 x 256 65 and 51, this 61 and 43.
bool takes_wide_tile(const GemmArgs* g, int n, const GroupPlan& wide, const GroupPlan& other, double other_us) {
    const GemmArgs& largest = *std::max_element(g, g + n, [](const GemmArgs& a, const GemmArgs& b) { return a.N * a.K < b.N * b.K; });
    if ((largest.trans_b ? largest.K : largest.N) % 64 != 0) return false;
    int64_t workgroups = 0;
    for (int j = 0; j < wide.njobs; ++j) workgroups += (int64_t)wide.job[j].count * wide.job[j].shares;
    if (workgroups > compute_units() || workgroups * 16 < compute_units() * 9) return false;
    return few_rows_us(g, n, wide) < (GROUP_TILES[other.tile].turns ? few_rows_us(g, n, other) / 1.035 : other_us / 1.25);
}

GroupPlan make_group_plan(const GemmArgs* g, int n) {
    const int forced = n == 1 ? 256 : options().gemm_group;       // one GEMM: see by_turns
    double us = INFINITY;
    GroupPlan best = make_small_plan(g, n, forced, &us);
    const bool weight_grads = std::any_of(g, g + n, [](const GemmArgs& a) { return a.trans_a != 0; });
    for (int t = 0; t < GROUP_TILE_COUNT; ++t) {
        const GroupTile& gt = GROUP_TILES[t];
        if (!gt.turns || (forced > 0 ? forced != gt.option : t == WIDE_TILE)) continue;
        const GroupPlan p = make_pp_plan(g, n, gt, us);
        int64_t workgroups = 0;
        for (int i = 0; i < p.njobs; ++i) workgroups += (int64_t)p.job[i].count * p.job[i].shares;
        bool at_once = workgroups <= compute_units();             // uncut, one to a unit
        for (int i = 0; i < p.njobs; ++i) at_once &= p.job[i].shares == 1;
        const double put_at = p.us * (weight_grads && !at_once ? TURNS_LEAD : 1.0);
        if (put_at < us) { best = p; best.tile = t; us = put_at; }
    }
    if (forced <= 0 && std::all_of(g, g + n, [](const GemmArgs& a) { return a.M <= FEW_TOKENS && !a.trans_a; })) {
        GroupPlan p = make_pp_plan(g, n, GROUP_TILES[WIDE_TILE], INFINITY);
        p.tile = WIDE_TILE;
        if (takes_wide_tile(g, n, p, best, us)) best = p;
    }
    return best;
}
// As plan_for.  A layer has two groups in either direction.
GroupPlan plan_group(const GemmArgs* g, int n) {
    static PlanCache<GroupPlan, 2 + 4 * GROUP_MAX, 256> cache;
    int64_t key[2 + 4 * GROUP_MAX] = {n, (int64_t)options().generation};
    for (int i = 0; i < n; ++i) {
        int64_t* k = key + 2 + 4 * i;
        // a group of one is planned for its size alone (by_turns)
        k[0] = g[i].M; k[1] = g[i].N; k[2] = g[i].K; k[3] = n == 1 ? 0 : (g[i].trans_a ? 1 : 0) | (g[i].trans_b ? 2 : 0) | g[i].epi << 2;
    }
    return cache.get(key, [&] { return make_group_plan(g, n); });
}
size_t share_bytes(const GemmArgs& a, int shares) {               // float partial sums, column sums included
    return shares > 1 ? (size_t)shares * ((size_t)a.M * a.N + (size_t)a.N) * sizeof(float) : 0;
}
}  // namespace

// Scratch of the K shares of a plan on the tiles of gemm_bf16_pp.h: the tiles' sums, and column sums of a group's weight gradients.
static size_t pp_colsum_floats(const GemmArgs& a, int n) { return n > 1 && a.trans_a ? (size_t)(a.N + 3) / 4 * 4 : 0; }
static size_t pp_bytes(const GroupPlan& pl, const GemmArgs* g, int n) {
    size_t need = 0;
    for (int j = 0; j < pl.njobs; ++j)
        if (pl.job[j].shares > 1)
            need += (size_t)pl.job[j].shares * ((size_t)pl.job[j].count * GROUP_TILES[pl.tile].bm * GROUP_TILES[pl.tile].bn + pp_colsum_floats(g[pl.job[j].gemm], n)) * sizeof(float);
    return need;
}
size_t gemm_bf16_group_workspace_bytes(const GemmArgs* g, int n) {
    const GroupPlan pl = plan_group(g, n);
    if (GROUP_TILES[pl.tile].turns) return pp_bytes(pl, g, n);
    size_t need = 0;
    for (int i = 0; i < n; ++i) need += share_bytes(g[i], pl.shares[i]);
    return need;
}

template <typename TL, typename Params>
static hipError_t launch_group(void (*kernel)(Params), int threads, const Params& gp, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, TL::LDS_BYTES);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kernel, dim3((unsigned)gp.first[gp.n]), dim3(threads), TL::LDS_BYTES, s, gp);
    return hipGetLastError();
}

template <typename TL>
static hipError_t launch_pp_jobs(const GroupPlan& pl, const GemmArgs* g, int n, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (pp_bytes(pl, g, n) > (ws ? ws_bytes : 0)) return hipErrorInvalidValue;
    PPGroupParams gp{}, sp{};                                     // all jobs; the sums of those that were cut
    float* part = static_cast<float*>(ws);
    gp.n = pl.njobs;
    for (int j = 0; j < pl.njobs; ++j) {
        const PPJob& job = pl.job[j];
        const GemmArgs& a = g[job.gemm];
        GemmParams& p = gp.g[j];
        p = gemm_params(a);
        p.tiles_m = (int)((a.M + TL::BM - 1) / TL::BM);
        p.tiles_n = (int)((a.N + TL::BN - 1) / TL::BN);
        p.band = choose_band(p.tiles_m, TL::BM, TL::BN, TL::LDS_BYTES);
        p.colsum = a.trans_a ? (bf16_t*)a.colsum_b : nullptr;
        gp.layout[j] = a.trans_a ? 2 : a.trans_b ? 1 : 0;
        gp.run[j] = PPRun{job.tile0, job.count, job.nk, nullptr};
        gp.shares[j] = job.shares;
        gp.first[j + 1] = gp.first[j] + job.count * job.shares;
        if (job.shares == 1) continue;
        gp.run[j].partial = part;
        part += (size_t)job.shares * job.count * TL::FLOATS;
        p.colsum_part = part;
        part += (size_t)job.shares * pp_colsum_floats(a, n);
        sp.g[sp.n] = p;
        sp.run[sp.n] = gp.run[j];
        sp.shares[sp.n] = job.shares;
        sp.first[sp.n + 1] = sp.first[sp.n] + job.count * 4 * TL::UA;
        ++sp.n;
    }
    const hipError_t e = launch_group<TL>(&gemm_bf16_group_pp_kernel<TL>, 512, gp, stream);
    if (e != hipSuccess || sp.n == 0) return e;
    hipLaunchKernelGGL(gemm_group_pp_sum_kernel<TL>, dim3((unsigned)sp.first[sp.n]), dim3(512), 0, stream, sp);
    return hipGetLastError();
}

static hipError_t launch_pp(const GroupPlan& pl, const GemmArgs* g, int n, void* ws, size_t ws_bytes, hipStream_t stream) {
    const GroupTile& t = GROUP_TILES[pl.tile];
    return t.bn == 128   ? launch_pp_jobs<PPTile<4, 1>>(pl, g, n, ws, ws_bytes, stream)
           : t.bm == 128 ? launch_pp_jobs<PPTile<2, 1>>(pl, g, n, ws, ws_bytes, stream)
                         : launch_pp_jobs<PPTile<2, 2>>(pl, g, n, ws, ws_bytes, stream);
}

hipError_t gemm_bf16_group(const GemmArgs* g, int n, void* ws, size_t ws_bytes, hipStream_t stream) {
    if (n < 1 || n > GROUP_MAX) return hipErrorInvalidValue;
    const GroupPlan pl = plan_group(g, n);
    const int bm = GROUP_TILES[pl.tile].bm;
    if (GROUP_TILES[pl.tile].turns) return launch_pp(pl, g, n, ws, ws_bytes, stream);
    int order[GROUP_MAX] = {0, 1, 2, 3};
    std::stable_sort(order, order + n, [&](int a, int b) { return pl.nk[a] > pl.nk[b]; });
    GroupParams gp{}, sp{};                                       // the GEMMs; the sums of those that were cut
    gp.n = n;
    char* part = static_cast<char*>(ws);
    size_t used = 0;
    for (int q = 0; q < n; ++q) {
        const GemmArgs& a = g[order[q]];
        const int shares = pl.shares[order[q]];
        GemmParams p = gemm_params(a);
        p.nk = pl.nk[order[q]];
        p.tiles_m = (int)((a.M + bm - 1) / bm);
        p.tiles_n = (int)((a.N + bm - 1) / bm);
        p.band = choose_band(p.tiles_m, bm, bm, 0);
        p.colsum = a.trans_a ? (bf16_t*)a.colsum_b : nullptr;
        if (shares > 1) {
            const size_t bytes = share_bytes(a, shares);
            if (!ws || used + bytes > ws_bytes) return hipErrorInvalidValue;
            p.partial = reinterpret_cast<float*>(part + used);
            p.colsum_part = p.partial + (size_t)shares * a.M * a.N;
            used += bytes;
            sp.g[sp.n] = p;
            sp.shares[sp.n] = shares;
            const int64_t chunks = a.M * a.N / 8 + (p.colsum ? a.N / 8 : 0);
            sp.first[sp.n + 1] = sp.first[sp.n] + (int)((chunks + 255) / 256);
            ++sp.n;
        }
        gp.g[q] = p;
        gp.shares[q] = shares;
        gp.layout[q] = a.trans_a ? 2 : a.trans_b ? 1 : 0;
        gp.first[q + 1] = gp.first[q] + p.tiles_m * p.tiles_n * shares;
    }
    hipError_t e = bm == 192   ? launch_group<Tile<3, 3, 3>>(&gemm_bf16_group_kernel<Tile<3, 3, 3>>, 256, gp, stream)
                   : bm == 128 ? launch_group<Tile<2, 2, 4>>(&gemm_bf16_group_kernel<Tile<2, 2, 4>>, 256, gp, stream)
                               : launch_group<Tile<1, 1, 6>>(&gemm_bf16_group_kernel<Tile<1, 1, 6>>, 256, gp, stream);
    if (e != hipSuccess || sp.n == 0) return e;
    hipLaunchKernelGGL(gemm_group_sum_kernel, dim3((unsigned)sp.first[sp.n]), dim3(256), 0, stream, sp);
    return hipGetLastError();
}

// ---- one GEMM ----------------------------------------------------------------------------------------------------------
// On the 256 x 256 tile of gemm_bf16_pp.h where there is enough of it that its estimate and that of make_plan, which is long for
// short GEMMs, can be compared, and the tile's is less.  Measured over 55 GEMMs, us, kernel of make_plan and tile by turns: NN
// 2048 x 15360 x 1280 87 and 82, 2048 x 49152 x 1536 286 and 261, 2048 x 12288 x 6144 240 and 230, NT 2048 x 1536 x 49152 344 and
// 250, 2048 x 1536 x 12288 80 and 76, TN 1280 x 15360 x 2048 88 and 82; estimates of less than 60 us: 0.98 to 1.8 times as long, the
// 256 x 128 tile 0.8 to 1.8.  Its kernels are built for the layouts of a layer (NN, NT, TN), and the overrides are about the others.
constexpr double BY_TURNS_MIN_US = 60.0;
constexpr int TURNS_VARIANT = NVARIANTS;       // option gemm_tile: this tile for every GEMM in those layouts
static bool by_turns(int64_t M, int64_t N, int64_t K, bool trans_a, bool trans_b, GroupPlan* plan) {
    const Options& o = options();
    if (trans_a && trans_b) return false;
    if (o.gemm_tile == TURNS_VARIANT && o.gemm_shares > 0) {
        const int nk = (int)((K + DK - 1) / DK), per = ((nk + o.gemm_shares - 1) / o.gemm_shares + 1) & ~1;   // two k-steps at a time
        *plan = GroupPlan{};
        plan->njobs = 1;
        plan->job[0] = PPJob{0, 0, (int)(((M + 255) / 256) * ((N + 255) / 256)), per < nk ? per : nk, per < nk ? (nk + per - 1) / per : 1};
        return true;
    }
    if (o.gemm_tile != TURNS_VARIANT && (o.gemm_tile >= 0 || o.gemm_shares > 0 || o.gemm_force[0] || o.gemm_band > 0 || o.fuse_colsum)) return false;
    const double other_us = 0.95 * plan_for(M, N, K, !trans_a, trans_b).us;
    if (o.gemm_tile != TURNS_VARIANT && other_us <= BY_TURNS_MIN_US) return false;
    GemmArgs a{};
    a.dtype = BF16; a.M = M; a.N = N; a.K = K; a.epi = EPI_NONE;
    *plan = plan_group(&a, 1);
    return o.gemm_tile == TURNS_VARIANT || (plan->us >= BY_TURNS_MIN_US && plan->us < other_us);
}
size_t gemm_bf16_share_bytes(int64_t M, int64_t N, int64_t K, bool trans_a, bool trans_b) {
    const Plan pl = plan_for(M, N, K, !trans_a, trans_b);
    return pl.shares > 1 ? (size_t)pl.shares * (size_t)M * (size_t)N * sizeof(float) : 0;
}
size_t gemm_bf16_workspace_bytes(int64_t M, int64_t N, int64_t K, bool trans_a, bool trans_b) {
    size_t need = gemm_bf16_share_bytes(M, N, K, trans_a, trans_b);
    GroupPlan gp;
    const GemmArgs a{};
    if (by_turns(M, N, K, trans_a, trans_b, &gp)) need = std::max(need, pp_bytes(gp, &a, 1));
    return need;
}

hipError_t gemm_bf16(const GemmArgs& a, bool* colsum_done) {
    if (colsum_done) *colsum_done = false;
    GroupPlan gp;
    if (by_turns(a.M, a.N, a.K, a.trans_a != 0, a.trans_b != 0, &gp) && pp_bytes(gp, &a, 1) <= (a.ws ? a.ws_bytes : 0)) {
        GemmArgs one = a;
        one.colsum_b = nullptr;
        return launch_pp(gp, &one, 1, a.ws, a.ws_bytes, a.stream);
    }
    GemmParams p = gemm_params(a);
    const Plan pl = plan_for(a.M, a.N, a.K, !a.trans_a, a.trans_b != 0);
    p.nk = pl.nk_share;
    // the column sums of B ride along only on request (option fuse_colsum), in the weight-gradient kernel (both operands
    // MN-major) with K unsplit
    p.colsum = (a.colsum_b && options().fuse_colsum && pl.variant == 7 && pl.shares == 1 && a.trans_a && !a.trans_b)
                   ? (bf16_t*)a.colsum_b : nullptr;
    if (colsum_done) *colsum_done = p.colsum != nullptr;
    if (pl.shares > 1) {
        if (a.ws == nullptr || a.ws_bytes < (size_t)pl.shares * (size_t)a.M * (size_t)a.N * sizeof(float))
            return hipErrorInvalidValue;
        p.partial = (float*)a.ws;
    }
    hipError_t e;
    switch (pl.variant) {
        case 4: e = launch_spec_layout<SpecTile<4, 3>>(p, a, pl.shares); break;   // 256 x 192, fetch and math wavefronts
        case 1: e = launch_layout<Tile<4, 3, 4>>(p, a, pl.shares); break;    // 256 x 192
        case 2: e = launch_layout<Tile<2, 2, 4>>(p, a, pl.shares); break;    // 128 x 128, two workgroups per CU
        case 3: e = launch_layout<Tile<3, 3, 3>>(p, a, pl.shares); break;    // 192 x 192, two workgroups per CU
        case 5: e = launch_w8_layout<Tile8<2, 3, 5>>(p, a, pl.shares); break;      // 256 x 192, 8 wavefronts, 16x16x32
        case 7: e = launch_x16s_layout<Tile<3, 3, 3>>(p, a, pl.shares); break;     // 192 x 192, 2 workgroups/CU, 16x16x32
        case 6:                                                                    // 256 x 192, fetch + math, 16x16x32
            e = a.trans_b ? launch_spec16<SpecTile<4, 3>, true>(p, a, pl.shares)
                          : launch_spec16<SpecTile<4, 3>, false>(p, a, pl.shares);
            break;
        default: e = launch_layout<Tile<4, 4, 4>>(p, a, pl.shares); break;   // 256 x 256
    }
    if (e != hipSuccess || pl.shares == 1) return e;
    const int64_t chunks = a.M * a.N / 8;
    hipLaunchKernelGGL(gemm_sum_shares_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, a.stream, p, pl.shares);
    return hipGetLastError();
}

}  // namespace tpl

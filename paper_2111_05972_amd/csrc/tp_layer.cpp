// C-ABI entry points: descriptor validation, buffer layouts, and the order in which the kernels of
// one tensor-parallel rank's forward and backward pass are enqueued (App. F.1 of the paper).
#include "../../include/tp_layer.h"

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <initializer_list>

#include "kernels.h"

using namespace tpl;

// ---- tuning overrides (see Options in kernels.h) -------------------------------------------------------------------
namespace tpl {
namespace {
bool parse_int(const char* v, int unset, int lo, int hi, int* out) {
    if (!v || !*v) { *out = unset; return true; }
    char* end = nullptr;
    const long x = strtol(v, &end, 10);
    if (end == v || *end != 0 || x < lo || x > hi) return false;
    *out = (int)x;
    return true;
}
Options& mutable_options() {
    static Options opt = [] {
        Options o;                                      // the environment is read here, once per process
        parse_int(getenv("TPL_GEMM_TILE"), -1, 0, 63, &o.gemm_tile);
        parse_int(getenv("TPL_GEMM_SHARES"), 0, 0, 64, &o.gemm_shares);
        parse_int(getenv("TPL_GEMM_BAND"), 0, 0, 1 << 20, &o.gemm_band);
        parse_int(getenv("TPL_ATTN_CHUNK"), -1, 0, 1 << 16, &o.attn_chunk);
        if (const char* f = getenv("TPL_GEMM_FORCE")) { strncpy(o.gemm_force, f, sizeof(o.gemm_force) - 1); }
        return o;
    }();
    return opt;
}
}  // namespace
const Options& options() { return mutable_options(); }
bool set_option(const char* name, const char* value) {
    if (!name) return false;
    Options& o = mutable_options();
    bool ok = false;
    if (!strcmp(name, "gemm_tile")) ok = parse_int(value, -1, 0, 63, &o.gemm_tile);
    else if (!strcmp(name, "gemm_shares")) ok = parse_int(value, 0, 0, 64, &o.gemm_shares);
    else if (!strcmp(name, "gemm_band")) ok = parse_int(value, 0, 0, 1 << 20, &o.gemm_band);
    else if (!strcmp(name, "attn_chunk")) ok = parse_int(value, -1, 0, 1 << 16, &o.attn_chunk);
    else if (!strcmp(name, "gemm_group")) {
        int v;
        ok = parse_int(value, -1, 0, 512, &v) && (v <= 0 || v == 64 || v == 128 || v == 192 || v == 256 || v == 384 || v == 512);
        if (ok) o.gemm_group = v;
    }
    else if (!strcmp(name, "fuse_colsum")) ok = parse_int(value, 0, 0, 1, &o.fuse_colsum);
    else if (!strcmp(name, "side_chains")) ok = parse_int(value, 0, 2, 3, &o.side_chains);
    else if (!strcmp(name, "gemm_force")) {
        const char* v = value ? value : "";
        if (strlen(v) < sizeof(o.gemm_force)) { strcpy(o.gemm_force, v); ok = true; }
    }
    if (ok) ++o.generation;
    return ok;
}
}  // namespace tpl

namespace {

constexpr size_t ALIGN = 256;
inline size_t up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

// Resolved sizes of a valid descriptor.
struct Dims {
    int64_t H, nh, dh, I, T, r, S, B, M, nl, Hl, Il;
    int dtype;
    size_t esz;
    bool causal, row_epi, side_stream;
};

int resolve(const tp_layer_desc* d, Dims* o) {
    if (!d) return TPL_EINVAL;
    if (d->hidden <= 0 || d->heads <= 0 || d->tp_degree <= 0 || d->seq <= 0 || d->micro_batch <= 0)
        return TPL_EINVAL;
    if (d->head_dim < 0 || d->intermediate < 0) return TPL_EINVAL;
    if (d->dtype != TPL_F32 && d->dtype != TPL_BF16) return TPL_EINVAL;
    if (d->flags & ~(uint32_t)(TPL_CAUSAL | TPL_ROW_EPILOGUE | TPL_SIDE_STREAM)) return TPL_EINVAL;
    if (d->tp_rank < 0 || d->tp_rank >= d->tp_degree) return TPL_EINVAL;
    Dims x;
    x.H = d->hidden; x.nh = d->heads; x.T = d->tp_degree; x.r = d->tp_rank;
    x.S = d->seq; x.B = d->micro_batch;
    if (x.H % x.nh) return TPL_EINVAL;
    x.dh = d->head_dim ? d->head_dim : x.H / x.nh;
    if (x.dh * x.nh != x.H) return TPL_EINVAL;
    x.I = d->intermediate ? d->intermediate : 4 * x.H;
    if (x.nh % x.T || x.I % x.T) return TPL_EINVAL;
    x.M = x.B * x.S; x.nl = x.nh / x.T; x.Hl = x.nl * x.dh; x.Il = x.I / x.T;
    x.dtype = d->dtype; x.esz = d->dtype == TPL_F32 ? 4 : 2;
    x.causal = d->flags & TPL_CAUSAL; x.row_epi = d->flags & TPL_ROW_EPILOGUE;
    x.side_stream = d->flags & TPL_SIDE_STREAM;
    if (x.M > (int64_t)1 << 24 || x.H > (int64_t)1 << 20 || x.I > (int64_t)1 << 24) return TPL_EUNSUPPORTED;
    if (x.dh > 256) return TPL_EUNSUPPORTED;
    // 16-byte rows for every matrix the kernels touch
    if (x.dtype == TPL_BF16 && (x.H % 8 || x.Hl % 8 || x.Il % 8)) return TPL_EUNSUPPORTED;
    if (x.dtype == TPL_F32 && (x.H % 4 || x.Hl % 4 || x.Il % 4)) return TPL_EUNSUPPORTED;
    if (o) *o = x;
    return TPL_OK;
}

void saved_layout(const Dims& x, tp_layer_saved_layout* L) {
    size_t off = 0;
    L->qkv = off; off += up((size_t)x.M * 3 * x.Hl * x.esz);
    L->o = off;   off += up((size_t)x.M * x.Hl * x.esz);
    L->lse = off; off += up((size_t)x.B * x.nl * x.S * sizeof(float));
    L->u = off;   off += up((size_t)x.M * x.Il * x.esz);
    L->g = off;   off += up((size_t)x.M * x.Il * x.esz);
    L->total = off;
}

size_t gemm_ws(int dtype, int64_t M, int64_t N, int64_t K, bool trans_a, bool trans_b) {
    return up(dtype == TPL_BF16 ? gemm_bf16_workspace_bytes(M, N, K, trans_a, trans_b) : gemm_f32_workspace_bytes(M, N, K));
}

// Forward scratch: of the GEMMs (each: one chain's; 0 where they go out in groups), then of attention.
struct FwdWs { bool groups; size_t gemm_each, gemm_all, attn_bytes, total; };
// Backward scratch: dU, dO, dQKV, D, and per chain (attention, MLP) column-sum partials and GEMM scratch.
struct BwdWs { bool groups; size_t du, d_o, dqkv, dsum, colsum, colsum2, gemm, gemm2, gemm3, gemm_each, gemm_all, attn, attn_bytes, total; };

// Float partials of attention strips cut into chunks: inside a layer pass only when TPL_ATTN_CHUNK forces a chunk
// length (own_chunking stays 0: see attn_bf16.hip), so normally 0.
size_t attn_ws(const Dims& x, bool bwd) {
    AttnArgs a{};
    a.dtype = x.dtype; a.B = (int)x.B; a.S = (int)x.S; a.nl = (int)x.nl; a.dh = (int)x.dh; a.causal = x.causal;
    if (x.dtype != BF16 || !attn_bf16_supported(a)) return 0;
    return up(attn_bf16_workspace_bytes(a, bwd));
}

// ---- GEMMs of a pass as groups ---------------------------------------------------------------------------------------
// The GEMMs of a pass that do not depend on each other, over both blocks, form one launch each:
//   forward   {up, qkv}, attention, {down, out}
//   backward  {dW_dn, dW_o, dU, dO}, attention, {dW_up, dW_qkv, dx_mlp, dx_attn}; the bias gradients are column sums of
//             the weight gradients' second operands and ride in them
GemmArgs gemm_args(const Dims& x, int ta, int tb, int64_t M, int64_t N, int64_t K, const void* A = nullptr,
                   const void* B = nullptr, void* C = nullptr) {
    GemmArgs g{};
    g.dtype = x.dtype; g.trans_a = ta; g.trans_b = tb; g.M = M; g.N = N; g.K = K;
    g.A = A; g.B = B; g.C = C; g.epi = EPI_NONE;
    return g;
}
size_t group_ws(const Dims& x, bool bwd) {
    GemmArgs first[4], second[4];
    int n1 = 0, n2 = 0;
    if (!bwd) {                                      // as launched: plans go by shapes, layouts and GeLU epilogues
        first[n1++] = gemm_args(x, 0, 0, x.M, x.Il, x.H);
        first[0].epi = EPI_GELU;
        first[n1++] = gemm_args(x, 0, 0, x.M, 3 * x.Hl, x.H);
        second[n2++] = gemm_args(x, 0, 0, x.M, x.H, x.Il);
        second[n2++] = gemm_args(x, 0, 0, x.M, x.H, x.Hl);
    } else {
        first[n1++] = gemm_args(x, 1, 0, x.Il, x.H, x.M);
        first[n1++] = gemm_args(x, 1, 0, x.Hl, x.H, x.M);
        first[n1++] = gemm_args(x, 0, 1, x.M, x.Il, x.H);
        first[2].epi = EPI_DGELU;
        first[n1++] = gemm_args(x, 0, 1, x.M, x.Hl, x.H);
        second[n2++] = gemm_args(x, 1, 0, x.H, x.Il, x.M);
        second[n2++] = gemm_args(x, 1, 0, x.H, 3 * x.Hl, x.M);
        second[n2++] = gemm_args(x, 0, 1, x.M, x.H, x.Il);
        second[n2++] = gemm_args(x, 0, 1, x.M, x.H, 3 * x.Hl);
    }
    const auto bytes = x.dtype == BF16 ? gemm_bf16_group_workspace_bytes : gemm_f32_group_workspace_bytes;
    return up(std::max(bytes(first, n1), bytes(second, n2)));
}
bool use_groups(const Dims& x);
// Largest scratch of a list of GEMMs launched one by one.
struct GemmShape { int trans_a, trans_b; int64_t M, N, K; };
size_t single_ws(const Dims& x, std::initializer_list<GemmShape> list, bool launched) {
    size_t need = ALIGN;
    for (const GemmShape& g : list)
        need = std::max(need, launched || x.dtype != BF16 ? gemm_ws(x.dtype, g.M, g.N, g.K, g.trans_a, g.trans_b)
                                                          : up(gemm_bf16_share_bytes(g.M, g.N, g.K, g.trans_a, g.trans_b)));
    return need;
}
// Only what the pass launches is sized: a call does this before its first launch.
void fwd_layout(const Dims& x, FwdWs* W) {
    W->groups = use_groups(x);
    W->gemm_each = W->groups ? 0 : single_ws(x, {{0, 0, x.M, 3 * x.Hl, x.H}, {0, 0, x.M, x.H, x.Hl}, {0, 0, x.M, x.Il, x.H}, {0, 0, x.M, x.H, x.Il}}, true);
    W->gemm_all = W->groups ? std::max(group_ws(x, false), ALIGN) : 2 * W->gemm_each;
    W->attn_bytes = attn_ws(x, false);
    W->total = W->gemm_all + W->attn_bytes;
}

void bwd_layout(const Dims& x, BwdWs* W) {
    size_t off = 0;
    W->groups = use_groups(x);
    W->du = off;   off += up((size_t)x.M * x.Il * x.esz);
    W->d_o = off;  off += up((size_t)x.M * x.Hl * x.esz);
    W->dqkv = off; off += up((size_t)x.M * 3 * x.Hl * x.esz);
    W->dsum = off; off += up((size_t)x.B * x.nl * x.S * sizeof(float));
    int64_t nmax = std::max(std::max(x.Il, 3 * x.Hl), x.H);
    W->colsum = off; off += up(colsum_scratch_bytes(x.M, nmax));
    W->colsum2 = off; off += up(colsum_scratch_bytes(x.M, nmax));
    W->gemm_each = single_ws(x, {{0, 1, x.M, x.Il, x.H}, {1, 0, x.Il, x.H, x.M}, {1, 0, x.H, x.Il, x.M}, {0, 1, x.M, x.H, x.Il},
                                 {0, 1, x.M, x.Hl, x.H}, {1, 0, x.Hl, x.H, x.M}, {1, 0, x.H, 3 * x.Hl, x.M}, {0, 1, x.M, x.H, 3 * x.Hl}}, !W->groups);
    W->gemm = off;
    W->gemm2 = W->gemm + W->gemm_each;
    W->gemm3 = W->gemm2 + W->gemm_each;                // the two weight gradients that depend on nothing computed in the pass (third chain)
    // groups: no less than two chains of single GEMMs cut on the other tiles, which callers have room for
    off += W->groups ? std::max(group_ws(x, true), 2 * W->gemm_each) : 3 * W->gemm_each;
    W->gemm_all = off - W->gemm;
    W->attn_bytes = attn_ws(x, true);
    W->attn = off; off += W->attn_bytes;
    W->total = off;
}

inline bool misaligned(const void* p) { return ((uintptr_t)p & 15u) != 0; }

// Diagnostic timing of GEMM launches, single or grouped, with HIP events on the launch stream (off by default).
struct GemmProfile {
    static constexpr int CAP = 4096;
    bool on = false;
    int n = 0;
    hipEvent_t start[CAP], stop[CAP];
    bool created[CAP] = {};
} g_prof;

// The attention block and the MLP block of one pass share no tensor (each has its own input, output and
// gradients).  By default both are enqueued on the caller's stream, in the order written.  With TPL_SIDE_STREAM in
// the descriptor's flags they are enqueued as two chains: the attention chain on the caller's stream and the MLP
// chain on a second stream that the library creates once per device (default priority, non-blocking).  The second
// stream is forked from the caller's stream and joined back to it with events, so the caller sees one pass on its
// stream and the host never waits.  What the overlap can buy: tiles of one chain fill the compute units the other
// leaves idle (a GEMM whose tile count is below the number of compute units, the attention kernels, the start and
// end of every kernel).  Per-GEMM timing (tp_layer_profile) keeps everything on the caller's stream.
struct SideStream {
    hipStream_t stream = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    int state = 0;       // 0 = not tried, 1 = ready, -1 = unavailable
};
constexpr int MAX_DEVICES = 64;
constexpr int MAX_SIDE = 2;
SideStream g_side[MAX_DEVICES][MAX_SIDE];

// Returns the stream for the second chain, already waiting for everything enqueued on s so far; s itself when
// the second stream is not used.
hipStream_t side_fork(hipStream_t s, bool wanted, int which = 0) {
    if (!wanted || g_prof.on) return s;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return s;
    SideStream& ss = g_side[dev][which];
    if (ss.state == 0) {
        ss.state = (hipStreamCreateWithFlags(&ss.stream, hipStreamNonBlocking) == hipSuccess &&
                    hipEventCreateWithFlags(&ss.fork, hipEventDisableTiming) == hipSuccess &&
                    hipEventCreateWithFlags(&ss.join, hipEventDisableTiming) == hipSuccess) ? 1 : -1;
    }
    if (ss.state != 1) return s;
    if (hipEventRecord(ss.fork, s) != hipSuccess || hipStreamWaitEvent(ss.stream, ss.fork, 0) != hipSuccess) return s;
    return ss.stream;
}
// Makes s wait for everything enqueued on the second stream.
int side_join(hipStream_t s, hipStream_t s2, int which = 0) {
    if (s2 == s) return TPL_OK;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return TPL_EHIP;
    SideStream& ss = g_side[dev][which];
    if (hipEventRecord(ss.join, s2) != hipSuccess || hipStreamWaitEvent(s, ss.join, 0) != hipSuccess) return TPL_EHIP;
    return TPL_OK;
}
// A pass that fails after the fork still joins: the caller's stream must not run ahead of work already enqueued
// on the second stream that touches the caller's buffers.
struct SideJoin {
    hipStream_t s, s2;
    int which = 0;
    bool done = false;
    int finish() { done = true; return side_join(s, s2, which); }
    ~SideJoin() { if (!done) side_join(s, s2, which); }
};

// Runs launch() between the two events of a record where launches are timed.
template <typename Launch>
int profiled(hipStream_t stream, Launch launch) {
    int slot = -1;
    if (g_prof.on && g_prof.n < GemmProfile::CAP) {
        slot = g_prof.n++;
        if (!g_prof.created[slot]) {
            if (hipEventCreate(&g_prof.start[slot]) != hipSuccess || hipEventCreate(&g_prof.stop[slot]) != hipSuccess)
                return TPL_EHIP;
            g_prof.created[slot] = true;
        }
        if (hipEventRecord(g_prof.start[slot], stream) != hipSuccess) return TPL_EHIP;
    }
    const hipError_t e = launch();
    if (slot >= 0 && hipEventRecord(g_prof.stop[slot], stream) != hipSuccess) return TPL_EHIP;
    return e == hipSuccess ? TPL_OK : TPL_EHIP;
}

int run_gemm(GemmArgs& g) {
    return profiled(g.stream, [&] {
        g.colsum_done = false;
        if (g.dtype == BF16 && gemm_bf16_supported(g)) return gemm_bf16(g, &g.colsum_done);
        return gemm_f32_supported(g) ? gemm_f32(g) : gemm_simple(g);
    });
}

int run_attn(AttnArgs& a, bool bwd) {
    hipError_t e;
    if (a.dtype == BF16 && attn_bf16_supported(a)) e = bwd ? attn_bf16_bwd(a) : attn_bf16_fwd(a);
    else if (attn_f32_supported(a)) e = bwd ? attn_f32_bwd(a) : attn_f32_fwd(a);
    else e = bwd ? attn_simple_bwd(a) : attn_simple_fwd(a);
    return e == hipSuccess ? TPL_OK : TPL_EHIP;
}

// Scratch handed to every GEMM of one entry-point call.
struct GemmScratch { void* ws; size_t bytes; hipStream_t stream; };

GemmArgs mk(const Dims& x, int ta, int tb, int64_t M, int64_t N, int64_t K, const void* A,
            const void* B, void* C, GemmScratch& sc) {
    GemmArgs g = gemm_args(x, ta, tb, M, N, K, A, B, C);
    g.ws = sc.ws; g.ws_bytes = sc.bytes; g.stream = sc.stream;
    return g;
}

// Whether the GEMMs of a pass go out as groups.
bool use_groups(const Dims& x) {
    const Options& o = options();
    if (o.gemm_group == 0) return false;
    // every operand within the matrix-core kernels' 32-bit offsets (whole 16-byte rows are given, in either type)
    const int64_t widest = std::max(std::max(x.Il, 3 * x.Hl), x.H);
    if (std::max(x.M, x.H) * widest * x.esz >= 0x7FFFFFFFll) return false;
    if (o.gemm_group > 0) return true;
    // the other GEMM overrides speak about launches of one GEMM and about chains
    if (o.gemm_tile >= 0 || o.gemm_shares > 0 || o.gemm_force[0] || o.gemm_band > 0 || o.side_chains || o.fuse_colsum) return false;
    // groups are ahead at every size (whole steps, groups against single GEMMs on two chains where the caller allows: BERT-large
    // TP 4 156 and 236 us, GPT-3 13B TP 4 1700 and 1840, GPT-3 175B TP 8 2200 and 2290, where attention runs beside GEMMs)
    return true;
}
int run_group(const GemmArgs* g, int n, const GemmScratch& sc) {
    const auto group = g[0].dtype == BF16 ? gemm_bf16_group : gemm_f32_group;
    return profiled(sc.stream, [&] { return group(g, n, sc.ws, sc.bytes, sc.stream); });
}

// Forward kernels in order.  With row_parallel == false the two row-parallel GEMMs (whose outputs the
// backward pass never reads) are skipped: that is the recomputation done in checkpoint mode.
int fwd_impl(const Dims& x, const FwdWs& W, const tp_layer_params* p, const void* x_attn, const void* x_mlp, void* y_attn,
             void* y_mlp, void* saved, void* ws, hipStream_t s, bool row_parallel) {
    int rc;
    tp_layer_saved_layout L;
    saved_layout(x, &L);
    char* sv = (char*)saved;
    void *qkv = sv + L.qkv, *o = sv + L.o, *u = sv + L.u, *g = sv + L.g;
    float* lse = (float*)(sv + L.lse);
    const bool groups = W.groups;
    hipStream_t s2 = side_fork(s, x.side_stream && !groups);
    SideJoin sj{s, s2};
    GemmScratch sc{ws, W.gemm_each, s}, sc2{(char*)ws + W.gemm_each, W.gemm_each, s2}, all{ws, W.gemm_all, s};

    // MLP block (second chain): column-parallel up-projection + GeLU, row-parallel down-projection
    GemmArgs g4 = mk(x, 0, 0, x.M, x.Il, x.H, x_mlp, p->w_up, g, sc2);
    g4.bias = p->b_up; g4.aux = u; g4.epi = EPI_GELU;
    GemmArgs g5 = mk(x, 0, 0, x.M, x.H, x.Il, g, p->w_dn, y_mlp, sc2);
    if (x.row_epi) { g5.bias = p->b_dn; g5.resid = x_mlp; }
    if (!groups) {
        if ((rc = run_gemm(g4))) return rc;
        if (row_parallel && (rc = run_gemm(g5))) return rc;
    }
    // attention block: column-parallel fused QKV, attention on the local heads, row-parallel out-proj
    GemmArgs g1 = mk(x, 0, 0, x.M, 3 * x.Hl, x.H, x_attn, p->w_qkv, qkv, sc);
    g1.bias = p->b_qkv;
    if (groups) {
        const GemmArgs first[] = {g4, g1};
        if ((rc = run_group(first, 2, all))) return rc;
    } else if ((rc = run_gemm(g1))) {
        return rc;
    }
    AttnArgs at{};
    at.dtype = x.dtype; at.B = (int)x.B; at.S = (int)x.S; at.nl = (int)x.nl; at.dh = (int)x.dh;
    at.causal = x.causal; at.qkv = qkv; at.o = o; at.lse = lse; at.stream = s;
    at.ws_bytes = W.attn_bytes;
    at.ws = at.ws_bytes ? (char*)ws + W.gemm_all : nullptr;
    if ((rc = run_attn(at, false))) return rc;
    if (row_parallel) {
        GemmArgs g3 = mk(x, 0, 0, x.M, x.H, x.Hl, o, p->w_o, y_attn, sc);
        if (x.row_epi) { g3.bias = p->b_o; g3.resid = x_attn; }
        if (groups) {
            const GemmArgs second[] = {g5, g3};
            if ((rc = run_group(second, 2, all))) return rc;
        } else if ((rc = run_gemm(g3))) {
            return rc;
        }
    }
    return sj.finish();
}

// Argument checks shared by the entry points: NULL pointers, then alignment.  `row_parallel`: the forward pass
// runs its two row-parallel GEMMs (they need b_o, b_dn on the epilogue rank); the recomputation of checkpoint
// mode does not.
int fwd_check(const Dims& x, const tp_layer_params* p, const void* x_attn, const void* x_mlp, const void* ws,
              bool row_parallel) {
    if (!p || !x_attn || !x_mlp || !ws) return TPL_EINVAL;
    if (!p->w_qkv || !p->b_qkv || !p->w_o || !p->w_up || !p->b_up || !p->w_dn) return TPL_EINVAL;
    if (row_parallel && x.row_epi && (!p->b_o || !p->b_dn)) return TPL_EINVAL;
    const void* ptrs[] = {x_attn, x_mlp, ws, p->w_qkv, p->b_qkv, p->w_o, p->b_o, p->w_up, p->b_up, p->w_dn, p->b_dn};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    return TPL_OK;
}

int bwd_check(const Dims& x, const tp_layer_params* p, const void* x_attn, const void* x_mlp, const void* dy_attn,
              const void* dy_mlp, const tp_layer_grads* gr, const void* dx_attn, const void* dx_mlp, const void* ws) {
    if (!p || !gr || !x_attn || !x_mlp || !dy_attn || !dy_mlp || !dx_attn || !dx_mlp || !ws) return TPL_EINVAL;
    if (!p->w_qkv || !p->w_o || !p->w_up || !p->w_dn) return TPL_EINVAL;
    if (!gr->dw_qkv || !gr->db_qkv || !gr->dw_o || !gr->dw_up || !gr->db_up || !gr->dw_dn) return TPL_EINVAL;
    if (x.row_epi && (!gr->db_o || !gr->db_dn)) return TPL_EINVAL;
    const void* ptrs[] = {x_attn, x_mlp, dy_attn, dy_mlp, dx_attn, dx_mlp, ws, p->w_qkv, p->w_o,
                          p->w_up, p->w_dn, gr->dw_qkv, gr->db_qkv, gr->dw_o, gr->db_o, gr->dw_up,
                          gr->db_up, gr->dw_dn, gr->db_dn};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    return TPL_OK;
}

// Backward kernels in order (arguments already checked, ws large enough).
int bwd_impl(const Dims& x, const BwdWs& W, const tp_layer_params* p, const void* x_attn, const void* x_mlp, const void* dy_attn,
             const void* dy_mlp, const void* saved, const tp_layer_grads* gr, void* dx_attn, void* dx_mlp, void* ws,
             hipStream_t s) {
    int rc;
    tp_layer_saved_layout L;
    saved_layout(x, &L);
    const char* sv = (const char*)saved;
    const void *qkv = sv + L.qkv, *o = sv + L.o, *u = sv + L.u, *g = sv + L.g;
    const float* lse = (const float*)(sv + L.lse);
    char* w = (char*)ws;
    void *du = w + W.du, *d_o = w + W.d_o, *dqkv = w + W.dqkv;
    float *dsum = (float*)(w + W.dsum), *cs = (float*)(w + W.colsum), *cs2 = (float*)(w + W.colsum2);
    const bool groups = W.groups, side = x.side_stream && !groups;
    hipStream_t s2 = side_fork(s, side);
    SideJoin sj{s, s2};
    // dW_dn and dW_o need only the pass's inputs and saved activations: with option side_chains = 3 they are a third chain on a
    // stream of their own (-4 % of the step of a RoBERTa-large shard launched GEMM by GEMM, +1 to +2 % where GEMMs fill the
    // chip; the layers it helps go out as groups, so it is not taken by size)
    hipStream_t s3 = options().side_chains == 3 ? side_fork(s, side, 1) : nullptr;
    SideJoin sj3{s, s3 ? s3 : s, 1};
    GemmScratch sc{w + W.gemm, W.gemm_each, s}, sc2{w + W.gemm2, W.gemm_each, s2};
    GemmScratch sc3a{w + W.gemm3, W.gemm_each, s3 ? s3 : s2}, sc3b{w + W.gemm3, W.gemm_each, s3 ? s3 : s};

    // dU = (dy_m W_dn^T) * gelu'(U) in one GEMM epilogue.  Weight gradients are not read again in the pass; the bias
    // gradients are the column sums of their second operand (colsum_b), left by the same launch where it can.
    GemmArgs b5 = mk(x, 0, 1, x.M, x.Il, x.H, dy_mlp, p->w_dn, du, sc2);
    b5.aux = const_cast<void*>(u); b5.epi = EPI_DGELU;
    GemmArgs w5 = mk(x, 1, 0, x.Il, x.H, x.M, g, dy_mlp, gr->dw_dn, s3 ? sc3a : sc2);
    GemmArgs w4 = mk(x, 1, 0, x.H, x.Il, x.M, x_mlp, du, gr->dw_up, sc2);
    GemmArgs d4 = mk(x, 0, 1, x.M, x.H, x.Il, du, p->w_up, dx_mlp, sc2);
    GemmArgs d3 = mk(x, 0, 1, x.M, x.Hl, x.H, dy_attn, p->w_o, d_o, sc);
    GemmArgs w3 = mk(x, 1, 0, x.Hl, x.H, x.M, o, dy_attn, gr->dw_o, s3 ? sc3b : sc);
    GemmArgs w1 = mk(x, 1, 0, x.H, 3 * x.Hl, x.M, x_attn, dqkv, gr->dw_qkv, sc);
    GemmArgs d1 = mk(x, 0, 1, x.M, x.H, 3 * x.Hl, dqkv, p->w_qkv, dx_attn, sc);
    w5.c_streaming = w4.c_streaming = w3.c_streaming = w1.c_streaming = true;
    w4.colsum_b = gr->db_up;
    w1.colsum_b = gr->db_qkv;
    if (x.row_epi) { d4.resid = dy_mlp; d1.resid = dy_attn; }
    AttnArgs at{};
    at.dtype = x.dtype; at.B = (int)x.B; at.S = (int)x.S; at.nl = (int)x.nl; at.dh = (int)x.dh;
    at.causal = x.causal; at.qkv = qkv; at.o = const_cast<void*>(o); at.lse = const_cast<float*>(lse);
    at.d_o = d_o; at.dqkv = dqkv; at.dsum = dsum; at.stream = s;
    at.ws_bytes = W.attn_bytes;
    at.ws = W.attn_bytes ? w + W.attn : nullptr;

    if (groups) {
        if (x.row_epi) { w5.colsum_b = gr->db_dn; w3.colsum_b = gr->db_o; }
        const GemmScratch all{w + W.gemm, W.gemm_all, s};
        const GemmArgs first[] = {w5, w3, b5, d3}, second[] = {w4, w1, d4, d1};
        if ((rc = run_group(first, 4, all))) return rc;
        if ((rc = run_attn(at, true))) return rc;
        return run_group(second, 4, all);
    }

    // MLP block (second chain)
    if ((rc = run_gemm(b5))) return rc;
    if ((rc = run_gemm(w5))) return rc;
    if ((rc = run_gemm(w4))) return rc;
    if (!w4.colsum_done && colsum(x.dtype, x.M, x.Il, du, gr->db_up, cs2, s2) != hipSuccess) return TPL_EHIP;
    if ((rc = run_gemm(d4))) return rc;
    if (x.row_epi && colsum(x.dtype, x.M, x.H, dy_mlp, gr->db_dn, cs2, s2) != hipSuccess) return TPL_EHIP;
    // attention block
    if ((rc = run_gemm(d3))) return rc;
    if ((rc = run_gemm(w3))) return rc;
    if (x.row_epi && colsum(x.dtype, x.M, x.H, dy_attn, gr->db_o, cs, s) != hipSuccess) return TPL_EHIP;
    if ((rc = run_attn(at, true))) return rc;
    if ((rc = run_gemm(w1))) return rc;
    if (!w1.colsum_done && colsum(x.dtype, x.M, 3 * x.Hl, dqkv, gr->db_qkv, cs, s) != hipSuccess) return TPL_EHIP;
    if ((rc = run_gemm(d1))) return rc;
    if ((rc = sj3.finish())) { return rc; }
    return sj.finish();
}
}  // namespace

extern "C" {

int tp_layer_validate(const tp_layer_desc* desc) { return resolve(desc, nullptr); }

size_t tp_layer_saved_bytes(const tp_layer_desc* desc) {
    Dims x;
    if (resolve(desc, &x) != TPL_OK) return 0;
    tp_layer_saved_layout L;
    saved_layout(x, &L);
    return L.total;
}

int tp_layer_saved_offsets(const tp_layer_desc* desc, tp_layer_saved_layout* out) {
    Dims x;
    int rc = resolve(desc, &x);
    if (rc != TPL_OK) return rc;
    if (!out) return TPL_EINVAL;
    saved_layout(x, out);
    return TPL_OK;
}

size_t tp_layer_workspace_bytes(const tp_layer_desc* desc, int bwd) {
    Dims x;
    if (resolve(desc, &x) != TPL_OK) return 0;
    if (!bwd) {
        FwdWs F;
        fwd_layout(x, &F);
        return F.total;
    }
    BwdWs W;
    bwd_layout(x, &W);
    return W.total;
}

int tp_layer_fwd(const tp_layer_desc* desc, const tp_layer_params* p, const void* x_attn,
                 const void* x_mlp, void* y_attn, void* y_mlp, void* saved, void* ws,
                 size_t ws_bytes, void* hip_stream) {
    Dims x;
    int rc = resolve(desc, &x);
    if (rc != TPL_OK) return rc;
    if ((rc = fwd_check(x, p, x_attn, x_mlp, ws, true))) return rc;
    if (!y_attn || !y_mlp || !saved) return TPL_EINVAL;
    if (misaligned(y_attn) || misaligned(y_mlp) || misaligned(saved)) return TPL_EALIGN;
    FwdWs W;
    fwd_layout(x, &W);
    if (ws_bytes < W.total) return TPL_EWORKSPACE;
    return fwd_impl(x, W, p, x_attn, x_mlp, y_attn, y_mlp, saved, ws, (hipStream_t)hip_stream, true);
}

int tp_layer_bwd(const tp_layer_desc* desc, const tp_layer_params* p, const void* x_attn,
                 const void* x_mlp, const void* dy_attn, const void* dy_mlp, const void* saved,
                 const tp_layer_grads* gr, void* dx_attn, void* dx_mlp, void* ws, size_t ws_bytes,
                 void* hip_stream) {
    Dims x;
    int rc = resolve(desc, &x);
    if (rc != TPL_OK) return rc;
    if ((rc = bwd_check(x, p, x_attn, x_mlp, dy_attn, dy_mlp, gr, dx_attn, dx_mlp, ws))) return rc;
    if (!saved) return TPL_EINVAL;
    if (misaligned(saved)) return TPL_EALIGN;
    BwdWs W;
    bwd_layout(x, &W);
    if (ws_bytes < W.total) return TPL_EWORKSPACE;
    return bwd_impl(x, W, p, x_attn, x_mlp, dy_attn, dy_mlp, saved, gr, dx_attn, dx_mlp, ws, (hipStream_t)hip_stream);
}

size_t tp_layer_workspace_bytes_recompute(const tp_layer_desc* desc) {
    Dims x;
    if (resolve(desc, &x) != TPL_OK) return 0;
    tp_layer_saved_layout L;
    saved_layout(x, &L);
    FwdWs F;
    fwd_layout(x, &F);
    BwdWs W;
    bwd_layout(x, &W);
    return up(L.total) + std::max(W.total, F.total);
}

int tp_layer_bwd_recompute(const tp_layer_desc* desc, const tp_layer_params* p, const void* x_attn,
                           const void* x_mlp, const void* dy_attn, const void* dy_mlp,
                           const tp_layer_grads* gr, void* dx_attn, void* dx_mlp, void* ws, size_t ws_bytes,
                           void* hip_stream) {
    Dims x;
    int rc = resolve(desc, &x);
    if (rc != TPL_OK) return rc;
    // everything either pass needs is checked before the recomputed forward is enqueued
    if ((rc = fwd_check(x, p, x_attn, x_mlp, ws, false))) return rc;
    if ((rc = bwd_check(x, p, x_attn, x_mlp, dy_attn, dy_mlp, gr, dx_attn, dx_mlp, ws))) return rc;
    tp_layer_saved_layout L;
    saved_layout(x, &L);
    FwdWs F;
    fwd_layout(x, &F);
    BwdWs W;
    bwd_layout(x, &W);
    if (ws_bytes < up(L.total) + std::max(W.total, F.total)) return TPL_EWORKSPACE;
    char* saved = (char*)ws;
    char* rest = saved + up(L.total);
    // recompute QKV, O, LSE, U, G from the block inputs, then the ordinary backward
    rc = fwd_impl(x, F, p, x_attn, x_mlp, nullptr, nullptr, saved, rest, (hipStream_t)hip_stream, false);
    if (rc != TPL_OK) return rc;
    return bwd_impl(x, W, p, x_attn, x_mlp, dy_attn, dy_mlp, saved, gr, dx_attn, dx_mlp, rest, (hipStream_t)hip_stream);
}

static int ln_check(int dtype, int64_t M, int64_t H) {
    if (dtype != TPL_F32 && dtype != TPL_BF16) return TPL_EINVAL;
    if (M <= 0 || H <= 0) return TPL_EINVAL;
    if (!ln_supported(H)) return TPL_EUNSUPPORTED;
    return TPL_OK;
}

size_t tp_layer_ln_workspace_bytes(int64_t M, int64_t H) {
    if (M <= 0 || H <= 0) return 0;
    return up(ln_scratch_bytes(M, H));
}

int tp_layer_ln_fwd(int dtype, int64_t M, int64_t H, const void* a, const void* b, const void* gamma,
                    const void* beta, float eps, void* z, void* y, float* mean, float* rstd, void* hip_stream) {
    int rc = ln_check(dtype, M, H);
    if (rc) return rc;
    if (!a || !gamma || !beta || !y || !mean || !rstd || !(eps >= 0.0f)) return TPL_EINVAL;
    const void* ptrs[] = {a, b, gamma, beta, z, y, mean, rstd};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    LnArgs l{};
    l.dtype = dtype; l.M = M; l.H = H; l.a = a; l.b = b; l.gamma = gamma; l.beta = beta; l.eps = eps;
    l.z = z; l.y = y; l.mean = mean; l.rstd = rstd; l.stream = (hipStream_t)hip_stream;
    return ln_fwd(l) == hipSuccess ? TPL_OK : TPL_EHIP;
}

int tp_layer_ln_bwd(int dtype, int64_t M, int64_t H, const void* dy, const void* z, const float* mean,
                    const float* rstd, const void* gamma, void* dz, void* dgamma, void* dbeta, void* ws,
                    size_t ws_bytes, void* hip_stream) {
    int rc = ln_check(dtype, M, H);
    if (rc) return rc;
    if (!dy || !z || !mean || !rstd || !gamma || !dz || !dgamma || !dbeta || !ws) return TPL_EINVAL;
    const void* ptrs[] = {dy, z, mean, rstd, gamma, dz, dgamma, dbeta, ws};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    if (ws_bytes < tp_layer_ln_workspace_bytes(M, H)) return TPL_EWORKSPACE;
    LnArgs l{};
    l.dtype = dtype; l.M = M; l.H = H; l.dy = dy; l.z = const_cast<void*>(z); l.mean = const_cast<float*>(mean);
    l.rstd = const_cast<float*>(rstd); l.gamma = gamma; l.dz = dz; l.dgamma = dgamma; l.dbeta = dbeta;
    l.partials = (float*)ws; l.stream = (hipStream_t)hip_stream;
    return ln_bwd(l) == hipSuccess ? TPL_OK : TPL_EHIP;
}

static int dist_check(int dtype, int64_t M, int64_t Hs) {
    if (dtype != TPL_F32 && dtype != TPL_BF16) return TPL_EINVAL;
    if (M <= 0 || Hs <= 0) return TPL_EINVAL;
    if (!ln_supported(Hs)) return TPL_EUNSUPPORTED;
    return TPL_OK;
}
static int hip_rc(hipError_t e) { return e == hipSuccess ? TPL_OK : TPL_EHIP; }

int tp_layer_ln_moments(int dtype, int64_t M, int64_t Hs, const void* x_loc, float* sums, void* hip_stream) {
    int rc = dist_check(dtype, M, Hs);
    if (rc) return rc;
    if (!x_loc || !sums) return TPL_EINVAL;
    if (misaligned(x_loc) || misaligned(sums)) return TPL_EALIGN;
    return hip_rc(ln_dist_moments(dtype, M, Hs, x_loc, sums, (hipStream_t)hip_stream));
}

int tp_layer_ln_stats(int64_t M, int64_t H, float eps, const float* totals, float* mean, float* rstd,
                      void* hip_stream) {
    if (M <= 0 || H <= 0 || !(eps >= 0.0f) || !totals || !mean || !rstd) return TPL_EINVAL;
    return hip_rc(ln_dist_stats(M, H, eps, totals, mean, rstd, (hipStream_t)hip_stream));
}

int tp_layer_ln_apply_fwd(int dtype, int64_t M, int64_t Hs, const void* x_loc, const float* mean,
                          const float* rstd, const void* gamma_loc, const void* beta_loc, void* y,
                          void* hip_stream) {
    int rc = dist_check(dtype, M, Hs);
    if (rc) return rc;
    if (!x_loc || !mean || !rstd || !gamma_loc || !beta_loc || !y) return TPL_EINVAL;
    const void* ptrs[] = {x_loc, gamma_loc, beta_loc, y};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    return hip_rc(ln_dist_apply(dtype, M, Hs, x_loc, mean, rstd, gamma_loc, beta_loc, y, (hipStream_t)hip_stream));
}

int tp_layer_ln_apply_bwd_sums(int dtype, int64_t M, int64_t Hs, const void* dy, const void* x_loc,
                               const float* mean, const float* rstd, const void* gamma_loc, float* sums,
                               void* hip_stream) {
    int rc = dist_check(dtype, M, Hs);
    if (rc) return rc;
    if (!dy || !x_loc || !mean || !rstd || !gamma_loc || !sums) return TPL_EINVAL;
    const void* ptrs[] = {dy, x_loc, gamma_loc};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    return hip_rc(ln_dist_bwd_sums(dtype, M, Hs, dy, x_loc, mean, rstd, gamma_loc, sums, (hipStream_t)hip_stream));
}

size_t tp_layer_ln_apply_workspace_bytes(int64_t M, int64_t Hs) {
    if (M <= 0 || Hs <= 0) return 0;
    return up(ln_dist_scratch_bytes(M, Hs));
}

int tp_layer_ln_apply_bwd(int dtype, int64_t M, int64_t Hs, int64_t H, const void* dy, const void* x_loc,
                          const float* mean, const float* rstd, const void* gamma_loc, const float* totals,
                          const void* dx_add, void* dx, void* dgamma_loc, void* dbeta_loc, void* ws,
                          size_t ws_bytes, void* hip_stream) {
    int rc = dist_check(dtype, M, Hs);
    if (rc) return rc;
    if (H < Hs) return TPL_EINVAL;
    if (!dy || !x_loc || !mean || !rstd || !gamma_loc || !totals || !dx || !dgamma_loc || !dbeta_loc || !ws)
        return TPL_EINVAL;
    const void* ptrs[] = {dy, x_loc, gamma_loc, dx_add, dx, dgamma_loc, dbeta_loc, ws};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    if (ws_bytes < tp_layer_ln_apply_workspace_bytes(M, Hs)) return TPL_EWORKSPACE;
    return hip_rc(ln_dist_bwd_apply(dtype, M, Hs, H, dy, x_loc, mean, rstd, gamma_loc, totals, dx_add, dx,
                                    dgamma_loc, dbeta_loc, (float*)ws, (hipStream_t)hip_stream));
}

static int ew_check(int dtype, int64_t M, int64_t N) {
    if (dtype != TPL_F32 && dtype != TPL_BF16) return TPL_EINVAL;
    if (M <= 0 || N <= 0) return TPL_EINVAL;
    if (N % 8) return TPL_EUNSUPPORTED;
    return TPL_OK;
}

int tp_layer_slice_epilogue_fwd(int dtype, int act, int64_t M, int64_t N, const void* in, const void* bias,
                                const void* resid, void* u, void* out, void* hip_stream) {
    int rc = ew_check(dtype, M, N);
    if (rc) return rc;
    if (act != TPL_ACT_NONE && act != TPL_ACT_GELU) return TPL_EINVAL;
    if (!in || !bias || !out || (act == TPL_ACT_GELU && !u)) return TPL_EINVAL;
    const void* ptrs[] = {in, bias, resid, u, out};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    return hip_rc(slice_epilogue_fwd(dtype, act == TPL_ACT_GELU, M, N, in, bias, resid, u, out,
                                     (hipStream_t)hip_stream));
}

size_t tp_layer_slice_epilogue_workspace_bytes(int64_t M, int64_t N) {
    if (M <= 0 || N <= 0) return 0;
    return up(colsum_scratch_bytes(M, N));
}

int tp_layer_slice_epilogue_bwd(int dtype, int act, int64_t M, int64_t N, const void* dout, const void* u,
                                void* din, void* dbias, void* ws, size_t ws_bytes, void* hip_stream) {
    int rc = ew_check(dtype, M, N);
    if (rc) return rc;
    if (act != TPL_ACT_NONE && act != TPL_ACT_GELU) return TPL_EINVAL;
    if (!dout || !dbias || !ws || (act == TPL_ACT_GELU && (!u || !din))) return TPL_EINVAL;
    const void* ptrs[] = {dout, u, din, dbias, ws};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    if (ws_bytes < tp_layer_slice_epilogue_workspace_bytes(M, N)) return TPL_EWORKSPACE;
    hipStream_t s = (hipStream_t)hip_stream;
    const void* d = dout;
    if (act == TPL_ACT_GELU) {
        if (gelu_bwd(dtype, M, N, dout, u, din, s) != hipSuccess) return TPL_EHIP;
        d = din;
    }
    return hip_rc(colsum(dtype, M, N, d, dbias, (float*)ws, s));
}

size_t tp_layer_static_scratch_bytes(void) { return STATIC_SCRATCH_BYTES; }

int tp_layer_slice_epilogue_bwd_static(int dtype, int act, int64_t M, int64_t N, const void* dout, const void* u,
                                       void* din, void* dbias, void* hip_stream) {
    int rc = ew_check(dtype, M, N);
    if (rc) return rc;
    if (act != TPL_ACT_NONE && act != TPL_ACT_GELU) return TPL_EINVAL;
    if (!dout || !dbias || (act == TPL_ACT_GELU && (!u || !din))) return TPL_EINVAL;
    const void* ptrs[] = {dout, u, din, dbias};
    for (const void* q : ptrs) if (misaligned(q)) return TPL_EALIGN;
    // the column-sum partials must fit the static array: nothing is allocated here
    if (colsum_scratch_bytes(M, N) > STATIC_SCRATCH_BYTES) return TPL_EWORKSPACE;
    void* ws = nullptr;
    if (static_scratch(&ws) != hipSuccess) return TPL_EHIP;
    hipStream_t s = (hipStream_t)hip_stream;
    const void* d = dout;
    if (act == TPL_ACT_GELU) {
        if (gelu_bwd(dtype, M, N, dout, u, din, s) != hipSuccess) return TPL_EHIP;
        d = din;
    }
    // every partial the second stage reads is written by the first in the same call: nothing to clear
    return hip_rc(colsum(dtype, M, N, d, dbias, (float*)ws, s));
}

size_t tp_layer_gemm_workspace_bytes(int dtype, int64_t M, int64_t N, int64_t K) {
    if (M <= 0 || N <= 0 || K <= 0) return 0;
    size_t need = ALIGN;                                       // whichever operands are transposed
    for (int layout = 0; layout < 4; ++layout) need = std::max(need, gemm_ws(dtype, M, N, K, layout & 1, layout & 2));
    return need;
}

int tp_layer_gemm(int dtype, int trans_a, int trans_b, int64_t M, int64_t N, int64_t K,
                  const void* A, const void* B, void* C, const void* bias, const void* resid,
                  void* aux, int epi, void* ws, size_t ws_bytes, void* hip_stream) {
    if (dtype != TPL_F32 && dtype != TPL_BF16) return TPL_EINVAL;
    if (M <= 0 || N <= 0 || K <= 0 || !A || !B || !C || !ws) return TPL_EINVAL;
    if (epi != TPL_EPI_NONE && epi != TPL_EPI_GELU && epi != TPL_EPI_DGELU) return TPL_EINVAL;
    if (epi != TPL_EPI_NONE && !aux) return TPL_EINVAL;
    int64_t q = dtype == TPL_BF16 ? 8 : 4;
    if (M % q || N % q || K % q) return TPL_EUNSUPPORTED;
    const void* ptrs[] = {A, B, C, bias, resid, aux, ws};
    for (const void* pp : ptrs) if (misaligned(pp)) return TPL_EALIGN;
    if (ws_bytes < tp_layer_gemm_workspace_bytes(dtype, M, N, K)) return TPL_EWORKSPACE;
    GemmArgs g{};
    g.dtype = dtype; g.trans_a = trans_a != 0; g.trans_b = trans_b != 0; g.M = M; g.N = N; g.K = K;
    g.A = A; g.B = B; g.C = C; g.bias = bias; g.resid = resid; g.aux = aux; g.epi = epi;
    g.ws = ws; g.ws_bytes = ws_bytes; g.stream = (hipStream_t)hip_stream;
    return run_gemm(g);
}

// GEMMs that do not depend on each other.  One launch where the group kernels take them all.
static int group_items(int dtype, int n, const tp_layer_gemm_item* items, GemmArgs* g) {
    if (dtype != TPL_F32 && dtype != TPL_BF16) return TPL_EINVAL;
    if (n < 1 || n > 4 || !items) return TPL_EINVAL;
    const int64_t q = dtype == TPL_BF16 ? 8 : 4;
    for (int i = 0; i < n; ++i) {
        const tp_layer_gemm_item& t = items[i];
        if (t.M <= 0 || t.N <= 0 || t.K <= 0) return TPL_EINVAL;
        if (t.epi != TPL_EPI_NONE && t.epi != TPL_EPI_GELU && t.epi != TPL_EPI_DGELU) return TPL_EINVAL;
        if (t.M % q || t.N % q || t.K % q) return TPL_EUNSUPPORTED;
        g[i] = GemmArgs{};
        g[i].dtype = dtype; g[i].trans_a = t.trans_a != 0; g[i].trans_b = t.trans_b != 0; g[i].M = t.M; g[i].N = t.N; g[i].K = t.K;
        g[i].A = t.A; g[i].B = t.B; g[i].C = t.C; g[i].bias = t.bias; g[i].resid = t.resid; g[i].aux = t.aux; g[i].epi = t.epi;
    }
    return TPL_OK;
}
static bool items_in_one_launch(int n, const GemmArgs* g) {
    const Options& o = options();
    if (n < 2 || o.gemm_group == 0 || o.gemm_tile >= 0 || o.gemm_shares > 0 || o.gemm_force[0] || o.gemm_band > 0) return false;
    for (int i = 0; i < n; ++i)
        if ((g[i].trans_a && g[i].trans_b) || !(g[i].dtype == BF16 ? gemm_bf16_supported(g[i]) : gemm_f32_supported(g[i]))) return false;
    return true;
}
size_t tp_layer_gemm_group_workspace_bytes(int dtype, int n, const tp_layer_gemm_item* items) {
    GemmArgs g[4];
    if (group_items(dtype, n, items, g) != TPL_OK) return 0;
    if (items_in_one_launch(n, g)) return std::max(ALIGN, up(dtype == TPL_BF16 ? gemm_bf16_group_workspace_bytes(g, n) : gemm_f32_group_workspace_bytes(g, n)));
    size_t need = ALIGN;
    for (int i = 0; i < n; ++i) need = std::max(need, gemm_ws(dtype, g[i].M, g[i].N, g[i].K, g[i].trans_a, g[i].trans_b));
    return need;
}
int tp_layer_gemm_group(int dtype, int n, const tp_layer_gemm_item* items, void* ws, size_t ws_bytes, void* hip_stream) {
    GemmArgs g[4];
    int rc = group_items(dtype, n, items, g);
    if (rc) return rc;
    if (!ws) return TPL_EINVAL;
    for (int i = 0; i < n; ++i) {
        if (!g[i].A || !g[i].B || !g[i].C || (g[i].epi != EPI_NONE && !g[i].aux)) return TPL_EINVAL;
        const void* ptrs[] = {g[i].A, g[i].B, g[i].C, g[i].bias, g[i].resid, g[i].aux, ws};
        for (const void* pp : ptrs) if (misaligned(pp)) return TPL_EALIGN;
    }
    if (ws_bytes < tp_layer_gemm_group_workspace_bytes(dtype, n, items)) return TPL_EWORKSPACE;
    const GemmScratch sc{ws, ws_bytes, (hipStream_t)hip_stream};
    if (items_in_one_launch(n, g)) return run_group(g, n, sc);
    for (int i = 0; i < n; ++i) {
        g[i].ws = ws; g[i].ws_bytes = ws_bytes; g[i].stream = sc.stream;
        if ((rc = run_gemm(g[i]))) return rc;
    }
    return TPL_OK;
}

static int attn_check(int dtype, int B, int S, int nl, int dh) {
    if (dtype != TPL_F32 && dtype != TPL_BF16) return TPL_EINVAL;
    if (B <= 0 || S <= 0 || nl <= 0 || dh <= 0) return TPL_EINVAL;
    if (dh > 256 || (int64_t)nl * dh % (dtype == TPL_BF16 ? 8 : 4)) return TPL_EUNSUPPORTED;
    return TPL_OK;
}

size_t tp_layer_attn_workspace_bytes(int dtype, int B, int S, int nl, int dh, int causal, int bwd) {
    if (attn_check(dtype, B, S, nl, dh)) return 0;
    AttnArgs a{};
    a.dtype = dtype; a.B = B; a.S = S; a.nl = nl; a.dh = dh; a.causal = causal != 0; a.own_chunking = 1;
    if (dtype != BF16 || !attn_bf16_supported(a)) return 0;
    return up(attn_bf16_workspace_bytes(a, bwd != 0));
}

int tp_layer_attn_fwd(int dtype, int B, int S, int nl, int dh, int causal, const void* qkv, void* o,
                      float* lse, void* ws, size_t ws_bytes, void* hip_stream) {
    int rc = attn_check(dtype, B, S, nl, dh);
    if (rc) return rc;
    if (!qkv || !o || !lse) return TPL_EINVAL;
    if (misaligned(qkv) || misaligned(o) || misaligned(lse) || misaligned(ws)) return TPL_EALIGN;
    if (ws && ws_bytes < tp_layer_attn_workspace_bytes(dtype, B, S, nl, dh, causal, 0)) return TPL_EWORKSPACE;
    AttnArgs a{};
    a.dtype = dtype; a.B = B; a.S = S; a.nl = nl; a.dh = dh; a.causal = causal != 0;
    a.qkv = qkv; a.o = o; a.lse = lse; a.ws = ws; a.ws_bytes = ws_bytes; a.own_chunking = 1;
    a.stream = (hipStream_t)hip_stream;
    return run_attn(a, false);
}

int tp_layer_attn_bwd(int dtype, int B, int S, int nl, int dh, int causal, const void* qkv,
                      const void* o, const float* lse, const void* d_o, void* dqkv,
                      float* d_scratch, void* ws, size_t ws_bytes, void* hip_stream) {
    int rc = attn_check(dtype, B, S, nl, dh);
    if (rc) return rc;
    if (!qkv || !o || !lse || !d_o || !dqkv || !d_scratch) return TPL_EINVAL;
    const void* ptrs[] = {qkv, o, lse, d_o, dqkv, d_scratch, ws};
    for (const void* pp : ptrs) if (misaligned(pp)) return TPL_EALIGN;
    if (ws && ws_bytes < tp_layer_attn_workspace_bytes(dtype, B, S, nl, dh, causal, 1)) return TPL_EWORKSPACE;
    AttnArgs a{};
    a.dtype = dtype; a.B = B; a.S = S; a.nl = nl; a.dh = dh; a.causal = causal != 0;
    a.qkv = qkv; a.o = const_cast<void*>(o); a.lse = const_cast<float*>(lse); a.d_o = d_o;
    a.dqkv = dqkv; a.dsum = d_scratch; a.ws = ws; a.ws_bytes = ws_bytes; a.own_chunking = 1;
    a.stream = (hipStream_t)hip_stream;
    return run_attn(a, true);
}

int tp_layer_set_option(const char* name, const char* value) {
    return set_option(name, value) ? TPL_OK : TPL_EINVAL;
}

int tp_layer_profile(int enable) {
    g_prof.on = enable != 0;
    g_prof.n = 0;
    return TPL_OK;
}

int tp_layer_profile_read(float* ms_out, int capacity, int* count) {
    if (!ms_out || !count || capacity < 0) return TPL_EINVAL;
    int n = g_prof.n < capacity ? g_prof.n : capacity;
    for (int i = 0; i < n; ++i) {
        if (hipEventSynchronize(g_prof.stop[i]) != hipSuccess) return TPL_EHIP;
        if (hipEventElapsedTime(&ms_out[i], g_prof.start[i], g_prof.stop[i]) != hipSuccess) return TPL_EHIP;
    }
    *count = n;
    g_prof.n = 0;
    return TPL_OK;
}

const char* tp_layer_strerror(int status) {
    switch (status) {
        case TPL_OK: return "ok";
        case TPL_EINVAL: return "invalid argument (null pointer, non-positive or non-dividing size)";
        case TPL_EUNSUPPORTED: return "valid layer but unsupported shape or dtype";
        case TPL_EWORKSPACE: return "workspace too small (for a *_static entry point: the problem needs more scratch than the library's static array holds)";
        case TPL_EALIGN: return "pointer not 16-byte aligned";
        case TPL_EHIP: return "HIP launch failed";
        default: return "unknown status";
    }
}

}  // extern "C"

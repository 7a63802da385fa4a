// C ABI of the community-blocked ADMM sweep: context, workspace layout, and the schedule of one
// iteration of the paper's Algorithm 1 (W-update, Z-update, U-update) as a fixed sequence of kernel
// launches on one HIP stream.  Nothing is read back from the device inside cadmm_run.
#include "../../include/cadmm.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "host_graph.h"
#include "host_partition.h"
#include "kernels.h"

using namespace cadmm;

// Scratch of cadmm_op_wgrad_noalloc: the per-chunk partial matrices of the W-gradient product, for callers that cannot
// allocate.  Every GPU the library runs on holds its own copy of this array until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress; kernels get the per-device address looked up below.
constexpr size_t kStaticScratchFloats = (size_t)18 << 20;          // 72 MiB
static __device__ __align__(256) float scratch[kStaticScratchFloats];
constexpr int kMaxDevices = 64;
constexpr size_t kReadoutBytes = 16384;                            // pinned page for small readouts
constexpr int kProfFlags = 4096;
static float* g_scratch_ptr[kMaxDevices] = {};                     // device address of `scratch` on GPU d, once looked up
static std::mutex g_scratch_mutex;
static std::atomic<uint32_t> g_turns{0};                           // how often a process-wide knob has been turned (cadmm_tune)

struct cadmm_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;
    HostGraph hg;
    bool has_graph = false, has_model = false, has_ws = false, has_data = false, has_init = false;
    // model
    int L = 0;
    std::vector<int> C;
    // agg_first[l]: layer l forms T_l as A~ (Z_{l-1} W_l), aggregating on the narrow side C_l, instead of
    // (A~ Z_{l-1}) W_l.  Its W-update then needs three aggregations of width C_l, so it pays if
    // 3 C_l < C_{l-1}.  In those layers the slot H[l] holds A~ G_l (N x C_l).
    std::vector<char> agg_first;
    int risk = 0, max_bt = 60, J = 10, dual_form = 0, schedule = 0, step_policy = 0, fista_mode = 0;
    bool u_pending = false;      // dual_form 1: the dual step of the last sweep is still to be applied
    float nu = 0, rho = 0, tau0 = 0, theta0 = 0, eta = 2;
    // workspace
    char* ws = nullptr;
    size_t ws_bytes = 0;
    // graph on the device
    int32_t* d_row_comm = nullptr;
    int32_t* d_perm = nullptr;
    int32_t* d_seg1_pos = nullptr; int32_t* d_seg1_col = nullptr; float* d_seg1_val = nullptr;
    int32_t* d_segc_row = nullptr;
    // reduction chunk tables: layer l = 1..L-1 for its Z search, l = L (rows only) for the last-layer solve with backtracking
    struct DevChunks { int4* tab = nullptr; int32_t* unit_ptr = nullptr; int32_t n = 0; };
    std::vector<DevChunks> d_chunks;
    int32_t* d_labels = nullptr;
    int32_t* d_pred = nullptr;
    int64_t* d_row_seg_ptr = nullptr;
    int32_t* d_seg_comm = nullptr;
    int32_t* d_seg_pos = nullptr;
    int64_t n_labelled = 0;
    // split rows of the CSR row list and of the segment list; side buffer for their parts
    struct DevSchedule {               // device copy of a RowSchedule
        int4* rec = nullptr; int2* ent = nullptr; int32_t* long_row = nullptr; int32_t* long_ptr = nullptr;
        int4* blocks[7] = {};          // workgroup -> rows table per lane count of a gathered row
        int64_t n_blocks[7] = {};
        int64_t xcd_start[7][9] = {};
    };
    DevSchedule d_rows, d_segs;
    float* side = nullptr;
    // state and per-layer buffers, index l = 0..L (unused slots stay null)
    std::vector<float*> Z, W, H, T, G;
    float* U = nullptr;
    float* TLprev = nullptr;
    float* tmpA = nullptr;      // N x max width: staging, G W^T
    float* tmpB = nullptr;      // N x max hidden width: gradient of the Z subproblem
    float* tmpV = nullptr;      // N x max next width
    float* P = nullptr;         // n_seg x max next width, the buffer of the layer being searched
    float* Pbuf[2] = {nullptr, nullptr};   // layers alternate: P of layer l stays until layer l+1 is done
    float* gradW = nullptr;
    std::vector<float*> Wt;     // transposes of W_2 .. W_L, kept by the W steps
    float* tn_partial = nullptr;
    size_t tn_base_floats = 0;  // largest gemm_tn_base_floats that tn_partial serves
    double* partials = nullptr;
    double* row_sums = nullptr; // RowSums of the Z gradient being searched, for up to row_sum_tiles tiles
    int row_sum_tiles = 0;
    // For products on pairs of fp16: RowRange of H_l (h_range_tiles: the tiles of the aggregation that left it, 0: it did not), of
    // tmpA and of tmpB (their room in tiles), and the right operand in operand layout.
    std::vector<uint32_t*> h_range;
    std::vector<int> h_range_room, h_range_tiles;
    uint32_t* a_range = nullptr;
    uint32_t* b_range = nullptr;
    int a_range_room = 0, b_range_room = 0;
    unsigned short* planes = nullptr;
    int* columns = nullptr;
    Unit* unitsW = nullptr;     // [L]
    Unit* unitsZ = nullptr;     // [(L-1) * M]
    Unit* unitsF = nullptr;     // [M]: the L of the last-layer solve with backtracking (fista_mode 1)
    float* fistaX = nullptr;    // N x C_L each: x_j and y_j of that solve
    float* fistaY = nullptr;
    int32_t* gates = nullptr;          // [L]: whether any community of layer l = 1..L-1 takes a Z step (floor_first)
    int32_t* run_w = nullptr;          // [L+1] each: whether layer l's W and Z steps are worth forming (launch_rest_w)
    int32_t* run_z = nullptr;
    int32_t* left_g = nullptr;         // [L+1]: whether G_l has been left since the forward pass behind which the layers rest
    int32_t* forward_bad = nullptr;    // a hidden pre-activation of the forward pass is not finite
    LayerScalars* scalars = nullptr;   // [L+1]
    int32_t* status = nullptr;
    // What the buffers hold at the moment.  base_valid: every H_l and T_l belongs to the current iterate.  gl_valid /
    // gh_valid: so does G_L / do the G_l of the hidden layers that need one.  scal_valid: so do the readout scalars.
    // stepped: an iteration has been run since the state was set from outside (there is a dual residual).
    // rest_fresh: gates and unitsW tell what the last sweep moved (behind the forward pass: nothing), and since then nothing has been written but what a sweep
    // writes; rest: the sweep being enqueued knows that.
    bool base_valid = false, gl_valid = false, gh_valid = false, scal_valid = false, stepped = false, rest_fresh = false, rest = false;
    int iter = 0;
    // The pre-activations T_l = A~ Z_{l-1} W_l are carried from one iteration to the next instead of being
    // formed anew: the W step leaves T_l - Q/tau = A~ Z_{l-1}^k W_l^{k+1}, and the Z step of layer l-1 changes
    // it by - sum_c P_(i,c) / theta_c (T_1 does not depend on any Z at all).  t1_age counts such updates since
    // the last exact evaluation (-1: the T buffers are not images of the state); after t1_refresh of them
    // everything is formed again, which bounds the rounding drift.
    int t1_age = -1;
    int t1_refresh = 16;
    // One iteration captured as a HIP graph, per variant of the launch sequence (what of the base evaluation is
    // already at hand).  Replayed by cadmm_run when the stream is not the
    // default stream; launch-bound problem sizes gain most.
    bool use_graph = true;
    int use_lowrank = 1;         // 0: never, 1: by size, 2: wherever the widths allow it
    bool use_speculative = true;
    int use_floor_first = 1;     // 0: never, 1: by size, 2: wherever the row sums allow it
    struct GraphSlot { hipGraphExec_t exec = nullptr; bool tried = false, gl_after = false, rest_after = false; };
    GraphSlot graphs[64];
    uint32_t turns = g_turns;    // of the process-wide knobs that the graphs, rest_fresh and h_range_tiles know of (follow_tuning)
    // Kernel-level calls on a stream of the caller's (cadmm_op_stream): such a call is launched there, after what the context's
    // own stream holds (own_busy: something may still run on it) and after the kernel-level call before it; whatever uses
    // the own stream next waits for it (op_busy).  op_unrecorded: the last of them was on the null stream, and the event that
    // stands for it is recorded when somebody has to wait; op_streams: that has happened, and every call has its event.
    hipStream_t op_stream = nullptr;
    bool op_stream_set = false, op_busy = false, op_unrecorded = false, op_streams = false, own_busy = false;
    hipEvent_t ev_own = nullptr, ev_op = nullptr;
    // pinned host memory, allocated when first needed and freed with the context: two pieces through which large transfers
    // are pipelined, and a page for readouts of a few values
    char* stage[2] = {nullptr, nullptr};
    hipEvent_t stage_free[2] = {nullptr, nullptr};
    char* readout = nullptr;
    int64_t large_readouts = 0;
    // optional per-kernel-class timing with HIP events on the context's stream
    bool prof_on = false;
    // Whether a launch does its work may be decided on the device (a step floor): the flag is noted when it is written, and a
    // record whose launch did not is booked as what remains of it.  flag < 0: the launch always does its work.
    struct Unless { int flag = -1; int32_t idle_value = 0; int cls = 0; double bytes = 0.0; };
    struct ProfRec { int cls; hipEvent_t a, b; double bytes, flops; Unless unless; };
    std::vector<ProfRec> prof_recs;
    std::vector<int32_t*> prof_flags;      // pinned pieces of kProfFlags noted flags each
    int prof_flags_used = 0;
    std::vector<int> gate_notes;           // [L]: the note of gates[l] in the present iteration
    std::vector<hipEvent_t> prof_pool;
    double prof_ms[CADMM_PROFILE_CLASSES] = {0};
    int64_t prof_launches[CADMM_PROFILE_CLASSES] = {0};
    double prof_bytes[CADMM_PROFILE_CLASSES] = {0};
    double prof_flops[CADMM_PROFILE_CLASSES] = {0};
};

namespace {

int fail(cadmm_ctx* c, int code, const std::string& msg) {
    if (c) c->err = msg;
    return code;
}

int hip_fail(cadmm_ctx* c, hipError_t e, const char* what) {
    return fail(c, CADMM_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(ctx, call)                                        \
    do {                                                          \
        hipError_t e_ = (call);                                   \
        if (e_ != hipSuccess) return hip_fail(ctx, e_, #call);    \
    } while (0)

struct Bump {
    char* base;
    size_t off = 0;
    template <class T>
    T* take(size_t count) {
        off = (off + 255) & ~(size_t)255;
        T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

int max_of(const std::vector<int>& v, int lo, int hi) {
    int m = 0;
    for (int i = lo; i <= hi; ++i) m = v[i] > m ? v[i] : m;
    return m;
}

SpmmSchedule schedule_of(const cadmm_ctx* c, const cadmm_ctx::DevSchedule& d, const RowSchedule& rs);

// How the Z gradient of hidden layer l is formed (z_update_hidden).  The penalty term and the row sums are cheaper in the
// product's epilogue, which moves whole 512-byte pieces of rows, than in the aggregation's (a column tile at a time; 500000 x
// 512: 2140 us with the epilogue, 1320 without), so the product comes last unless the aggregation would be the wider for it.
// Product last against aggregation last, whole iterations: widths 256, 256 2 % less time (200000 nodes) and 1 % (20000),
// 128, 128 1 and 0 %; 128, 144 2 and 1 % more, 128, 256 5 and 1 % more, 64, 80 3 and 2 % more.  Up to 64 equal columns, a tile
// or two of the aggregation, there is no difference to be seen (five iterations, 200000 nodes: 64, 64 7.86 and 7.83 ms, 48, 48
// 7.37 and 7.46; 20000 nodes 1.84 and 1.84, 1.78 and 1.79), and the aggregation stays last.
enum GradPath { kGradLowRank, kGradProduct, kGradAggregate };
bool low_rank_form(const cadmm_ctx* c, int l) {
    const int Cl = c->C[l], Cn = c->C[l + 1];
    return Cn <= kLowRankMax && Cn < Cl && Cl % 4 == 0 && Cl <= 1024;
}
// The low-rank form saves a write and two reads of an N x C_l matrix; its product walks C_l in steps of 32 in workgroups of 128
// rows, which few rows or wide layers make a long chain in few workgroups.  us per iteration with the gradient stored and not:
// 20000 rows, widths 256, 16 199 and 211, 64, 8 147 and 142, 1000, 8 426 and 438; 50000 rows 320 and 309, 202 and 195, 845 and 818;
// 100000 rows 579 and 566, 302 and 281, 1523 and 1434; 2000 rows 113 and 132, 103 and 103, 165 and 227.
bool low_rank_shape(const cadmm_ctx* c, int l) { return low_rank_form(c, l) && c->hg.N >= (c->C[l] <= 64 ? 8192 : 32768); }
bool product_last(int Cl, int Cn) { return Cn < Cl || (Cn == Cl && Cl > 64); }
GradPath grad_path(const cadmm_ctx* c, int l) {
    if (c->use_lowrank == 2 ? low_rank_form(c, l) : c->use_lowrank == 1 && low_rank_shape(c, l)) return kGradLowRank;
    return product_last(c->C[l], c->C[l + 1]) ? kGradProduct : kGradAggregate;
}
// Column tiles in which the last kernel of that path leaves the rows' sums for the search; 0: it does not, the search reads the
// gradient (narrow layers, where that is little, and so many tiles that their sums would not be).
constexpr int kMaxSumTiles = 16;
int row_tiles(const cadmm_ctx* c, int width) { return spmm_tiles(schedule_of(c, c->d_rows, c->hg.row_sched), width); }
// Whether the product that forms the gradient of layer l (kGradProduct) runs on pairs.
bool grad_on_pairs(const cadmm_ctx* c, int l) {
    const int Cl = c->C[l], Cn = c->C[l + 1];
    return gemm_nn_pair(c->hg.N, Cn, Cl) && row_tiles(c, Cn) <= c->a_range_room;
}
int sum_tiles_of(const cadmm_ctx* c, int l, GradPath path) {
    const int Cl = c->C[l];
    int tiles = 0;
    if (path == kGradLowRank) tiles = 1;
    else if (path == kGradProduct) tiles = Cl > 32 ? gemm_nn_tiles(c->hg.N, Cl, grad_on_pairs(c, l)) : 0;
    else if (Cl >= 4) tiles = spmm_tiles(schedule_of(c, c->d_rows, c->hg.row_sched), Cl);
    return tiles <= kMaxSumTiles ? tiles : 0;
}
// What the workspace is laid out for: a number of the shapes alone, so that its size does not change with the tuning knobs
// (a knob that asks for more tiles later goes without the sums).
int sum_tiles_reserved(const cadmm_ctx* c, int l) {
    const int Cl = c->C[l], Cn = c->C[l + 1];
    int tiles = 0;
    if (product_last(Cl, Cn)) tiles = std::max(1, Cl > 32 ? gemm_nn_most_tiles(c->hg.N, Cl) : 0);
    else if (Cl >= 4) tiles = spmm_default_tiles(schedule_of(c, c->d_rows, c->hg.row_sched), Cl);
    return tiles <= kMaxSumTiles ? tiles : low_rank_shape(c, l) ? 1 : 0;
}

// Rows / segments per reduction chunk of layer l: a chunk is one workgroup's share of a pass over N x C_l (its rows) or
// n_seg x C_{l+1} (its segments).  16384 elements give a workgroup sixteen 16-byte loads per lane and array, enough to
// drown its fixed costs (three barriers, block sums); smaller problems get smaller chunks down to 2048 elements, so that
// about a thousand workgroups share the pass and the chip is full.
struct ChunkShape { int64_t rows, segs; };
ChunkShape chunk_shape(const cadmm_ctx* c, int l) {
    auto share = [](int64_t count, int width) {
        int64_t e = count * width / 1024;
        e = e < 2048 ? 2048 : e > 16384 ? 16384 : e;
        e /= width;
        return e < 1 ? (int64_t)1 : e;
    };
    ChunkShape cs;
    const int sum_tiles = l == c->L ? 0 : low_rank_shape(c, l) ? 1 : sum_tiles_reserved(c, l);
    cs.rows = share(c->hg.N, sum_tiles ? 6 * sum_tiles : c->C[l]);       // (three doubles per tile)
    cs.segs = l < c->L ? share(c->hg.n_seg, c->C[l + 1]) : 0;
    if (l == c->L) {
        // the last-layer solve is bound by its chains of fp64 exponentials: a workgroup gets the rows its lanes cover at once
        // (four classes per lane, lanes per row a power of two), or as many such sets as give 2048 workgroups
        int lanes = 1;
        while (4 * lanes < c->C[l]) lanes *= 2;
        const int64_t set = 256 / lanes;
        cs.rows = set * std::max<int64_t>(1, c->hg.N / (set * 2048));
    }
    return cs;
}

// Assign every device buffer inside the workspace; with base == nullptr only the size is computed.
size_t layout(cadmm_ctx* c, char* base) {
    const HostGraph& g = c->hg;
    const int L = c->L;
    const int64_t N = g.N;
    Bump b{base};
    c->d_row_comm = b.take<int32_t>(N);
    c->d_perm = b.take<int32_t>(N);
    auto take_schedule = [&](cadmm_ctx::DevSchedule& d, const RowSchedule& rs) {
        d.rec = b.take<int4>(rs.rec.size());
        d.ent = b.take<int2>(rs.ent.size());
        d.long_row = b.take<int32_t>(rs.n_long());
        d.long_ptr = b.take<int32_t>(rs.n_long() + 1);
        for (int l = 0; l < 7; ++l) {
            d.n_blocks[l] = count_blocks(rs, l);
            d.blocks[l] = b.take<int4>((size_t)d.n_blocks[l]);
        }
    };
    take_schedule(c->d_rows, g.row_sched);
    take_schedule(c->d_segs, g.seg_sched);
    c->d_seg1_pos = b.take<int32_t>(g.seg1_pos.size());
    c->d_seg1_col = b.take<int32_t>(g.seg1_pos.size());
    c->d_seg1_val = b.take<float>(g.seg1_pos.size());
    c->d_segc_row = b.take<int32_t>(g.n_seg);
    size_t nch = 0;
    c->d_chunks.assign(L + 1, cadmm_ctx::DevChunks());
    for (int l = 1; l <= L; ++l) {
        const ChunkShape cs = chunk_shape(c, l);
        c->d_chunks[l].n = (int32_t)count_chunks(g, cs.rows, cs.segs);
        c->d_chunks[l].tab = b.take<int4>(c->d_chunks[l].n);
        c->d_chunks[l].unit_ptr = b.take<int32_t>(g.M + 1);
        nch = nch > (size_t)c->d_chunks[l].n ? nch : (size_t)c->d_chunks[l].n;
    }
    c->d_labels = b.take<int32_t>(N);
    c->d_pred = b.take<int32_t>(N);
    c->d_row_seg_ptr = b.take<int64_t>(N + 1);
    c->d_seg_comm = b.take<int32_t>(g.n_seg);
    c->d_seg_pos = b.take<int32_t>(g.n_seg);
    {
        const int64_t np_ = g.row_sched.n_parts() > g.seg_sched.n_parts() ? g.row_sched.n_parts() : g.seg_sched.n_parts();
        c->side = b.take<float>((size_t)np_ * max_of(c->C, 0, L));
    }
    c->Z.assign(L + 1, nullptr);
    c->W.assign(L + 1, nullptr);
    c->H.assign(L + 1, nullptr);
    c->T.assign(L + 1, nullptr);
    c->G.assign(L + 1, nullptr);
    for (int l = 0; l <= L; ++l) c->Z[l] = b.take<float>(N * c->C[l]);
    for (int l = 1; l <= L; ++l) {
        c->W[l] = b.take<float>((size_t)c->C[l - 1] * c->C[l]);
        c->H[l] = b.take<float>(N * (c->agg_first[l] ? c->C[l] : c->C[l - 1]));
        c->T[l] = b.take<float>(N * c->C[l]);
        c->G[l] = b.take<float>(N * c->C[l]);
    }
    c->U = b.take<float>(N * c->C[L]);
    c->TLprev = b.take<float>(N * c->C[L]);
    c->tmpA = b.take<float>(N * max_of(c->C, 0, L));
    c->tmpB = b.take<float>(N * max_of(c->C, 1, L - 1));
    c->tmpV = b.take<float>(N * max_of(c->C, 2, L));
    c->Pbuf[0] = b.take<float>(g.n_seg * max_of(c->C, 2, L));
    c->Pbuf[1] = L > 2 ? b.take<float>(g.n_seg * max_of(c->C, 2, L)) : c->Pbuf[0];
    c->P = c->Pbuf[0];
    size_t wmax = 0, tnbase = 0;
    for (int l = 1; l <= L; ++l) {
        size_t w = (size_t)c->C[l - 1] * c->C[l];
        wmax = w > wmax ? w : wmax;
        size_t t = gemm_tn_base_floats(N, c->C[l - 1], c->C[l]);
        tnbase = t > tnbase ? t : tnbase;
    }
    c->gradW = b.take<float>(wmax);
    c->Wt.assign(L + 1, nullptr);
    for (int l = 2; l <= L; ++l) c->Wt[l] = b.take<float>((size_t)c->C[l - 1] * c->C[l]);
    c->tn_partial = b.take<float>(gemm_tn_reserve(tnbase));
    c->tn_base_floats = tnbase;
    size_t np = (size_t)kReduceBlocks * kRestCand;
    const size_t np2 = nch * kRestCand;
    np = np > np2 ? np : np2;
    for (int l = 1; l <= L; ++l) {               // block results of the products that also evaluate a candidate
        const size_t np3 = (size_t)std::max(gemm_nn_blocks(N, c->C[l], false), gemm_nn_blocks(N, c->C[l], true));
        np = np > np3 ? np : np3;
    }
    c->partials = b.take<double>(np);
    c->row_sum_tiles = 0;
    for (int l = 1; l < L; ++l) c->row_sum_tiles = std::max(c->row_sum_tiles, sum_tiles_reserved(c, l));
    c->row_sums = b.take<double>((size_t)N * c->row_sum_tiles * 3);
    // RowRange and operand planes by form alone, whatever the number of rows and the tuning make of it
    const SpmmSchedule rows = schedule_of(c, c->d_rows, g.row_sched);
    size_t planes = 0;
    auto want = [&](int K, int C) {
        if (!gemm_nn_pair_form(K, C)) return false;
        planes = std::max(planes, gemm_nn_pair_planes(K, C));
        return true;
    };
    c->h_range.assign(L + 1, nullptr);
    c->h_range_room.assign(L + 1, 0);
    c->h_range_tiles.assign(L + 1, 0);
    c->a_range_room = c->b_range_room = 0;
    for (int l = 1; l <= L; ++l) {
        const int K = c->C[l - 1], Cl = c->C[l];
        if (!c->agg_first[l] && want(K, Cl)) c->h_range_room[l] = spmm_default_tiles(rows, K);
        c->h_range[l] = b.take<uint32_t>((size_t)N * c->h_range_room[l]);
        if (l < 2) continue;
        if (product_last(K, Cl) && want(Cl, K)) c->a_range_room = std::max(c->a_range_room, spmm_default_tiles(rows, Cl));
        if (want(K, Cl)) c->b_range_room = std::max({c->b_range_room, spmm_default_tiles(rows, K), gemm_nn_pair_tiles(K)});
    }
    c->a_range = b.take<uint32_t>((size_t)N * c->a_range_room);
    c->b_range = b.take<uint32_t>((size_t)N * c->b_range_room);
    c->planes = b.take<unsigned short>(planes);
    c->columns = b.take<int>(planes ? 2 * (size_t)max_of(c->C, 0, L) : 0);
    c->unitsW = b.take<Unit>(L);
    c->unitsZ = b.take<Unit>((size_t)(L - 1) * g.M);
    c->unitsF = b.take<Unit>((size_t)g.M);
    if (c->fista_mode == 1) {
        c->fistaX = b.take<float>(N * c->C[L]);
        c->fistaY = b.take<float>(N * c->C[L]);
    }
    c->gates = b.take<int32_t>(L);
    c->run_w = b.take<int32_t>(L + 1);
    c->run_z = b.take<int32_t>(L + 1);
    c->left_g = b.take<int32_t>(L + 1);
    c->forward_bad = b.take<int32_t>(1);
    c->scalars = b.take<LayerScalars>(L + 1);
    c->status = b.take<int32_t>(4);
    return (b.off + 255) & ~(size_t)255;
}

template <class T, class V>
hipError_t upload(hipStream_t s, T* dst, const V& src) {
    static_assert(sizeof(T) == sizeof(src[0]), "the device reads the host's records as they are");
    if (src.empty()) return hipSuccess;
    return hipMemcpyAsync(dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice, s);
}

// One class per kernel symbol (and role, where one symbol serves two), so that the live timings can be
// set beside a profiler's per-kernel averages.
enum ProfClass {
    P_SPMM = 0, P_SPMM_GRADZ, P_SPMM_SEG, P_GEMM_NN_128, P_GEMM_NN_128_GRADZ, P_GEMM_NN_128_TRIAL, P_GEMM_NN_32, P_GEMM_TN, P_GEMM_TN_32, P_PHI_G,
    P_G_ONLY, P_W_TRIAL, P_Z_TRIAL, P_W_STEP, P_Z_STEP, P_LAST_LAYER, P_T_CARRY, P_GEMM_GRADZ, P_OTHER
};
const char* kProfNames[CADMM_PROFILE_CLASSES] = {
    "spmm_rows_kernel[rows]", "spmm_rows_kernel[rows,gradz]", "spmm_rows_kernel[segments]", "gemm_nn_kernel<128,0|3>",
    "gemm_nn_kernel<128,1>", "gemm_nn_kernel<128,2|4>+finish", "gemm_nn_kernel<32>", "gemm_tn_kernel<128>+reduce", "gemm_tn_kernel<32>+reduce",
    "phi_G_kernel", "G_only_kernel",
    "w_trial_kernel", "z_trial_kernel", "w_step_kernel", "z_step_kernel", "last_layer_kernel", "t_carry_kernel",
    "gemm_nn_gradz_kernel", "other"};

hipEvent_t prof_event(cadmm_ctx* c) {
    if (!c->prof_pool.empty()) {
        hipEvent_t e = c->prof_pool.back();
        c->prof_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// Notes a flag of the device at this point of the stream; returns the note's number, -1 where nothing is recorded (or there is no
// memory for it: the launches then count as done).
int note_flag(cadmm_ctx* c, const int32_t* flag) {
    if (!c->prof_on || !flag) return -1;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (c->stream && (hipStreamIsCapturing(c->stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone)) return -1;
    if ((size_t)c->prof_flags_used == c->prof_flags.size() * kProfFlags) {
        int32_t* piece = nullptr;
        if (hipHostMalloc(reinterpret_cast<void**>(&piece), kProfFlags * sizeof(int32_t), hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return -1;
        }
        c->prof_flags.push_back(piece);
    }
    const int note = c->prof_flags_used++;
    launch_note_flag(c->stream, flag, c->prof_flags[note / kProfFlags] + note % kProfFlags);
    return note;
}

// Times the launches enqueued by `body` as one record of class `cls` and books its algorithmic work, or what `unless` says.
using Unless = cadmm_ctx::Unless;
template <class F>
void timed(cadmm_ctx* c, int cls, double bytes, double flops, F body, const Unless& unless = Unless()) {
    if (!c->prof_on) { body(); return; }
    hipEvent_t a = prof_event(c), b = prof_event(c);
    if (a && b) (void)hipEventRecord(a, c->stream);
    body();
    if (a && b) {
        (void)hipEventRecord(b, c->stream);
        c->prof_recs.push_back({cls, a, b, bytes, flops, unless});
    }
}

SpmmSchedule schedule_of(const cadmm_ctx* c, const cadmm_ctx::DevSchedule& d, const RowSchedule& rs) {
    SpmmSchedule sc;
    sc.n_rows = rs.n_rows();
    sc.n_parts = rs.n_parts();
    sc.rec = d.rec; sc.ent = d.ent;
    sc.n_long = rs.n_long(); sc.long_row = d.long_row; sc.long_part_ptr = d.long_ptr;
    sc.side = c->side;
    sc.n_out = &rs == &c->hg.seg_sched ? c->hg.n_seg : c->hg.N;
    sc.n_cols = c->hg.N;
    sc.group_rows = c->hg.group_rows;
    for (int l = 0; l < 7; ++l) {
        sc.blocks[l] = d.blocks[l];
        sc.n_blocks[l] = d.n_blocks[l];
        for (int k = 0; k <= 8; ++k) sc.xcd_start[l][k] = d.xcd_start[l][k];
    }
    return sc;
}

double spmm_bytes(const cadmm_ctx* c, int64_t out_rows, int width, int extra_reads) {
    // entries (column id + value), row bounds, one read of the gathered matrix, one write of the result
    return 8.0 * (double)c->hg.nnz + 16.0 * (double)out_rows + 4.0 * (double)c->hg.N * width +
           4.0 * (double)out_rows * width * (1 + extra_reads);
}

void gemm_nn(cadmm_ctx* c, const float* A, const float* B, float* out, int64_t n, int K, int C,
             const GemmEpilogue& epi = GemmEpilogue(), const Unless& unless = Unless()) {
    const int passes = epi.kind == 3 ? (out ? 2 : 1) : epi.kind ? 3 : 1;        // matrices of the result's size that are read or written
    timed(c, C > 32 ? (epi.kind == 1 ? P_GEMM_NN_128_GRADZ : P_GEMM_NN_128) : P_GEMM_NN_32,
          4.0 * ((double)n * K + (double)K * C + (double)n * C * passes), 2.0 * (double)n * K * C,
          [&] { launch_gemm_nn(c->stream, A, B, out, n, K, C, epi); }, unless);
}

SearchParams search_params(const cadmm_ctx* c) {
    SearchParams sp;
    sp.nu = c->nu;
    sp.rho = c->rho;
    sp.eta = c->eta;
    sp.max_backtrack = c->max_bt;
    sp.relax = c->step_policy == 1 ? 1 : 0;
    return sp;
}

void aggregate(cadmm_ctx* c, const float* X, float* Y, int width, const SpmmEpilogue& epi, const Unless& unless = Unless()) {
    timed(c, epi.kind ? P_SPMM_GRADZ : P_SPMM, spmm_bytes(c, c->hg.N, width, epi.kind ? 2 : 0),
          2.0 * (double)c->hg.nnz * width, [&] {
              launch_spmm(c->stream, schedule_of(c, c->d_rows, c->hg.row_sched), X, Y, width, epi);
          }, unless);
}

// H_l = A~ X, with its RowRange where the products with H_l run on pairs.  gate (may be null): where *gate is 0 it is there already,
// and so is its RowRange if the launch that formed it has left just what this one would.
void aggregate_H(cadmm_ctx* c, const float* X, int l, const int32_t* gate = nullptr) {
    SpmmEpilogue e;
    const int K = c->C[l - 1], tiles = row_tiles(c, K);
    const int left = gemm_nn_pair(c->hg.N, K, c->C[l]) && tiles <= c->h_range_room[l] ? tiles : 0;
    if (left != c->h_range_tiles[l]) gate = nullptr;
    e.gate = gate;
    if (left) e.row_range = c->h_range[l];
    c->h_range_tiles[l] = left;
    aggregate(c, X, c->H[l], K, e, Unless{note_flag(c, gate), 0, P_OTHER, 0.0});
}

// For products with a left operand whose RowRange has that many tiles (0: there is none).
PairOperands pair_operands(const cadmm_ctx* c, const uint32_t* row_range, int tiles) {
    PairOperands p;
    if (tiles > 0) { p.row_range = row_range; p.range_tiles = tiles; p.planes = c->planes; p.columns = c->columns; }
    return p;
}
PairOperands pair_of_H(const cadmm_ctx* c, int l) { return pair_operands(c, c->h_range[l], c->h_range_tiles[l]); }

// P_{(i,c)} = sum over the entries of row i in community c of A~_ij V_j, one output row per segment, in the
// (community, row) order: the segments with several entries as a row list, those with one entry as scaled copies.
void aggregate_segments(cadmm_ctx* c, const float* V, float* P, int width, const int32_t* gate = nullptr,
                        const Unless& unless = Unless()) {
    timed(c, P_SPMM_SEG, spmm_bytes(c, c->hg.n_seg, width, 0), 2.0 * (double)c->hg.nnz * width, [&] {
        SpmmEpilogue e;
        e.gate = gate;
        launch_spmm(c->stream, schedule_of(c, c->d_segs, c->hg.seg_sched), V, P, width, e);
        launch_spmm_single(c->stream, c->d_seg1_pos, c->d_seg1_col, c->d_seg1_val, V, P, (int64_t)c->hg.seg1_pos.size(),
                           width, gate);
    }, unless);
}

bool t1_reusable(const cadmm_ctx* c) { return c->t1_age >= 0 && c->t1_age < c->t1_refresh; }

GemmEpilogue forward_epilogue(const cadmm_ctx* c, int l, float* relu_out) {
    GemmEpilogue e;
    e.pair = pair_of_H(c, l);
    e.bad = c->forward_bad;
    if (relu_out) { e.kind = 3; e.Tio = relu_out; }
    return e;
}

// How the Z search of hidden layer l goes about it: what its gradient and everything after that depends on.
// gate: the step floor is tested before grad W_{l+1} and the segment products are formed (null: with the search).  From the
// forward pass on an iteration's steps reach one layer further back each time; until then a layer's gradient is below
// resolution, and without a step in any community nothing of what only a step needs is formed.  That costs two launches
// (9 us in every iteration): 1 % and less of an iteration from 2^24 entries on (65536 x 256: 0.9 ms).
struct ZSearch { GradPath path; int sum_tiles; int32_t* gate; };
ZSearch z_search(const cadmm_ctx* c, int l) {
    ZSearch z;
    z.path = grad_path(c, l);
    z.sum_tiles = sum_tiles_of(c, l, z.path);
    if (z.sum_tiles > c->row_sum_tiles) z.sum_tiles = 0;      // (the tiles' width was tuned since the workspace was laid out)
    const bool large = c->hg.N * (int64_t)c->C[l] >= (int64_t)1 << 24;
    z.gate = z.sum_tiles > 0 && (c->use_floor_first == 2 || (c->use_floor_first == 1 && large)) ? c->gates + l : nullptr;
    return z;
}

// Whether a sweep keeps track of which layers rest: where any of them looks at the step floor first.
bool tracks_rest(const cadmm_ctx* c) {
    for (int l = 1; l < c->L && c->schedule == 0; ++l)
        if (z_search(c, l).gate) return true;
    return false;
}

// T_l = A~ Z_{l-1} W_l in the association chosen for the layer.  Used by the initial forward pass and
// by every base evaluation, so that re-evaluating an unchanged point reproduces T_l bit for bit.
// relu_out (may be null): also gets relu(T_l).
void compute_T(cadmm_ctx* c, int l, bool force = false, float* relu_out = nullptr) {
    const int64_t N = c->hg.N;
    const bool carried = !force && t1_reusable(c);     // T[l] already holds A~ Z_{l-1} W_l for the current state
    if (c->agg_first[l]) {
        if (carried) return;
        gemm_nn(c, c->Z[l - 1], c->W[l], c->tmpV, N, c->C[l - 1], c->C[l]);
        aggregate(c, c->tmpV, c->T[l], c->C[l], SpmmEpilogue());
        if (relu_out) launch_relu(c->stream, c->T[l], relu_out, N * c->C[l], 1);
    } else {
        // the W step needs H_l itself; where Z_{l-1} has not moved since it was formed it is as it was
        if (l >= 2) aggregate_H(c, c->Z[l - 1], l, c->rest_fresh && !force ? z_search(c, l - 1).gate : nullptr);
        if (carried) return;
        gemm_nn(c, c->H[l], c->W[l], c->T[l], N, c->C[l - 1], c->C[l], forward_epilogue(c, l, relu_out));
    }
}

// A hidden layer in the (A~ Z) W association feeds its pre-activation gradient to the W gradient only, where
// it is formed on the fly from T_l and Z_l; a sweep therefore skips phi_G for it (phi_l is a readout).
bool gradient_on_the_fly(const cadmm_ctx* c, int l) { return l < c->L && !c->agg_first[l]; }

// H_l and T_l = H_l W_l at the current iterate.
void form_T(cadmm_ctx* c) {
    if (c->base_valid) return;
    const bool reuse = t1_reusable(c);
    for (int l = 1; l <= c->L; ++l) compute_T(c, l);
    if (!reuse) {                                // every T_l was just formed exactly
        c->t1_age = 0;
        c->gl_valid = c->rest_fresh = false;
    }
    c->base_valid = true;
}

// What a sweep starts from: H_l, T_l, the dual step if one is pending, and the gradients G_l that are not formed on the fly.
void base_eval(cadmm_ctx* c) {
    const int L = c->L;
    const int64_t N = c->hg.N;
    form_T(c);
    if (c->u_pending) c->gl_valid = false;
    if (!c->gl_valid) {
        timed(c, P_G_ONLY, 4.0 * (double)N * c->C[L] * 4, 0.0, [&] {
            launch_G_only(c->stream, c->T[L], c->Z[L], c->U, c->G[L], c->u_pending ? 1 : 0, N * c->C[L], 1, c->nu, c->rho);
        });
        c->u_pending = false;
        c->gl_valid = true;
    }
    if (!c->gh_valid) {
        for (int l = 1; l < L; ++l)
            if (!gradient_on_the_fly(c, l))
                timed(c, P_G_ONLY, 4.0 * (double)N * c->C[l] * 3, 0.0, [&] {
                    launch_G_only(c->stream, c->T[l], c->Z[l], nullptr, c->G[l], 0, N * c->C[l], 0, c->nu, c->rho);
                });
        c->gh_valid = true;
    }
}

// The readout scalars of the current iterate: every phi_l, ||Z_L - T_L||, ||T_L - T_L(previous)||, R.
void eval_scalars(cadmm_ctx* c) {
    const int L = c->L;
    const int64_t N = c->hg.N;
    if (c->scal_valid) return;
    // carried pre-activations are at hand; what the next sweep needs beside them (H_l) is its own business
    if (!t1_reusable(c)) form_T(c);
    for (int l = 1; l <= L; ++l) {
        const double cnt = (double)N * c->C[l];
        const bool fly = gradient_on_the_fly(c, l);
        timed(c, P_PHI_G, 4.0 * cnt * (l == L ? 6 : fly ? 2 : 3), 0.0, [&] {
            launch_phi_G(c->stream, c->T[l], c->Z[l], c->U, fly ? nullptr : c->G[l], c->TLprev, c->stepped ? 1 : 0,
                         (l == L && c->u_pending) ? 1 : 0, N * c->C[l], l == L, c->nu, c->rho, c->partials, c->scalars + l);
        });
    }
    c->u_pending = false;
    c->gl_valid = c->gh_valid = true;
    launch_risk(c->stream, c->Z[L], c->d_labels, N, c->C[L], c->risk, c->partials, c->scalars + L);
    c->scal_valid = true;
}

CarryArgs carry_args(const cadmm_ctx* c, int l) {
    CarryArgs k;
    k.P = c->Pbuf[(l - 1) & 1];
    k.row_seg_ptr = c->d_row_seg_ptr; k.seg_comm = c->d_seg_comm; k.seg_pos = c->d_seg_pos;
    k.units = c->unitsZ + (size_t)(l - 2) * c->hg.M; k.M = c->hg.M;
    k.gate = z_search(c, l - 1).gate;
    return k;
}

// A launch that returns where no community of layer l takes a Z step, see ZSearch.
Unless unless_gated(const cadmm_ctx* c, int l, int cls = P_OTHER, double bytes = 0.0) {
    return Unless{c->gate_notes[l], 0, cls, bytes};
}

double carry_bytes(const cadmm_ctx* c, int l) {
    return 4.0 * ((double)c->hg.n_seg * c->C[l] + 2.0 * (double)c->hg.N * c->C[l]) + 8.0 * (double)c->hg.n_seg;
}

// T_l <- A~ Z_{l-1}^{k+1} W_l^{k+1}, from the segment products P of layer l-1 and its accepted theta.
void carry_T(cadmm_ctx* c, int l) {
    if (c->t1_refresh <= 0) return;
    timed(c, P_T_CARRY, carry_bytes(c, l), 0.0,
          [&] { launch_t_carry(c->stream, c->T[l], carry_args(c, l), c->hg.N, c->C[l]); }, unless_gated(c, l - 1));
}

// The searches of later candidates: four (what a search that has moved usually needs), then `second`, then the rest up to
// max_backtrack + 1 in all; where a pass over the data is cheap against a launch, all of them at once.  At once against in
// stages, ten iterations from the initial weights: 1.80 against 1.91 ms at 1.3e5 entries (2000 x 64), 2.30 against 2.27 at
// 5.1e5 (8000 x 64), 3.42 against 3.13 at 2.0e6 (32000 x 64).  The first iterations, which move far, lose from 2.6e5 on, later
// ones gain up to 1.0e6.
template <class F>
void later_candidates(const cadmm_ctx* c, double elements, int tried, int second, F pass) {
    int left = c->max_bt + 1 - tried;
    if (left > 0 && elements <= 524288.0) { pass(left); return; }
    for (int n : {4, second, kRestCand}) {
        if (left <= 0) return;
        pass(n);
        left -= n;
    }
}

// Whether the W step of hidden layer l leaves G_l for the Z step of layer l - 1: where nothing that G_l is made of changes in
// between.  (Layer by layer, W_l moves after Z_{l-1}.)
bool leaves_gradient(const cadmm_ctx* c, int l) { return c->schedule == 0 && l >= 2; }

// W_l <- W_l - grad phi_l / tau_l with backtracking on tau_l (Section 3.1), from the T_l, H_l (or Z_{l-1}) and G_l
// in memory; leaves T_l = A~ Z_{l-1} W_l^{new}, and where the Z step of layer l - 1 follows in the same sweep, its G_l.
void w_update(cadmm_ctx* c, int l) {
    const int L = c->L;
    const int64_t N = c->hg.N;
    hipStream_t s = c->stream;
    const SearchParams sp = search_params(c);
    const int K = c->C[l - 1], Cl = c->C[l];
    const int64_t count = N * Cl;
    const int last = (l == L);
    Unit* unit = c->unitsW + (l - 1);
    // grad phi = (A~ Z_{l-1})^T G_l = Z_{l-1}^T (A~ G_l)   (A~ is symmetric)
    const float* left = c->H[l];
    const float* right = c->G[l];
    if (c->agg_first[l]) {
        aggregate(c, c->G[l], c->H[l], Cl, SpmmEpilogue());
        left = c->Z[l - 1];
        right = c->H[l];
    }
    const bool fly = gradient_on_the_fly(c, l);    // G_l = nu (relu(T_l) - Z_l) 1[T_l > 0] formed inside the product
    // where the layer rests its search is left as it ended, with no step, and its G_l as it is
    const int32_t* const run = c->rest && fly && z_search(c, l).gate ? c->run_w + l : nullptr;
    const Unless resting{note_flag(c, run), 0, P_OTHER, 0.0};
    int n_norms = 0;
    timed(c, Cl > 32 ? P_GEMM_TN : P_GEMM_TN_32,
          4.0 * ((double)N * K + (double)N * Cl * (fly ? 2 : 1) + (double)K * Cl), 2.0 * (double)N * K * Cl,
          [&] {
              n_norms = launch_gemm_tn(s, left, fly ? c->T[l] : right, c->gradW, N, K, Cl, c->tn_partial,
                                       fly ? c->Z[l] : nullptr, c->nu, c->W[l], c->partials, run);
          }, resting);
    timed(c, P_OTHER, 16.0 * n_norms, 0.0, [&] { launch_w_begin(s, c->partials, n_norms, unit, sp, run); }, resting);
    const int skip = note_flag(c, &unit->skip);                                  // a step below resolution is not taken
    float* Q = c->G[l];                                                          // G_l is no longer needed
    const bool leave_g = !last && leaves_gradient(c, l);
    // T(W - g/tau) = T - Q/tau with Q = A~ Z_{l-1} gradW
    // In a wide hidden layer the product that forms Q also evaluates the first candidate of the search and
    // takes the step on T_l speculatively (tau rarely changes once found); later kernels repair it if needed.
    const bool spec = c->use_speculative && !c->agg_first[l] && !last && Cl > 32;
    if (c->agg_first[l]) {
        gemm_nn(c, c->Z[l - 1], c->gradW, c->tmpV, N, K, Cl);
        aggregate(c, c->tmpV, Q, Cl, SpmmEpilogue());
    } else if (spec) {
        GemmEpilogue ge;
        ge.kind = 2; ge.Zl = c->Z[l]; ge.nu = c->nu; ge.Tio = c->T[l]; ge.unit = unit; ge.partials = c->partials; ge.leave_g = leave_g;
        ge.pair = pair_of_H(c, l);
        ge.gate = run;
        const bool on_pairs = ge.pair.planes && gemm_nn_pair(N, K, Cl);
        timed(c, P_GEMM_NN_128_TRIAL, 4.0 * ((double)N * K + (double)K * Cl + (leave_g ? 4.0 : 3.0) * (double)count), 2.0 * (double)N * K * Cl,
              [&] {
                  launch_gemm_nn(s, c->H[l], c->gradW, Q, N, K, Cl, ge);
                  launch_w_trial_finish(s, c->partials, (int)gemm_nn_blocks(N, Cl, on_pairs), sp, unit, c->status);
                  GemmEpilogue again;          // Q itself, only if the step was taken ahead and then rejected
                  again.unit = unit;
                  again.pair = ge.pair;
                  again.pair.ready = true;
                  launch_gemm_nn(s, c->H[l], c->gradW, Q, N, K, Cl, again);
              }, Unless{skip, 1, P_OTHER, leave_g ? 12.0 * (double)count : 0.0});
    } else {
        GemmEpilogue ge;
        ge.pair = pair_of_H(c, l);
        gemm_nn(c, c->H[l], c->gradW, Q, N, K, Cl, ge);
    }
    // one pass reads T0, Q, Z_l (and U for the last layer); passes after an accepted one return at once
    timed(c, P_W_TRIAL, spec ? 0.0 : 4.0 * (double)count * (last ? 4 : 3), 0.0, [&] {
        if (last) {
            launch_w_last_search(s, c->T[l], Q, c->Z[l], c->U, count, sp, unit, c->partials, c->status);
            return;
        }
        if (!spec) launch_w_trial(s, c->T[l], Q, c->Z[l], count, 1, sp, unit, c->partials, c->status);
        later_candidates(c, (double)count, 1, kFreshCand, [&](int n) {
            launch_w_trial(s, c->T[l], Q, c->Z[l], count, n, sp, unit, c->partials, c->status, spec ? 1 : 0);
        });
    }, Unless{skip, 1, P_OTHER, 0.0});
    // G (and the last layer's old T) is left all the same
    const double unmoved = last ? (c->schedule == 1 ? 4.0 : 5.0) : leave_g && !spec ? 3.0 : 0.0;
    timed(c, P_W_STEP, 4.0 * ((spec ? 0.0 : last ? 7.0 : leave_g ? 5.0 : 3.0) * (double)count + 3.0 * K * Cl), 0.0, [&] {
        // W^{k+1}; T_l = A~ Z^k W^{k+1}; last layer: G_L of that T_L for the Z step of layer L-1
        if (last)
            launch_w_step_last(s, c->W[l], c->Wt[l], c->gradW, K, Cl, c->T[l], Q, count, unit, c->Z[l], c->U, c->G[l],
                               c->schedule == 1 ? nullptr : c->TLprev, c->rho);
        else
            launch_w_step(s, c->W[l], c->Wt[l], c->gradW, K, Cl, c->T[l], Q, count, unit, spec ? 1 : 0, leave_g ? c->Z[l] : nullptr, c->nu);
    }, Unless{skip, 1, unmoved > 0.0 ? P_W_STEP : P_OTHER, 4.0 * unmoved * (double)count});
    if (last) c->gl_valid = true;
    else c->gh_valid = false;
}

// Z_{l,m} <- Z_{l,m} - grad psi_{l,m} / theta_{l,m} for every community of hidden layer l (Appendix A, Eqs. 3, 4, 6-8),
// from T_l, T_{l+1}, Z_{l+1}, U, W_{l+1} in memory.  Leaves the segment products in Pbuf[l & 1].
void z_update_hidden(cadmm_ctx* c, int l) {
    const int L = c->L;
    const int64_t N = c->hg.N;
    const int M = c->hg.M;
    hipStream_t s = c->stream;
    const SearchParams sp = search_params(c);
    const int Cl = c->C[l], Cn = c->C[l + 1];
    const int next_last = (l + 1 == L);
    Unit* units = c->unitsZ + (size_t)(l - 1) * M;
    const float* Wt = c->Wt[l + 1];
    c->P = c->Pbuf[l & 1];
    if (next_last ? !c->gl_valid : !leaves_gradient(c, l + 1))                 // (else the W step of layer l + 1 has left it)
        timed(c, P_G_ONLY, 4.0 * (double)N * Cn * (next_last ? 4 : 3), 0.0, [&] {
            launch_G_only(s, c->T[l + 1], c->Z[l + 1], c->U, c->G[l + 1], 0, N * Cn, next_last, c->nu, c->rho);
        });
    // grad psi (all communities at once) = nu (Z_l - relu(T_l)) + A~ G_{l+1} W_{l+1}^T; aggregate on the
    // narrower of the two widths (grad_path), the penalty term rides in the epilogue of whichever kernel comes last.
    // With a very narrow next layer the gradient is never stored: its consumers (the product with
    // W_{l+1}, the search, the step) rebuild it per element from Z_l, T_l and the N x C_{l+1} factor
    // A~ G_{l+1}, which removes a full write and two full reads of an N x C_l matrix.
    const ZSearch how = z_search(c, l);
    const GradPath path = how.path;
    const bool lowrank = path == kGradLowRank;
    const int sum_tiles = how.sum_tiles;
    double* const row_sums = sum_tiles ? c->row_sums : nullptr;
    // grad W_{l+1} runs on pairs if whatever forms the gradient can leave its RowRange
    const bool want_range = !lowrank && gemm_nn_pair(N, Cl, Cn);
    int range_tiles = 0;
    // where the layer rests the gradient is below resolution as it was
    const int32_t* const run = c->rest && how.gate ? c->run_z + l : nullptr;
    const Unless resting{note_flag(c, run), 0, P_OTHER, 0.0};
    if (lowrank) {
        SpmmEpilogue epi;
        epi.gate = run;
        aggregate(c, c->G[l + 1], c->tmpA, Cn, epi, resting);                    // A~ G_{l+1}
        timed(c, P_GEMM_GRADZ, 4.0 * (2.0 * (double)N * Cl + 2.0 * (double)N * Cn), 2.0 * (double)N * Cl * Cn, [&] {
            launch_gemm_nn_gradz(s, c->Z[l], c->T[l], c->tmpA, Wt, c->tmpV, N, Cl, Cn, c->nu, row_sums, run);
        }, resting);
    } else if (path == kGradProduct) {
        const bool on_pairs = grad_on_pairs(c, l);
        SpmmEpilogue epi;
        epi.gate = run;
        if (on_pairs) epi.row_range = c->a_range;
        aggregate(c, c->G[l + 1], c->tmpA, Cn, epi, resting);                    // A~ G_{l+1}
        GemmEpilogue ge;
        ge.gate = run;
        if (on_pairs) {
            ge.pair = pair_operands(c, c->a_range, row_tiles(c, Cn));
            if (want_range) { ge.out_range = c->b_range; range_tiles = gemm_nn_pair_tiles(Cl); }
        }
        ge.kind = 1; ge.Zl = c->Z[l]; ge.Tl = c->T[l]; ge.nu = c->nu; ge.row_sums = row_sums;
        gemm_nn(c, c->tmpA, Wt, c->tmpB, N, Cn, Cl, ge, resting);
    } else {
        GemmEpilogue ge;
        ge.gate = run;
        gemm_nn(c, c->G[l + 1], Wt, c->tmpA, N, Cn, Cl, ge, resting);            // G_{l+1} W_{l+1}^T
        SpmmEpilogue epi;
        epi.kind = 1; epi.Zl = c->Z[l]; epi.Tl = c->T[l]; epi.nu = c->nu; epi.row_sums = row_sums;
        epi.gate = run;
        if (want_range && row_tiles(c, Cl) <= c->b_range_room) { epi.row_range = c->b_range; range_tiles = row_tiles(c, Cl); }
        aggregate(c, c->tmpA, c->tmpB, Cl, epi, resting);
    }
    ZTrialArgs a;
    const cadmm_ctx::DevChunks& ct = c->d_chunks[l];
    a.chunks = ct.tab;
    a.n_chunks = ct.n;
    a.unit_chunk_ptr = ct.unit_ptr; a.M = M;
    a.segc_row = c->d_segc_row;
    a.Zl = c->Z[l]; a.gradZ = lowrank ? nullptr : c->tmpB; a.Tl = c->T[l]; a.Cl = Cl;
    a.row_sums = row_sums; a.sum_tiles = sum_tiles; a.N = N;
    a.Tn = c->T[l + 1]; a.Zn = c->Z[l + 1]; a.P = c->P; a.Cn = Cn;
    a.Gn = c->G[l + 1];
    a.next_is_last = next_last;
    a.gate = how.gate;
    a.run = run;
    a.moved = tracks_rest(c) ? c->gates + l : nullptr;
    a.sp = sp; a.units = units; a.partials = c->partials; a.status = c->status;
    if (a.gate) timed(c, P_Z_TRIAL, 4.0 * 6.0 * sum_tiles * (double)N, 0.0, [&] { launch_z_floor(s, a); }, resting);
    c->gate_notes[l] = note_flag(c, a.gate);
    const Unless gated = unless_gated(c, l);
    if (!lowrank) {
        GemmEpilogue ge;
        ge.gate = a.gate;
        ge.pair = pair_operands(c, c->b_range, range_tiles);
        gemm_nn(c, c->tmpB, c->W[l + 1], c->tmpV, N, Cl, Cn, ge, gated);         // grad W_{l+1}
    }
    aggregate_segments(c, c->tmpV, c->P, Cn, a.gate, gated);                     // A~_{r,m} (grad W) per segment
    // one pass reads Z_l, grad, T_l (or their sums) over the rows and P with T_{l+1}, Z_{l+1} (or G_L alone) over the segments
    const double zt_bytes = 4.0 * ((a.gate ? 0.0 : sum_tiles ? 6.0 * sum_tiles * (double)N : 3.0 * (double)N * Cl) +
                                   (next_last ? 2.0 : 3.0) * (double)c->hg.n_seg * Cn) + 4.0 * (double)c->hg.n_seg;
    timed(c, P_Z_TRIAL, zt_bytes, 0.0, [&] {
        launch_z_first(s, a);
        if (!next_last) later_candidates(c, (double)c->hg.n_seg * Cn, 1, kMaxCand, [&](int n) { launch_z_more(s, a, n); });
    }, gated);
    timed(c, P_Z_STEP, 4.0 * (3.0 * (double)N * Cl + (double)N + (lowrank ? (double)N * Cn : 0.0)), 0.0, [&] {
        if (lowrank) launch_z_step_lowrank(s, c->Z[l], c->T[l], c->tmpA, Wt, c->nu, c->d_row_comm, N, Cl, Cn, units, M, a.gate);
        else launch_z_step(s, c->Z[l], c->tmpB, c->d_row_comm, N, Cl, units, M, a.gate);
    }, gated);
}

// last layer Z_L (Eq. 5) and, for dual_form 0, the dual step (Eq. 2), both from Z_L^k, U^k and the T_L in memory
// carry: T_L is also brought to the new Z_{L-1} and, with dual_form 0, the G_L of the next iteration is left.
void last_layer_update(cadmm_ctx* c, bool carry) {
    const int L = c->L;
    const int64_t N = c->hg.N;
    if (c->fista_mode == 1 && c->J > 0) {
        // FISTA with backtracking on the blocks Z_{L,m}: J + 1 passes over the rows, a device-side search per step
        FistaArgs a;
        a.ZL = c->Z[L]; a.U = c->U; a.TL = c->T[L]; a.Xb = c->fistaX; a.Yb = c->fistaY; a.labels = c->d_labels;
        const cadmm_ctx::DevChunks& ct = c->d_chunks[L];                      // chunks of rows
        a.chunks = ct.tab;
        a.n_chunks = ct.n; a.unit_chunk_ptr = ct.unit_ptr; a.M = c->hg.M;
        a.CL = c->C[L]; a.risk = c->risk; a.J = c->J; a.update_u = c->dual_form == 0 ? 1 : 0; a.rho = c->rho;
        a.sp = search_params(c); a.units = c->unitsF; a.partials = c->partials; a.status = c->status;
        // Candidates per step: sixteen in stage 0, where L climbs from rho; then the current L, a pass of four, a pass
        // of the rest.  Where the rows are few the pass of four costs its launch and not its arithmetic: its candidates
        // are then evaluated with the first.  Whole runs of five iterations, eight communities, four with the first against
        // one: 3 to 5 % less time at 1e5 entries (10000 x 10: 1.56 against 1.62 ms), between 4 % less and 1 % more at 2e5
        // and 3e5, up to 8 % more at 5e5 (50000 x 10: 2.99 against 2.82 ms), 5 to 15 % more at 1e6.
        const int first = (double)N * c->C[L] <= 3.0e5 ? 4 : 1;
        timed(c, P_LAST_LAYER, 4.0 * (double)N * c->C[L] * (3.0 + 7.0 * (c->J - 1) + 6.0) + 4.0 * (double)N * (c->J + 1), 0.0, [&] {
            double t = 1.0;
            for (int stage = 0; stage <= c->J; ++stage) {
                float mom = 0.f;
                if (stage > 0) {                        // the step taken in this stage is step stage-1
                    const double tn = 0.5 * (1.0 + std::sqrt(1.0 + 4.0 * t * t));
                    mom = (float)((t - 1.0) / tn);
                    t = tn;
                }
                const int n0 = stage == 0 ? kMaxCand : stage < c->J ? first : 1;
                launch_fista_stage(c->stream, a, stage, 0, n0, mom);
                if (stage < c->J) {
                    int left = c->max_bt + 1 - n0;
                    if (n0 == 1 && left > 0) { launch_fista_stage(c->stream, a, stage, 1, 4, 0.f); left -= 4; }
                    if (left > 0) launch_fista_stage(c->stream, a, stage, 1, left > 4 ? left : 5, 0.f);
                }
            }
        });
        if (carry) carry_T(c, L);
        return;
    }
    const bool with_carry = carry && c->t1_refresh > 0;
    const CarryArgs k = with_carry ? carry_args(c, L) : CarryArgs();
    const double solve_bytes = 4.0 * (5.0 * (double)N * c->C[L] + (double)N);
    timed(c, P_LAST_LAYER, solve_bytes + (with_carry ? carry_bytes(c, L) : 0.0), 0.0, [&] {
        launch_last_layer(c->stream, c->Z[L], c->U, c->T[L], c->d_labels, N, c->C[L], c->risk, c->rho, c->J,
                          c->dual_form == 0 ? 1 : 0, with_carry ? &k : nullptr,
                          c->dual_form == 0 ? c->G[L] : nullptr);
    }, with_carry ? unless_gated(c, L - 1, P_LAST_LAYER, solve_bytes) : Unless());
    if (with_carry && c->dual_form == 0) c->gl_valid = true;
}

// Serial baseline of Section 4.1 read as a Gauss-Seidel pass: for l = 1..L first W_l, then Z_l, each from the newest
// values.  T_l is formed anew once Z_{l-1} has changed; T_{l+1} = A~ Z_l^k W_{l+1}^k comes from the base evaluation.
void sweep_layer_by_layer(cadmm_ctx* c) {
    const int L = c->L;
    const int64_t N = c->hg.N;
    base_eval(c);
    launch_relu(c->stream, c->T[L], c->TLprev, N * c->C[L], 0);       // T_L is formed anew below: keep the old one
    for (int l = 1; l <= L; ++l) {
        if (l >= 2) {
            compute_T(c, l, true);
            if (!gradient_on_the_fly(c, l))
                timed(c, P_G_ONLY, 4.0 * (double)N * c->C[l] * (l == L ? 4 : 3), 0.0, [&] {
                    launch_G_only(c->stream, c->T[l], c->Z[l], c->U, c->G[l], 0, N * c->C[l], l == L, c->nu, c->rho);
                });
        }
        w_update(c, l);
        if (l < L) z_update_hidden(c, l);
        else last_layer_update(c, false);
    }
    c->gl_valid = false;
}

// Algorithm 1: every W_l from (W^k, Z^k, U^k), then every Z_{l,m} from (W^{k+1}, Z^k, U^k), then U.
void sweep(cadmm_ctx* c) {
    if (c->schedule == 1) {
        sweep_layer_by_layer(c);
    } else {
        const int L = c->L;
        base_eval(c);
        c->rest = c->rest_fresh && tracks_rest(c);
        if (c->rest) launch_rest_w(c->stream, L, c->unitsW, c->gates, c->left_g, c->run_w, c->run_z);
        for (int l = 1; l <= L; ++l) w_update(c, l);
        if (c->rest) launch_rest_z(c->stream, L, c->unitsW, c->run_z);
        // Ascending l keeps the Z update Jacobi although Z_l is overwritten in place: layer l reads Z_{l+1}^k
        // (not yet touched) and T_l, T_{l+1}, which were formed from Z^k before any Z changed.
        for (int l = 1; l <= L - 1; ++l) {
            z_update_hidden(c, l);
            // T_l is not read again in this sweep: bring it to the new Z_{l-1} (P and theta of layer l-1)
            if (l >= 2) carry_T(c, l);
        }
        c->gl_valid = false;                         // G_L belongs to the old Z_L and U now
        last_layer_update(c, true);
    }
    c->rest = false;
    c->rest_fresh = c->t1_age >= 0 && tracks_rest(c);
    if (c->dual_form == 1) c->u_pending = true;      // applied by the next base evaluation, on the new iterates
    c->gh_valid = c->base_valid = c->scal_valid = false;
    c->stepped = true;
    if (c->t1_age >= 0) c->t1_age++;
    c->iter++;
}

int check_launch(cadmm_ctx* c, const char* where) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(c, e, where);
    return CADMM_OK;
}

// An event for the context's streams: of the context's device, whichever is current for the calling thread.
hipError_t make_event(cadmm_ctx* c, hipEvent_t* e) {
    int current = c->device;
    hipError_t r = hipGetDevice(&current);
    if (r == hipSuccess && current != c->device) r = hipSetDevice(c->device);
    if (r == hipSuccess) r = hipEventCreateWithFlags(e, hipEventDisableTiming);
    if (r != hipSuccess) *e = nullptr;
    if (current != c->device) (void)hipSetDevice(current);
    return r;
}

// Large readouts into pageable memory go through two pinned pieces: the DMA of one runs while host threads copy the other
// out.  The runtime's own path is one thread, which also takes the page faults of a fresh destination: 128 MB came out in
// 12 ms, now in 4.  From kStageMin on the pieces pay once they are there (8 MB: 0.2 ms less), and getting them pays from
// kStageGet on or with the second such readout; a program that reads 8 MB once does not wait for pinned memory.  For
// uploads, whose source is there already, the runtime's path is the faster one at any size (27 GB/s).
constexpr size_t kStageBytes = (size_t)8 << 20;
constexpr size_t kStageMin = (size_t)4 << 20;
constexpr size_t kStageGet = (size_t)16 << 20;
constexpr int64_t kStageWork = 8 * 16384;        // HostPool work that asks for eight threads

bool have_stage(cadmm_ctx* c, size_t bytes) {
    if (bytes < kStageMin || (++c->large_readouts < 2 && bytes < kStageGet)) return false;
    for (int k = 0; k < 2; ++k) {
        if (!c->stage[k] && hipHostMalloc(reinterpret_cast<void**>(&c->stage[k]), kStageBytes, hipHostMallocDefault) != hipSuccess) {
            c->stage[k] = nullptr;
            (void)hipGetLastError();
            return false;
        }
    }
    for (hipEvent_t& e : c->stage_free)
        if (!e && make_event(c, &e) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
    return true;
}

void copy_with(HostPool& pool, char* dst, const char* src, size_t bytes) {
    pool.run((int64_t)bytes, 512 << 10, [&](int64_t lo, int64_t hi, int) { std::memcpy(dst + lo, src + lo, (size_t)(hi - lo)); });
}

// device -> host, waits for the stream
int copy_out(cadmm_ctx* c, void* dst, const void* src, size_t bytes) {
    if (!have_stage(c, bytes)) {
        HIP_TRY(c, hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, c->stream));
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        return CADMM_OK;
    }
    // (Pieces of 2 MB, up to eight in flight, instead: the same to 3 % less at 4 and 8 MB, 8 % more at 12 and 16 MB, 10 % at 32.)
    const size_t n = (bytes + kStageBytes - 1) / kStageBytes;
    auto size_of = [&](size_t k) { return k + 1 < n ? kStageBytes : bytes - k * kStageBytes; };
    auto issue = [&](size_t k) {
        hipError_t e = hipMemcpyAsync(c->stage[k & 1], static_cast<const char*>(src) + k * kStageBytes, size_of(k), hipMemcpyDeviceToHost, c->stream);
        return e != hipSuccess ? e : hipEventRecord(c->stage_free[k & 1], c->stream);
    };
    for (size_t k = 0; k < n && k < 2; ++k) HIP_TRY(c, issue(k));        // on their way while the threads start
    HostPool pool(kStageWork);
    for (size_t k = 0; k < n; ++k) {
        HIP_TRY(c, hipEventSynchronize(c->stage_free[k & 1]));
        copy_with(pool, static_cast<char*>(dst) + k * kStageBytes, c->stage[k & 1], size_of(k));
        if (k + 2 < n) HIP_TRY(c, issue(k + 2));
    }
    return CADMM_OK;
}

// A page of pinned memory for small readouts (null if there is none to be had: the caller's pageable memory then serves).
char* readout_page(cadmm_ctx* c) {
    if (!c->readout && hipHostMalloc(reinterpret_cast<void**>(&c->readout), kReadoutBytes, hipHostMallocDefault) != hipSuccess) {
        c->readout = nullptr;
        (void)hipGetLastError();
    }
    return c->readout;
}

// copy an N x C matrix out in the caller's node order
int download_rows(cadmm_ctx* c, const float* src_internal, int C, float* dst_host) {
    const int64_t N = c->hg.N;
    launch_permute_rows(c->stream, src_internal, c->tmpA, c->d_perm, N, C, 1);   // tmpA[perm[r]] = src[r]
    const int rc = copy_out(c, dst_host, c->tmpA, (size_t)N * C * sizeof(float));
    if (rc != CADMM_OK) return rc;
    return check_launch(c, "download_rows");
}

int upload_rows(cadmm_ctx* c, const float* src, int on_device, int C, float* dst_internal) {
    const int64_t N = c->hg.N;
    const size_t bytes = (size_t)N * C * sizeof(float);
    HIP_TRY(c, hipMemcpyAsync(c->tmpA, src, bytes, on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, c->stream));
    launch_permute_rows(c->stream, c->tmpA, dst_internal, c->d_perm, N, C, 0);   // dst[r] = tmpA[perm[r]]
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return check_launch(c, "upload_rows");
}

// The event behind the kernel-level calls, where it has not been recorded with them.  (The null stream is the one of the current
// device; a capture that some other stream is in has nothing to do with it.)
hipError_t record_op(cadmm_ctx* c) {
    if (!c->op_unrecorded) return hipSuccess;
    int current = c->device;
    hipError_t e = hipGetDevice(&current);
    if (e == hipSuccess && current != c->device) e = hipSetDevice(c->device);
    if (e == hipSuccess) {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        e = hipEventRecord(c->ev_op, nullptr);
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    if (current != c->device) (void)hipSetDevice(current);
    if (e == hipSuccess) { c->op_unrecorded = false; c->op_streams = true; }
    return e;
}

void drop_graphs(cadmm_ctx* c) {
    bool waited = false;
    for (auto& slot : c->graphs) {
        if (slot.exec && !waited) {                  // the last iterations may still be on their way
            hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
            if (hipStreamIsCapturing(c->stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone) (void)hipStreamSynchronize(c->stream);
            waited = true;
        }
        if (slot.exec) (void)hipGraphExecDestroy(slot.exec);
        slot.exec = nullptr;
        slot.tried = false;
    }
}

// What was enqueued under other settings of the process-wide knobs, by whichever context they were turned, is neither replayed
// nor built upon: captured iterations are dropped, and nothing rests on what was left for launches of another shape.
void follow_tuning(cadmm_ctx* c) {
    const uint32_t turns = g_turns.load();
    if (c->turns == turns) return;
    c->turns = turns;
    c->rest_fresh = false;
    drop_graphs(c);
}

// Called by everything that enqueues on the context's own stream.
hipError_t own_stream(cadmm_ctx* c) {
    follow_tuning(c);
    if (!c->op_busy) return hipSuccess;
    // A capture cannot wait for work outside of it, and what runs next on the stream itself still has to.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (c->stream) {
        const hipError_t e = hipStreamIsCapturing(c->stream, &cap);
        if (e != hipSuccess) return e;
    }
    if (cap != hipStreamCaptureStatusNone) return hipSuccess;
    hipError_t e = record_op(c);
    if (e == hipSuccess) e = hipStreamWaitEvent(c->stream, c->ev_op, 0);
    if (e != hipSuccess) return e;
    c->op_busy = false;
    c->own_busy = true;              // (also where the caller is refused after this and enqueues nothing itself)
    return hipSuccess;
}

// Runs a kernel-level call on the stream chosen by cadmm_op_stream.  Launching there, instead of on the context's stream with
// both streams made to wait for each other around the call, takes two cross-queue waits out of every call (45 -> 14 us for
// a small product).  A stream that is being captured is the exception: work of the context's stream cannot be waited for
// from inside a capture, so there the context's stream is drawn into the capture and back.
// Calls on the null stream follow each other there, and it is never destroyed: one waits for another only where the stream
// changes.  Without a workspace nothing else of the context can be waiting for them, and until a call goes to another stream
// the event is not recorded with every call (2000 x 256 x 64: 11.4 -> 8.8 us a call).  The first call on another stream then waits
// for whatever the null stream holds by that time; from it on each call has its event behind it, so that a call waits for
// the one before it and not for what the program has put on the null stream since.
template <class F>
int on_op_stream(cadmm_ctx* c, const char* what, F body) {
    if (!c->op_stream_set || c->op_stream == c->stream) {
        HIP_TRY(c, own_stream(c));
        body();
        c->own_busy = true;
        return check_launch(c, what);
    }
    if (!c->op_stream) {
        int current = c->device;
        HIP_TRY(c, hipGetDevice(&current));
        if (current != c->device) return fail(c, CADMM_EHIP, std::string(what) + ": the null stream is that of another device, which is current");
    }
    for (hipEvent_t* e : {&c->ev_own, &c->ev_op})
        if (!*e) HIP_TRY(c, make_event(c, e));
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (c->op_stream) HIP_TRY(c, hipStreamIsCapturing(c->op_stream, &cap));
    if (cap != hipStreamCaptureStatusNone) {
        hipEvent_t in = nullptr, out = nullptr;
        HIP_TRY(c, make_event(c, &in));
        HIP_TRY(c, make_event(c, &out));
        HIP_TRY(c, hipEventRecord(in, c->op_stream));
        HIP_TRY(c, hipStreamWaitEvent(c->stream, in, 0));
        body();
        HIP_TRY(c, hipEventRecord(out, c->stream));
        HIP_TRY(c, hipStreamWaitEvent(c->op_stream, out, 0));
        (void)hipEventDestroy(in);
        (void)hipEventDestroy(out);
        return check_launch(c, what);
    }
    if (c->own_busy) {
        HIP_TRY(c, hipEventRecord(c->ev_own, c->stream));
        HIP_TRY(c, hipStreamWaitEvent(c->op_stream, c->ev_own, 0));
    }
    // (also where the handles are equal: a stream may have got the address of one that was destroyed)
    if (c->op_busy && !(c->op_unrecorded && !c->op_stream)) {
        HIP_TRY(c, record_op(c));
        HIP_TRY(c, hipStreamWaitEvent(c->op_stream, c->ev_op, 0));
    }
    const hipStream_t own = c->stream;
    c->stream = c->op_stream;
    body();
    c->stream = own;
    c->op_unrecorded = !c->op_stream && !c->has_ws && !c->op_streams;
    if (!c->op_unrecorded) HIP_TRY(c, hipEventRecord(c->ev_op, c->op_stream));
    c->own_busy = false;             // what the own stream held comes before what this stream holds now
    c->op_busy = true;
    return check_launch(c, what);
}

}  // namespace

extern "C" {

int cadmm_create(cadmm_ctx** out, int device, void* hip_stream) {
    if (!out) return CADMM_EINVAL;
    *out = nullptr;
    if (device >= 0) {
        int ndev = 0;
        if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) return CADMM_EHIP;
        if (hipSetDevice(device) != hipSuccess) return CADMM_EHIP;
    }
    cadmm_ctx* c = new (std::nothrow) cadmm_ctx();
    if (!c) return CADMM_ENOMEM;
    c->device = device;
    c->stream = reinterpret_cast<hipStream_t>(hip_stream);
    *out = c;
    return CADMM_OK;
}

void cadmm_destroy(cadmm_ctx* ctx) {
    if (!ctx) return;
    if (ctx->device >= 0) {
        (void)own_stream(ctx);
        (void)hipStreamSynchronize(ctx->stream);
        for (auto& r : ctx->prof_recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
        for (auto e : ctx->prof_pool) (void)hipEventDestroy(e);
        drop_graphs(ctx);
        for (int k = 0; k < 2; ++k)
            if (ctx->stage[k]) (void)hipHostFree(ctx->stage[k]);
        for (hipEvent_t e : ctx->stage_free)
            if (e) (void)hipEventDestroy(e);
        if (ctx->readout) (void)hipHostFree(ctx->readout);
        for (int32_t* piece : ctx->prof_flags) (void)hipHostFree(piece);
        if (ctx->ev_own) (void)hipEventDestroy(ctx->ev_own);
        if (ctx->ev_op) (void)hipEventDestroy(ctx->ev_op);
    }
    delete ctx;
}

const char* cadmm_last_error(cadmm_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

int cadmm_partition(cadmm_ctx* c, int64_t N, int64_t n_edges, const int32_t* src, const int32_t* dst, int32_t M,
                    int32_t* comm) {
    if (!c) return CADMM_EINVAL;
    std::string e = partition_graph(N, n_edges, src, dst, M, comm);
    if (!e.empty()) return fail(c, CADMM_EINVAL, e);
    return CADMM_OK;
}

int cadmm_build_graph(cadmm_ctx* c, int64_t N, int64_t n_edges, const int32_t* src, const int32_t* dst, int32_t M,
                      const int32_t* comm) {
    if (!c) return CADMM_EINVAL;
    if (c->has_ws) return fail(c, CADMM_EORDER, "graph cannot change after the workspace is set");
    std::string e = build_host_graph(c->hg, N, n_edges, src, dst, M, comm);
    if (!e.empty()) { c->has_graph = false; return fail(c, CADMM_EINVAL, e); }
    c->has_graph = true;
    return CADMM_OK;
}

int cadmm_graph_sizes(cadmm_ctx* c, int64_t* nnz, int64_t* n_segments, int64_t* n_halo_rows) {
    if (!c) return CADMM_EINVAL;
    if (!c->has_graph) return fail(c, CADMM_EORDER, "build_graph first");
    if (nnz) *nnz = c->hg.nnz;
    if (n_segments) *n_segments = c->hg.n_seg;
    if (n_halo_rows) *n_halo_rows = c->hg.n_halo_rows;
    return CADMM_OK;
}

int cadmm_get_graph(cadmm_ctx* c, int32_t* perm, int64_t* row_ptr, int32_t* col, float* val, int64_t* seg_ptr,
                    int32_t* seg_row, int32_t* seg_comm, int64_t* comm_row_ptr, uint8_t* neighbour) {
    if (!c) return CADMM_EINVAL;
    if (!c->has_graph) return fail(c, CADMM_EORDER, "build_graph first");
    const HostGraph& g = c->hg;
    auto cp = [](auto* dst, const auto& v) { if (dst && !v.empty()) std::memcpy(dst, v.data(), v.size() * sizeof(v[0])); };
    cp(perm, g.perm); cp(row_ptr, g.row_ptr); cp(col, g.col); cp(val, g.val);
    cp(seg_ptr, g.seg_ptr); cp(seg_row, g.seg_row); cp(seg_comm, g.seg_comm);
    cp(comm_row_ptr, g.comm_row_ptr); cp(neighbour, g.neighbour);
    return CADMM_OK;
}

int cadmm_get_segment_order(cadmm_ctx* c, int64_t* order) {
    if (!c || !order) return CADMM_EINVAL;
    if (!c->has_graph) return fail(c, CADMM_EORDER, "build_graph first");
    if (!c->hg.segc_order.empty()) std::memcpy(order, c->hg.segc_order.data(), c->hg.segc_order.size() * sizeof(int64_t));
    return CADMM_OK;
}

int cadmm_set_model(cadmm_ctx* c, const cadmm_model* m) {
    if (!c || !m || !m->C) return CADMM_EINVAL;
    if (c->has_ws) return fail(c, CADMM_EORDER, "model cannot change after the workspace is set");
    if (m->L < 2 || m->L > 64) return fail(c, CADMM_EINVAL, "L must be in [2, 64]");
    for (int l = 0; l <= m->L; ++l)
        if (m->C[l] < 1 || m->C[l] > 4096) return fail(c, CADMM_EINVAL, "layer width must be in [1, 4096]");
    if (m->C[m->L] > 64) return fail(c, CADMM_EUNSUPPORTED, "at most 64 classes");
    if (m->risk != 0 && m->risk != 1) return fail(c, CADMM_EINVAL, "risk must be 0 or 1");
    if (!(m->nu > 0) || !(m->rho > 0) || !(m->tau0 > 0) || !(m->theta0 > 0) || !(m->eta > 1))
        return fail(c, CADMM_EINVAL, "nu, rho, tau0, theta0 must be positive and eta > 1");
    if (m->max_backtrack < 0 || m->max_backtrack > 64) return fail(c, CADMM_EINVAL, "max_backtrack must be in [0, 64]");
    if (m->fista_iters < 0) return fail(c, CADMM_EINVAL, "fista_iters must be non-negative");
    if (m->dual_form != 0 && m->dual_form != 1) return fail(c, CADMM_EINVAL, "dual_form must be 0 or 1");
    if (m->schedule != 0 && m->schedule != 1) return fail(c, CADMM_EINVAL, "schedule must be 0 or 1");
    if (m->step_policy != 0 && m->step_policy != 1) return fail(c, CADMM_EINVAL, "step_policy must be 0 or 1");
    if (m->fista_mode != 0 && m->fista_mode != 1) return fail(c, CADMM_EINVAL, "fista_mode must be 0 or 1");
    c->L = m->L;
    c->C.assign(m->C, m->C + m->L + 1);
    c->risk = m->risk;
    c->nu = m->nu; c->rho = m->rho; c->tau0 = m->tau0; c->theta0 = m->theta0; c->eta = m->eta;
    c->max_bt = m->max_backtrack;
    c->J = m->fista_iters;
    c->dual_form = m->dual_form;
    c->schedule = m->schedule;
    c->step_policy = m->step_policy;
    c->fista_mode = m->fista_mode;
    c->gate_notes.assign(c->L + 1, -1);
    c->agg_first.assign(c->L + 1, 0);
    for (int l = 2; l <= c->L; ++l) c->agg_first[l] = (3 * c->C[l] < c->C[l - 1]) ? 1 : 0;
    c->has_model = true;
    return CADMM_OK;
}

int cadmm_workspace_bytes(cadmm_ctx* c, size_t* bytes) {
    if (!c || !bytes) return CADMM_EINVAL;
    if (!c->has_graph || !c->has_model) return fail(c, CADMM_EORDER, "build_graph and set_model first");
    if (c->has_ws) { *bytes = c->ws_bytes; return CADMM_OK; }
    *bytes = layout(c, nullptr);
    return CADMM_OK;
}

int cadmm_set_workspace(cadmm_ctx* c, void* dev_ptr, size_t bytes) {
    if (!c || !dev_ptr) return CADMM_EINVAL;
    if (!c->has_graph || !c->has_model) return fail(c, CADMM_EORDER, "build_graph and set_model first");
    if (c->has_ws) return fail(c, CADMM_EORDER, "workspace already set");
    if (c->device < 0) return fail(c, CADMM_EUNSUPPORTED, "host-only context (device -1) has no device path");
    if ((reinterpret_cast<uintptr_t>(dev_ptr) & 255) != 0) return fail(c, CADMM_EINVAL, "workspace must be 256-byte aligned");
    const size_t need = layout(c, nullptr);
    if (bytes < need) return fail(c, CADMM_ENOMEM, "workspace too small");
    HIP_TRY(c, hipSetDevice(c->device));
    layout(c, static_cast<char*>(dev_ptr));
    c->ws = static_cast<char*>(dev_ptr);
    c->ws_bytes = need;
    const HostGraph& g = c->hg;
    hipStream_t s = c->stream;
    HIP_TRY(c, upload(s, c->d_row_comm, g.row_comm));
    HIP_TRY(c, upload(s, c->d_perm, g.perm));
    auto upload_schedule = [&](cadmm_ctx::DevSchedule& d, const RowSchedule& rs, const BlockTable* tables) -> hipError_t {
        hipError_t e;
        for (int l = 0; l < 7; ++l) {
            const BlockTable& bt = tables[l];            // built and checked with the graph
            if ((int64_t)bt.blocks.size() != d.n_blocks[l]) return hipErrorInvalidValue;
            for (int k = 0; k <= 8; ++k) d.xcd_start[l][k] = bt.xcd_start[k];
            if ((e = upload(s, d.blocks[l], bt.blocks)) != hipSuccess) return e;
        }
        if ((e = upload(s, d.rec, rs.rec)) != hipSuccess) return e;
        if ((e = upload(s, d.ent, rs.ent)) != hipSuccess) return e;
        if ((e = upload(s, d.long_row, rs.long_row)) != hipSuccess) return e;
        return upload(s, d.long_ptr, rs.long_part_ptr);
    };
    HIP_TRY(c, upload_schedule(c->d_rows, g.row_sched, g.row_tables));
    HIP_TRY(c, upload_schedule(c->d_segs, g.seg_sched, g.seg_tables));
    HIP_TRY(c, upload(s, c->d_seg1_pos, g.seg1_pos));
    HIP_TRY(c, upload(s, c->d_seg1_col, g.seg1_col));
    HIP_TRY(c, upload(s, c->d_seg1_val, g.seg1_val));
    HIP_TRY(c, upload(s, c->d_segc_row, g.segc_row));
    std::vector<std::vector<Chunk>> tabs(c->L + 1);                 // alive until the stream has been waited for below
    std::vector<std::vector<int32_t>> ptrs(c->L + 1);
    for (int l = 1; l <= c->L; ++l) {
        const ChunkShape cs = chunk_shape(c, l);
        build_chunks(g, cs.rows, cs.segs, tabs[l], ptrs[l]);
        if ((int32_t)tabs[l].size() != c->d_chunks[l].n) return fail(c, CADMM_EINVAL, "internal error: reduction chunks");
        HIP_TRY(c, upload(s, c->d_chunks[l].tab, tabs[l]));
        HIP_TRY(c, upload(s, c->d_chunks[l].unit_ptr, ptrs[l]));
    }
    HIP_TRY(c, upload(s, c->d_row_seg_ptr, g.row_seg_ptr));
    HIP_TRY(c, upload(s, c->d_seg_comm, g.seg_comm));
    HIP_TRY(c, upload(s, c->d_seg_pos, g.seg_pos));
    HIP_TRY(c, hipMemsetAsync(c->status, 0, 4 * sizeof(int32_t), s));
    HIP_TRY(c, hipStreamSynchronize(s));     // the host vectors above must outlive the copies
    for (int l = 0; l < 7; ++l) c->hg.row_tables[l] = c->hg.seg_tables[l] = BlockTable();
    c->has_ws = true;
    return CADMM_OK;
}

int cadmm_set_data(cadmm_ctx* c, const float* X, const int32_t* labels, int x_on_device) {
    if (!c || !X || !labels) return CADMM_EINVAL;
    if (!c->has_ws) return fail(c, CADMM_EORDER, "set_workspace first");
    HIP_TRY(c, own_stream(c));
    const int64_t N = c->hg.N;
    int64_t labelled = 0;
    bool bad = false;
    const int32_t n_classes = c->C[c->L];
    for (int64_t i = 0; i < N; ++i) {
        bad |= labels[i] < -1 || labels[i] >= n_classes;
        labelled += labels[i] >= 0;
    }
    if (bad) return fail(c, CADMM_EINVAL, "label out of range");
    c->n_labelled = labelled;
    HIP_TRY(c, hipMemcpyAsync(c->d_pred, labels, (size_t)N * sizeof(int32_t), hipMemcpyHostToDevice, c->stream));
    // class ids are moved as 32-bit words
    launch_permute_rows(c->stream, reinterpret_cast<const float*>(c->d_pred), reinterpret_cast<float*>(c->d_labels), c->d_perm, N, 1, 0);
    const int rc = upload_rows(c, X, x_on_device, c->C[0], c->Z[0]);         // synchronises
    if (rc != CADMM_OK) return rc;
    c->has_data = true;
    c->has_init = false;
    return CADMM_OK;
}

int cadmm_init(cadmm_ctx* c, const float* const* W0) {
    if (!c || !W0) return CADMM_EINVAL;
    if (!c->has_data) return fail(c, CADMM_EORDER, "set_data first");
    const int L = c->L;
    const int64_t N = c->hg.N;
    hipStream_t s = c->stream;
    HIP_TRY(c, own_stream(c));
    c->rest_fresh = false;
    for (int l = 1; l <= L; ++l) {
        if (!W0[l - 1]) return fail(c, CADMM_EINVAL, "null weight pointer");
        HIP_TRY(c, hipMemcpyAsync(c->W[l], W0[l - 1], (size_t)c->C[l - 1] * c->C[l] * sizeof(float),
                                  hipMemcpyHostToDevice, s));
    }
    c->t1_age = -1;
    for (int l = 2; l <= L; ++l) launch_transpose(s, c->W[l], c->Wt[l], c->C[l - 1], c->C[l]);
    bool noted = tracks_rest(c);                                  // whether every hidden product tells of numbers that are not finite
    if (noted) HIP_TRY(c, hipMemsetAsync(c->forward_bad, 0, sizeof(int32_t), s));
    aggregate_H(c, c->Z[0], 1);                                   // A~ Z_0 never changes
    for (int l = 1; l <= L; ++l) {
        compute_T(c, l, false, l < L ? c->Z[l] : nullptr);
        if (l == L) launch_relu(s, c->T[l], c->Z[l], N * c->C[l], 0);
        else noted = noted && !c->agg_first[l] && gemm_nn_notes_bad(c->C[l]);
    }
    HIP_TRY(c, hipMemsetAsync(c->U, 0, (size_t)N * c->C[L] * sizeof(float), s));
    HIP_TRY(c, hipMemsetAsync(c->status, 0, 4 * sizeof(int32_t), s));
    launch_fill_units(s, c->unitsW, L, (double)c->tau0);
    launch_fill_units(s, c->unitsZ, (L - 1) * c->hg.M, (double)c->theta0);
    launch_fill_units(s, c->unitsF, c->hg.M, (double)c->rho);
    uint64_t ungated = 0;
    for (int l = 1; l < L; ++l) ungated |= (uint64_t)(z_search(c, l).gate == nullptr) << l;
    if (noted) launch_rest_start(s, L, c->hg.M, c->unitsW, c->unitsZ, c->gates, ungated, c->left_g, c->forward_bad);
    c->rest_fresh = noted;
    HIP_TRY(c, hipStreamSynchronize(s));                           // W0 host buffers may be freed by the caller
    c->iter = 0;
    c->base_valid = true;                                          // the forward pass left every H_l and T_l
    c->t1_age = 0;
    c->gl_valid = c->gh_valid = c->scal_valid = c->stepped = false;
    c->u_pending = false;
    c->has_init = true;
    return check_launch(c, "init");
}

int cadmm_run(cadmm_ctx* c, int32_t k) {
    if (!c || k < 0) return CADMM_EINVAL;
    if (!c->has_init) return fail(c, CADMM_EORDER, "init first");
    HIP_TRY(c, own_stream(c));
    c->own_busy = true;
    for (int i = 0; i < k; ++i) {
        const bool graphable = c->use_graph && c->stream != nullptr && !c->prof_on;
        if (!graphable) { sweep(c); continue; }
        // what the launch sequence of an iteration depends on
        const bool reuse = !c->base_valid && t1_reusable(c);
        const bool gl = c->gl_valid && (c->base_valid || reuse);
        cadmm_ctx::GraphSlot& slot = c->graphs[(c->base_valid ? 1 : 0) | (reuse ? 2 : 0) | (gl ? 4 : 0) | (c->gh_valid ? 8 : 0) |
                                               (c->u_pending ? 16 : 0) | (c->rest_fresh ? 32 : 0)];
        if (!slot.tried) {
            // capture this variant once; the capture enqueues nothing, sweep() only advances the host flags
            slot.tried = true;
            const bool bv = c->base_valid, glv = c->gl_valid, ghv = c->gh_valid, scv = c->scal_valid, st = c->stepped, up = c->u_pending, rf = c->rest_fresh;
            const int it = c->iter, age = c->t1_age;
            if (hipStreamBeginCapture(c->stream, hipStreamCaptureModeRelaxed) == hipSuccess) {
                sweep(c);
                slot.gl_after = c->gl_valid;
                slot.rest_after = c->rest_fresh;
                hipGraph_t graph = nullptr;
                hipError_t e = hipStreamEndCapture(c->stream, &graph);
                if (e == hipSuccess && graph) {
                    if (hipGraphInstantiate(&slot.exec, graph, nullptr, nullptr, 0) != hipSuccess) slot.exec = nullptr;
                    (void)hipGraphDestroy(graph);
                }
                c->base_valid = bv; c->gl_valid = glv; c->gh_valid = ghv; c->scal_valid = scv; c->stepped = st; c->u_pending = up;
                c->rest_fresh = rf;
                c->iter = it; c->t1_age = age;
            }
            (void)hipGetLastError();
        }
        if (slot.exec && hipGraphLaunch(slot.exec, c->stream) == hipSuccess) {
            // the host-side bookkeeping sweep() would have done
            if (!c->base_valid && !reuse) c->t1_age = 0;
            if (c->t1_age >= 0) c->t1_age++;
            c->gl_valid = slot.gl_after;
            c->rest_fresh = slot.rest_after;
            c->base_valid = c->gh_valid = c->scal_valid = false;
            c->stepped = true;
            c->u_pending = c->dual_form == 1;
            c->iter++;
        } else {
            sweep(c);
        }
    }
    return check_launch(c, "run");
}

int cadmm_eval(cadmm_ctx* c, cadmm_stats* out, double* layer_penalty) {
    if (!c || !out) return CADMM_EINVAL;
    if (!c->has_init) return fail(c, CADMM_EORDER, "init first");
    const int L = c->L;
    HIP_TRY(c, own_stream(c));
    eval_scalars(c);
    // the scalars and, behind them, the status word in one copy
    const size_t bytes = (size_t)(reinterpret_cast<char*>(c->status) - reinterpret_cast<char*>(c->scalars)) + 4 * sizeof(int32_t);
    std::vector<char> pageable;
    char* page = bytes <= kReadoutBytes ? readout_page(c) : nullptr;
    if (!page) { pageable.resize(bytes); page = pageable.data(); }
    HIP_TRY(c, hipMemcpyAsync(page, c->scalars, bytes, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    const LayerScalars* sc = reinterpret_cast<const LayerScalars*>(page);
    int32_t st[4];
    std::memcpy(st, page + bytes - sizeof(st), sizeof(st));
    double pen = 0.0;
    for (int l = 1; l < L; ++l) {
        pen += sc[l].phi;
        if (layer_penalty) layer_penalty[l - 1] = sc[l].phi;
    }
    out->risk = sc[L].risk;
    out->objective = sc[L].risk + pen;
    out->lagrangian = out->objective + sc[L].phi;
    out->primal_res = std::sqrt(sc[L].res2);
    out->dual_res = c->stepped ? (double)c->rho * std::sqrt(sc[L].dT2) : 0.0;
    out->iter = c->iter;
    out->status = st[0];
    if (!std::isfinite(out->lagrangian)) out->status |= CADMM_STATUS_NONFINITE;
    return check_launch(c, "eval");
}

int cadmm_predict(cadmm_ctx* c, int32_t* pred, float* logits, double* accuracy) {
    if (!c) return CADMM_EINVAL;
    if (!c->has_init) return fail(c, CADMM_EORDER, "init first");
    const int L = c->L;
    const int64_t N = c->hg.N;
    hipStream_t s = c->stream;
    HIP_TRY(c, own_stream(c));
    // forward pass of Problem 1's constraints with the current weights; the per-layer scratch of the
    // sweep is reused, so the next sweep or readout recomputes its base evaluation
    const float* in = c->Z[0];
    for (int l = 1; l <= L; ++l) {
        if (c->agg_first[l]) {
            gemm_nn(c, in, c->W[l], c->tmpV, N, c->C[l - 1], c->C[l]);
            aggregate(c, c->tmpV, c->T[l], c->C[l], SpmmEpilogue());
        } else {
            if (l >= 2) aggregate_H(c, in, l);
            // (of a hidden layer only the activation is needed)
            gemm_nn(c, c->H[l], c->W[l], l < L ? nullptr : c->T[l], N, c->C[l - 1], c->C[l], forward_epilogue(c, l, l < L ? c->G[l] : nullptr));
        }
        if (l < L) {
            if (c->agg_first[l]) launch_relu(s, c->T[l], c->G[l], N * c->C[l], 1);
            in = c->G[l];
        }
    }
    // the T and G buffers now hold the forward pass, not images of the state
    c->base_valid = c->gl_valid = c->gh_valid = c->scal_valid = c->rest_fresh = false;
    c->t1_age = -1;
    // classes in the caller's node order, and per workgroup how many labelled nodes have their label
    static_assert(kArgmaxBlocks * sizeof(int32_t) <= kReadoutBytes, "the counts fit the readout page");
    int32_t* const hits_dev = reinterpret_cast<int32_t*>(c->partials);
    launch_argmax_rows(s, c->T[L], c->d_pred, c->d_perm, c->d_labels, hits_dev, N, c->C[L]);
    std::vector<int32_t> hits_host;
    int32_t* hits = reinterpret_cast<int32_t*>(readout_page(c));
    if (!hits) { hits_host.resize(kArgmaxBlocks); hits = hits_host.data(); }
    HIP_TRY(c, hipMemcpyAsync(hits, hits_dev, kArgmaxBlocks * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    if (pred) {
        const int rc = copy_out(c, pred, c->d_pred, (size_t)N * sizeof(int32_t));
        if (rc != CADMM_OK) return rc;
    } else {
        HIP_TRY(c, hipStreamSynchronize(s));
    }
    if (accuracy) {
        int64_t hit = 0;
        for (int b = 0; b < kArgmaxBlocks; ++b) hit += hits[b];
        *accuracy = c->n_labelled ? (double)hit / (double)c->n_labelled : 0.0;
    }
    if (logits) {
        int rc = download_rows(c, c->T[L], c->C[L], logits);
        if (rc != CADMM_OK) return rc;
    }
    return check_launch(c, "predict");
}

int cadmm_get_W(cadmm_ctx* c, int32_t l, float* dst) {
    if (!c || !dst) return CADMM_EINVAL;
    if (!c->has_init) return fail(c, CADMM_EORDER, "init first");
    if (l < 1 || l > c->L) return fail(c, CADMM_EINVAL, "layer out of range");
    HIP_TRY(c, own_stream(c));
    HIP_TRY(c, hipMemcpyAsync(dst, c->W[l], (size_t)c->C[l - 1] * c->C[l] * sizeof(float), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return CADMM_OK;
}

int cadmm_get_Z(cadmm_ctx* c, int32_t l, float* dst) {
    if (!c || !dst) return CADMM_EINVAL;
    if (!c->has_data) return fail(c, CADMM_EORDER, "set_data first");
    if (l < 0 || l > c->L) return fail(c, CADMM_EINVAL, "layer out of range");
    if (l > 0 && !c->has_init) return fail(c, CADMM_EORDER, "init first");
    HIP_TRY(c, own_stream(c));
    return download_rows(c, c->Z[l], c->C[l], dst);
}

int cadmm_get_U(cadmm_ctx* c, float* dst) {
    if (!c || !dst) return CADMM_EINVAL;
    if (!c->has_init) return fail(c, CADMM_EORDER, "init first");
    HIP_TRY(c, own_stream(c));
    if (c->u_pending) base_eval(c);          // dual_form 1: the step of the last sweep rides on the base evaluation
    return download_rows(c, c->U, c->C[c->L], dst);
}

int cadmm_get_steps(cadmm_ctx* c, double* tau, double* theta, int32_t* n_trials, double* sq_grad) {
    if (!c) return CADMM_EINVAL;
    if (!c->has_init) return fail(c, CADMM_EORDER, "init first");
    const int L = c->L, M = c->hg.M;
    const int nz = (L - 1) * M;
    // unitsW and, behind it, unitsZ in one copy
    const size_t bytes = (size_t)(reinterpret_cast<char*>(c->unitsZ + nz) - reinterpret_cast<char*>(c->unitsW));
    std::vector<char> pageable;
    char* page = bytes <= kReadoutBytes ? readout_page(c) : nullptr;
    if (!page) { pageable.resize(bytes); page = pageable.data(); }
    HIP_TRY(c, hipMemcpyAsync(page, c->unitsW, bytes, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    const Unit* uw = reinterpret_cast<const Unit*>(page);
    const Unit* uz = reinterpret_cast<const Unit*>(page + bytes - nz * sizeof(Unit));
    for (int l = 0; l < L; ++l) {
        if (tau) tau[l] = uw[l].step;
        if (n_trials) n_trials[l] = uw[l].ntrials;
        if (sq_grad) sq_grad[l] = uw[l].g;
    }
    for (int i = 0; i < nz; ++i) {
        if (theta) theta[i] = uz[i].step;
        if (n_trials) n_trials[L + i] = uz[i].ntrials;
        if (sq_grad) sq_grad[L + i] = uz[i].g;
    }
    return CADMM_OK;
}

int cadmm_get_fista(cadmm_ctx* c, double* L, int32_t* n_trials) {
    if (!c) return CADMM_EINVAL;
    if (!c->has_init) return fail(c, CADMM_EORDER, "init first");
    const int M = c->hg.M;
    std::vector<Unit> u(M);
    HIP_TRY(c, hipMemcpyAsync(u.data(), c->unitsF, M * sizeof(Unit), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    for (int m = 0; m < M; ++m) {
        if (L) L[m] = u[m].step;
        if (n_trials) n_trials[m] = u[m].total + u[m].ntrials;     // the last step's count is not yet added up
    }
    return CADMM_OK;
}

int cadmm_set_state(cadmm_ctx* c, const float* const* W, const float* const* Z, const float* U, const double* tau,
                    const double* theta) {
    if (!c) return CADMM_EINVAL;
    if (!c->has_init) return fail(c, CADMM_EORDER, "init first");
    const int L = c->L, M = c->hg.M;
    hipStream_t s = c->stream;
    HIP_TRY(c, own_stream(c));
    if (c->u_pending) base_eval(c);          // finish the pending dual step before anything is overwritten
    c->t1_age = -1;
    c->rest_fresh = false;
    if (W)
        for (int l = 1; l <= L; ++l)
            if (W[l - 1])
                HIP_TRY(c, hipMemcpyAsync(c->W[l], W[l - 1], (size_t)c->C[l - 1] * c->C[l] * sizeof(float), hipMemcpyHostToDevice, s));
    if (W)
        for (int l = 2; l <= L; ++l)
            if (W[l - 1]) launch_transpose(s, c->W[l], c->Wt[l], c->C[l - 1], c->C[l]);
    if (Z)
        for (int l = 1; l <= L; ++l)
            if (Z[l - 1]) {
                int rc = upload_rows(c, Z[l - 1], 0, c->C[l], c->Z[l]);
                if (rc != CADMM_OK) return rc;
            }
    if (U) {
        int rc = upload_rows(c, U, 0, c->C[L], c->U);
        if (rc != CADMM_OK) return rc;
    }
    if (tau || theta) {
        const int nz = (L - 1) * M;
        std::vector<Unit> uw(L), uz(nz);
        HIP_TRY(c, hipMemcpyAsync(uw.data(), c->unitsW, L * sizeof(Unit), hipMemcpyDeviceToHost, s));
        if (nz) HIP_TRY(c, hipMemcpyAsync(uz.data(), c->unitsZ, nz * sizeof(Unit), hipMemcpyDeviceToHost, s));
        HIP_TRY(c, hipStreamSynchronize(s));
        if (tau) for (int l = 0; l < L; ++l) { if (!(tau[l] > 0)) return fail(c, CADMM_EINVAL, "tau must be positive"); uw[l].step = tau[l]; }
        if (theta) for (int i = 0; i < nz; ++i) { if (!(theta[i] > 0)) return fail(c, CADMM_EINVAL, "theta must be positive"); uz[i].step = theta[i]; }
        HIP_TRY(c, hipMemcpyAsync(c->unitsW, uw.data(), L * sizeof(Unit), hipMemcpyHostToDevice, s));
        if (nz) HIP_TRY(c, hipMemcpyAsync(c->unitsZ, uz.data(), nz * sizeof(Unit), hipMemcpyHostToDevice, s));
    }
    HIP_TRY(c, hipStreamSynchronize(s));
    c->base_valid = c->gl_valid = c->gh_valid = c->scal_valid = c->stepped = false;
    return CADMM_OK;
}

int cadmm_profile(cadmm_ctx* c, int enable) {
    if (!c) return CADMM_EINVAL;
    if (c->device < 0) return fail(c, CADMM_EUNSUPPORTED, "host-only context");
    c->prof_on = enable != 0;
    if (enable) {
        HIP_TRY(c, own_stream(c));               // (records of kernel-level calls are on the caller's stream)
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        for (auto& r : c->prof_recs) { c->prof_pool.push_back(r.a); c->prof_pool.push_back(r.b); }
        c->prof_recs.clear();
        c->prof_flags_used = 0;
        for (int i = 0; i < CADMM_PROFILE_CLASSES; ++i) {
            c->prof_ms[i] = 0; c->prof_launches[i] = 0; c->prof_bytes[i] = 0; c->prof_flops[i] = 0;
        }
    }
    return CADMM_OK;
}

int cadmm_get_profile(cadmm_ctx* c, double* ms, int64_t* records, double* bytes, double* flops) {
    if (!c) return CADMM_EINVAL;
    if (c->device < 0) return fail(c, CADMM_EUNSUPPORTED, "host-only context");
    HIP_TRY(c, own_stream(c));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    for (auto& r : c->prof_recs) {
        float t = 0.f;
        if (hipEventElapsedTime(&t, r.a, r.b) != hipSuccess) {
            // (recorded into a capture: there is no time)
            (void)hipGetLastError();
            (void)hipEventDestroy(r.a);
            (void)hipEventDestroy(r.b);
            continue;
        }
        const int note = r.unless.flag;
        const bool idle = note >= 0 && c->prof_flags[note / kProfFlags][note % kProfFlags] == r.unless.idle_value;
        const int cls = idle ? r.unless.cls : r.cls;
        c->prof_ms[cls] += (double)t;
        c->prof_launches[cls] += 1;
        c->prof_bytes[cls] += idle ? r.unless.bytes : r.bytes;
        c->prof_flops[cls] += idle ? 0.0 : r.flops;
        c->prof_pool.push_back(r.a);
        c->prof_pool.push_back(r.b);
    }
    c->prof_recs.clear();
    c->prof_flags_used = 0;
    for (int i = 0; i < CADMM_PROFILE_CLASSES; ++i) {
        if (ms) ms[i] = c->prof_ms[i];
        if (records) records[i] = c->prof_launches[i];
        if (bytes) bytes[i] = c->prof_bytes[i];
        if (flops) flops[i] = c->prof_flops[i];
    }
    return CADMM_OK;
}

const char* cadmm_profile_class_name(int32_t cls) {
    if (cls < 0 || cls >= CADMM_PROFILE_CLASSES) return "";
    if (get_gemm_split()) {                      // the wide products run as the 16-bit split kernels: name those
        if (cls == P_GEMM_NN_128) return "gemm_nn_pair|split_kernel<0|3>";
        if (cls == P_GEMM_NN_128_GRADZ) return "gemm_nn_pair|split_kernel<1>";
        if (cls == P_GEMM_NN_128_TRIAL) return "gemm_nn_pair|split_kernel<2|4>+finish";
        if (cls == P_GEMM_TN) return "gemm_tn_split|wide_kernel+reduce";
    }
    return kProfNames[cls];
}

int cadmm_tune(cadmm_ctx* c, const char* key, int32_t value) {
    if (!c || !key) return CADMM_EINVAL;
    if (std::strcmp(key, "use_graph") == 0) { c->use_graph = value != 0; return CADMM_OK; }
    const bool k_lowrank = std::strcmp(key, "use_lowrank") == 0, k_spec = std::strcmp(key, "use_speculative") == 0;
    const bool k_split = std::strcmp(key, "gemm_split") == 0, k_refresh = std::strcmp(key, "t1_refresh") == 0;
    const bool k_floor = std::strcmp(key, "use_floor_first") == 0;
    const bool k_tile = std::strcmp(key, "spmm_tile_cols") == 0, k_remap = std::strcmp(key, "spmm_xcd_remap") == 0;
    if (k_split || k_tile || k_remap) {              // process-wide: every context follows with its next call
        if (k_split) set_gemm_split(value);
        else if (k_tile) set_spmm_tile_cols(value);
        else set_spmm_xcd_remap(value);
        ++g_turns;
        return CADMM_OK;
    }
    if (k_lowrank || k_spec || k_refresh || k_floor) {
        // each of these changes the launch sequence of an iteration: captured iterations of this context are dropped
        if (k_lowrank) c->use_lowrank = value == 0 || value == 2 ? value : 1;
        else if (k_spec) c->use_speculative = value != 0;
        else if (k_floor) c->use_floor_first = value;
        else { c->t1_refresh = value; c->t1_age = -1; }
        c->rest_fresh = false;
        drop_graphs(c);
        return CADMM_OK;
    }
    return fail(c, CADMM_EINVAL, "unknown tuning key");
}

int cadmm_op_stream(cadmm_ctx* c, void* hip_stream) {
    if (!c) return CADMM_EINVAL;
    if (c->device < 0) return fail(c, CADMM_EUNSUPPORTED, "host-only context");
    c->op_stream = reinterpret_cast<hipStream_t>(hip_stream);
    c->op_stream_set = true;
    return CADMM_OK;
}

int cadmm_op_aggregate(cadmm_ctx* c, const float* X, int32_t width, float* Y) {
    if (!c || !X || !Y || width < 1) return CADMM_EINVAL;
    if (!c->has_ws) return fail(c, CADMM_EORDER, "set_workspace first");
    if (width > max_of(c->C, 0, c->L)) return fail(c, CADMM_ENOMEM, "width exceeds the widest layer the workspace was sized for");
    return on_op_stream(c, "op_aggregate", [&] { aggregate(c, X, Y, width, SpmmEpilogue()); });
}

int cadmm_op_aggregate_segments(cadmm_ctx* c, const float* V, int32_t width, float* P) {
    if (!c || !V || !P || width < 1) return CADMM_EINVAL;
    if (!c->has_ws) return fail(c, CADMM_EORDER, "set_workspace first");
    if (width > max_of(c->C, 0, c->L)) return fail(c, CADMM_ENOMEM, "width exceeds the widest layer the workspace was sized for");
    return on_op_stream(c, "op_aggregate_segments", [&] { aggregate_segments(c, V, P, width); });
}

int cadmm_op_transform(cadmm_ctx* c, const float* A, int64_t n, int32_t K, const float* B, int32_t C, float* out) {
    if (!c || !A || !B || !out || n < 1 || K < 1 || C < 1) return CADMM_EINVAL;
    if (c->device < 0) return fail(c, CADMM_EUNSUPPORTED, "host-only context (device -1) has no device path");
    return on_op_stream(c, "op_transform", [&] { gemm_nn(c, A, B, out, n, K, C); });
}

int cadmm_op_wgrad(cadmm_ctx* c, const float* A, const float* G, int64_t n, int32_t K, int32_t C, float* out) {
    if (!c || !A || !G || !out || n < 1 || K < 1 || C < 1) return CADMM_EINVAL;
    if (!c->has_ws) return fail(c, CADMM_EORDER, "set_workspace first");
    if (gemm_tn_base_floats(n, K, C) > c->tn_base_floats) return fail(c, CADMM_ENOMEM, "shape needs more scratch than the model reserved");
    return on_op_stream(c, "op_wgrad", [&] {
        timed(c, C > 32 ? P_GEMM_TN : P_GEMM_TN_32, 4.0 * ((double)n * K + (double)n * C + (double)K * C),
              2.0 * (double)n * K * C, [&] { launch_gemm_tn(c->stream, A, G, out, n, K, C, c->tn_partial); });
    });
}

int cadmm_op_wgrad_noalloc(cadmm_ctx* c, const float* A, const float* G, int64_t n, int32_t K, int32_t C, float* out) {
    if (!c || !A || !G || !out || n < 1 || K < 1 || C < 1) return CADMM_EINVAL;
    if (c->device < 0) return fail(c, CADMM_EUNSUPPORTED, "host-only context (device -1) has no device path");
    if (c->device >= kMaxDevices) return fail(c, CADMM_EUNSUPPORTED, "device index beyond the static scratch table");
    const size_t need = gemm_tn_base_floats(n, K, C);
    if (need > kStaticScratchFloats)
        return fail(c, CADMM_ENOMEM, "shape needs " + std::to_string(need) + " floats of scratch, the static scratch holds " +
                                         std::to_string(kStaticScratchFloats) + "; use cadmm_op_wgrad with a workspace");
    int current = -1;
    HIP_TRY(c, hipGetDevice(&current));
    if (current != c->device) HIP_TRY(c, hipSetDevice(c->device));
    float* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[c->device]) {
            // once per device, with that device current: every GPU has its own copy of the array at its own address
            void* p = nullptr;
            hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p) {
                if (current != c->device) (void)hipSetDevice(current);
                return hip_fail(c, e, "hipGetSymbolAddress(scratch)");
            }
            g_scratch_ptr[c->device] = static_cast<float*>(p);
        }
        ptr = g_scratch_ptr[c->device];
    }
    // every entry of the partial matrices that the reduction reads is written by the product first: nothing to clear
    const int rc = on_op_stream(c, "op_wgrad_noalloc", [&] { launch_gemm_tn(c->stream, A, G, out, n, K, C, ptr); });
    if (current != c->device) (void)hipSetDevice(current);
    return rc;
}

int cadmm_op_calibrate(cadmm_ctx* c, int32_t kind, const float* src, float* dst, int64_t count, int32_t reps,
                       double* rate) {
    if (!c || !dst || !rate || count < 4 || reps < 1 || kind < 0 || kind > 8) return CADMM_EINVAL;
    if (c->device < 0) return fail(c, CADMM_EUNSUPPORTED, "host-only context");
    const int blocks = 2048;
    if ((kind == 0 || kind == 8) && (!src || count % 4 != 0)) return fail(c, CADMM_EINVAL, "copy needs src and a multiple of four floats");
    if ((kind == 1 || (kind >= 4 && kind <= 7)) && count > (1 << 24)) return fail(c, CADMM_EINVAL, "at most 2^24 MFMA steps per launch");
    if (kind == 2 || kind == 3) {
        if (!c->has_ws) return fail(c, CADMM_EORDER, "set_workspace first");
        if (!src || (count != 4 && count != 8 && count != 16 && count != 32 && count != 64 && count != 128 && count != 256))
            return fail(c, CADMM_EINVAL, "gather calibration needs src and a row width of 4, 8, ... 256 floats");
    }
    HIP_TRY(c, own_stream(c));
    hipEvent_t a = nullptr, b = nullptr;
    HIP_TRY(c, hipEventCreate(&a));
    if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return fail(c, CADMM_EHIP, "hipEventCreate"); }
    double work = 0.0;
    auto once = [&] {
        if (kind == 0) { launch_stream_copy(c->stream, src, dst, count); work += 8.0 * (double)count; }
        else if (kind == 8) { launch_stream_update(c->stream, src, dst, count); work += 12.0 * (double)count; }
        else if (kind == 1) work += launch_mfma_chain(c->stream, dst, blocks, (int)count);
        else if (kind >= 4 && kind <= 7) work += launch_mfma_bf16_chain(c->stream, dst, blocks, (int)count, kind == 4 ? 0 : kind == 5 ? 4 : kind == 6 ? 6 : 8);
        else {
            const RowSchedule& rs = kind == 2 ? c->hg.row_sched : c->hg.seg_sched;
            work += launch_gather_calibration(c->stream, schedule_of(c, kind == 2 ? c->d_rows : c->d_segs, rs), rs.n_chunks(), src,
                                              (int)count, dst);
        }
    };
    once();                                     // untimed first launch
    work = 0.0;
    (void)hipEventRecord(a, c->stream);
    for (int i = 0; i < reps; ++i) once();
    (void)hipEventRecord(b, c->stream);
    hipError_t e = hipEventSynchronize(b);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    if (e != hipSuccess) return hip_fail(c, e, "op_calibrate");
    *rate = ms > 0.f ? work / ((double)ms * 1e-3) / ((kind == 1 || (kind >= 4 && kind <= 7)) ? 1e12 : 1e9) : 0.0;
    return check_launch(c, "op_calibrate");
}

}  // extern "C"

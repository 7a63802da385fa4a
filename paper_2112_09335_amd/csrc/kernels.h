// Launch wrappers of the HIP kernels (gfx950).  All pointers are device pointers; all work is
// enqueued on `s`.  Row-major fp32 matrices whose leading dimension equals their width.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace cadmm {

// A word of RowRange: the exponent field of the largest magnitude m of some entries, and the number of those that are near it, that
// is at least 2^-binades of the power of two in m, less a sixteenth of the number that are not zero (rounded up).  0: all are zero.
constexpr int kRangeBias = 1 << 20;
__device__ __forceinline__ uint32_t range_exponent(uint32_t word) { return word >> 23; }
__device__ __forceinline__ int range_reach(uint32_t word) { return (int)(word & 0x7fffffu) - kRangeBias; }
__device__ __forceinline__ uint32_t range_word(uint32_t exponent, int reach) { return exponent << 23 | (uint32_t)(reach + kRangeBias); }
__device__ __forceinline__ uint32_t magnitude_exponent(float m) { return __float_as_uint(m) >> 23 & 255; }
// From where on an entry counts as near (m: no negative number).
__device__ __forceinline__ float range_near(float m, int binades) {
    const int e = (int)magnitude_exponent(m) - binades;
    return __uint_as_float((uint32_t)(e > 0 ? e : 1) << 23);
}
// counts: near entries, and 2^16 times those that are not zero
__device__ __forceinline__ uint32_t range_word_of(float m, int counts) {
    return m > 0.f ? range_word(magnitude_exponent(m), (counts & 0xffff) - ((counts >> 16) + 15) / 16) : 0u;
}
// The value of a neighbour that has not been seen yet when steps 1, 2, 4 and 8 follow each other, in 2, 4, 8 and 16 lanes: within a
// quad by exchange, then from the mirrored place of the other quad or half (any lane of it will do).  Vector instructions, where a
// shuffle is an access to LDS.
template <int STEP>
__device__ __forceinline__ int neighbour(int v) {
    constexpr int ctrl = STEP == 1 ? 0xB1 : STEP == 2 ? 0x4E : STEP == 4 ? 0x141 : 0x140;
    return __builtin_amdgcn_update_dpp(v, v, ctrl, 0xf, 0xf, false);
}
template <int LANES, class F>
__device__ __forceinline__ int over_lanes(int v, F f) {              // f over 2 .. 16 neighbouring lanes; every one of them gets it
    v = f(v, neighbour<1>(v));
    if constexpr (LANES > 2) v = f(v, neighbour<2>(v));
    if constexpr (LANES > 4) v = f(v, neighbour<4>(v));
    if constexpr (LANES > 8) v = f(v, neighbour<8>(v));
    return v;
}
// What a part adds to the whole: entries that are near the largest of a part whose exponent is up to `binades` below the whole's
// stay near enough; of any other part (of at most 16 * few entries) none counts.
__device__ __forceinline__ int range_share(uint32_t word, uint32_t exponent, int binades, int few) {
    return word == 0 ? 0 : range_exponent(word) + binades >= exponent ? range_reach(word) : -few;
}

// ---------------------------------------------------------------- sparse aggregation (spmm.hip)
// Y[r,:] = sum_{p in [lo[r], hi[r])} val[p] * X[col[p],:]   for r < nrows.
// epilogue 0: store;  1: Y = nu * (Zl - relu(Tl)) + sum  (gradient of the Z subproblem).
// RowSums: with row_sums (epilogue 1, widths of four and more) the launch also leaves, per column tile and row, the three
// sums over the tile's columns that the search for theta needs of the gradient g just formed: sum e g with
// e = Zl - relu(Tl), sum g^2, sum Zl^2 (three doubles at row_sums + (tile * rows + row) * 3), so that the search does not
// have to read the three N x C_l matrices again.
// RowRange: with row_range (widths of four and more) the launch leaves, per column tile and row, a word (at row_range + tile *
// rows + row) that says how large the largest entries of the result are and how many come near them, for a product that takes the
// result as its left operand (gemm_nn_pair_kernel): see range_word.
// gate (may be null): the launch does nothing where *gate is 0, see ZTrialArgs.
struct SpmmEpilogue {
    int kind = 0;
    const int32_t* gate = nullptr;
    const float* Zl = nullptr;
    const float* Tl = nullptr;
    float nu = 0.f;
    double* row_sums = nullptr;
    uint32_t* row_range = nullptr;
};
// Device view of a row list laid out for the aggregation (RowSchedule on the host).  rec[i] = (first chunk, one past
// the last chunk, output row, 0) of scheduled row i; a chunk is 8 (column, value) pairs of 8 bytes, padded with
// weight zero, chunk 0 all padding.  Records from n_rows on are the parts of rows that were too long for one lane
// group: their output row is a row of `side` (n_parts x width), and a combine kernel adds a split row's parts in
// order and applies the epilogue.
// blocks[l] / n_blocks[l] / xcd_start[l]: the workgroup -> rows table for 2^l lanes per gathered row (BlockTable).
struct SpmmSchedule {
    int64_t n_rows = 0;
    int64_t n_parts = 0;
    const int4* rec = nullptr;
    const int2* ent = nullptr;
    int64_t n_long = 0;
    const int32_t* long_row = nullptr;
    const int32_t* long_part_ptr = nullptr;
    float* side = nullptr;
    int64_t n_out = 0;             // output rows
    int64_t n_cols = 0;            // rows of the gathered matrix
    double group_rows = 0.0;       // rows of the community an average gather goes to
    const int4* blocks[7] = {};
    int64_t n_blocks[7] = {};
    int64_t xcd_start[7][9] = {};
};
int spmm_tiles(const SpmmSchedule& sched, int width);          // column tiles of such a launch (width >= 4)
int spmm_default_tiles(const SpmmSchedule& sched, int width);  // the same without the tuned tile width
void launch_spmm(hipStream_t s, const SpmmSchedule& sched, const float* X, float* Y, int width, const SpmmEpilogue& epi);
// calibration: only the gathers of the row list's column stream, rows of `width` floats (4, 8, 16, ... 256) of X;
// out: 256 floats (never written in practice); returns the bytes the launch asks the memory system for
double launch_gather_calibration(hipStream_t s, const SpmmSchedule& sc, int64_t n_chunks, const float* X, int width,
                                 float* out);
// Y[pos[k], :] = val[k] * X[col[k], :] for k < n: the output rows that have a single entry.
void launch_spmm_single(hipStream_t s, const int32_t* pos, const int32_t* col, const float* val, const float* X,
                        float* Y, int64_t n, int width, const int32_t* gate = nullptr);
// columns of the feature matrix handled at a time, if fewer than the launch's own choice (0 = that choice); smaller tiles
// keep a community's share of the gathered matrix inside one XCD's L2 at the price of re-reading the entries once per tile
void set_spmm_tile_cols(int cols);
// 1: every XCD walks one contiguous slice of the workgroup table, whole communities one after the other (default);
// 0: workgroups in plain table order, which deals consecutive row blocks round-robin to the XCDs
void set_spmm_xcd_remap(int on);

// ---------------------------------------------------------------- dense contractions (gemm.hip)
struct Unit;
// out[n x C] = A[n x K] * B[K x C];  epilogue 1: out = nu * (Zl - relu(Tl)) + A B.
// epilogue 2 (hidden layer, W search): with Q = A B, t0 = Tio, t1 = t0 - Q / unit->step0 the first candidate of
// the search is evaluated in the same pass, partials[block] = nu/2 sum ((relu(t1) - Zl)^2 - (relu(t0) - Zl)^2), and
// either the step is taken ahead of the decision (unit->spec: Tio = t1, Q is not stored) or out = Q is stored.
// If the search then rejects the first candidate, a plain product with kind 0 and `unit` set forms Q after all
// (its workgroups leave at once otherwise) and w_step repairs Tio from it.  The step is only taken ahead of the
// decision when the previous search accepted its first candidate: then Q/step0 is small against Tio and
// undoing it costs one rounding; with a step0 far too small (first iterations) it would wipe out Tio.
// leave_g: where the step is taken ahead, out gets the gradient G = nu (relu(t1) - Zl) 1[t1 > 0] for the Z step of the layer
// before (launch_w_step leaves it otherwise): one more store here instead of a pass that reads two matrices again.
// Where the search takes no step at all (unit->skip) nothing reads Q: the product is not formed, out gets G with leave_g.
// epilogue 3 (forward pass): Tio = relu(A B), and out = A B unless out is null; a pass over the pre-activations of its own
// would read them once more (200000 x 256: 76 us).
// What a product needs to run on pairs of fp16 (gemm_nn_pair): RowRange of A, and scratch for B in operand layout; ready: the
// scratch holds it already.
struct PairOperands {
    const uint32_t* row_range = nullptr;
    int range_tiles = 0;
    unsigned short* planes = nullptr;    // gemm_nn_pair_planes(K, C) of them
    int* columns = nullptr;              // 2 C
    bool ready = false;
};
struct GemmEpilogue {
    int kind = 0;
    PairOperands pair;
    const float* Zl = nullptr;
    const float* Tl = nullptr;
    float nu = 0.f;
    float* Tio = nullptr;
    const Unit* unit = nullptr;
    // where *gate is 0 the result is not wanted (ZTrialArgs, launch_rest): epilogue 0 forms nothing there, epilogues 1, 2 and 4
    // form it all the same in the kernels of small products
    const int32_t* gate = nullptr;
    bool leave_g = false;
    double* partials = nullptr;
    int32_t* bad = nullptr;        // epilogue 3: set to 1 if a result is not finite, where gemm_nn_notes_bad
    double* row_sums = nullptr;    // epilogue 1, C > 32: RowSums per tile of gemm_nn_tiles(n, C, pair) column tiles
    uint32_t* out_range = nullptr;      // epilogue 1 on pairs: RowRange of the result, per tile as row_sums
};
// Whether a product with PairOperands runs on them: by form (for what is laid out), by form and size.
bool gemm_nn_pair_form(int K, int C);
bool gemm_nn_pair(int64_t n, int K, int C);
int gemm_nn_pair_tiles(int C);
size_t gemm_nn_pair_planes(int K, int C);
bool gemm_nn_notes_bad(int C);
int gemm_nn_tiles(int64_t n, int C, bool pair);        // column tiles of the launch (C > 32); pair: with PairOperands, gemm_nn_pair
int gemm_nn_most_tiles(int64_t n, int C);      // most of them, whatever set_gemm_split says
void launch_gemm_nn(hipStream_t s, const float* A, const float* B, float* out, int64_t n, int K, int C,
                    const GemmEpilogue& epi = GemmEpilogue());
// 1: products wider than 32 columns split both operands for the 16-bit matrix cores (2: into pairs of fp16 wherever the form
// allows, for tests), 0: fp32 MFMA
void set_gemm_split(int mode);
int get_gemm_split();
// calibration kernels: chains of fp32 MFMAs on registers (returns the flops of the launch; out: blocks * 256 floats),
// and a plain copy of count floats (count % 4 == 0)
double launch_mfma_chain(hipStream_t s, float* out, int blocks, int iters);
// the same with bf16 32x32x16 MFMAs, each followed by `valu` (0, 4, 6, 8) independent vector instructions
double launch_mfma_bf16_chain(hipStream_t s, float* out, int blocks, int iters, int valu);
void launch_stream_copy(hipStream_t s, const float* src, float* dst, int64_t count);
// dst = 0.999 dst + src in place (count % 4 == 0): two reads and one write-back per element
void launch_stream_update(hipStream_t s, const float* src, float* dst, int64_t count);
int64_t gemm_nn_blocks(int64_t n, int C, bool pair);   // grid size of that launch (= block results of epilogue 2)
// out[n x C] = g W with g = nu (Zl - relu(Tl)) + SG Wt, the product (grad_Z psi) W with the gradient never stored (Wt: the
// transpose of W, K1 x C; SG: n x C; C <= kLowRankMax, K1 % 4 == 0).  The rows' RowSums (one tile) are left on the way.  The operations
// that form an element of g and their order are those of launch_z_step_lowrank.  gate (may be null): nothing is formed where *gate is 0.
void launch_gemm_nn_gradz(hipStream_t s, const float* Zl, const float* Tl, const float* SG, const float* Wt,
                          float* out, int64_t n, int K1, int C, float nu, double* row_sums, const int32_t* gate);
// out[K x C] = A[n x K]^T * G[n x C]; partial: scratch of gemm_tn_scratch_floats(n,K,C) floats.
size_t gemm_tn_scratch_floats(int64_t n, int K, int C);
size_t gemm_tn_base_floats(int64_t n, int K, int C);            // what decides whether a caller's scratch will do ...
size_t gemm_tn_reserve(size_t base);                            // ... and the scratch that serves every shape of that base
// With Zl != nullptr, G holds the pre-activation T of a hidden layer and the right operand is
// nu (relu(T) - Zl) 1[T > 0], formed on the fly.  With W (K x C), norms gets block sums of ||out||^2 and ||W||^2 (pairs);
// returns how many (at most kReduceBlocks).  gate (with Zl): where *gate is 0 the result is not wanted.
int launch_gemm_tn(hipStream_t s, const float* A, const float* G, float* out, int64_t n, int K, int C,
                   float* partial, const float* Zl = nullptr, float nu = 0.f, const float* W = nullptr,
                   double* norms = nullptr, const int32_t* gate = nullptr);
// out[C x K] = in[K x C]^T (small)
void launch_transpose(hipStream_t s, const float* in, float* out, int K, int C);

// ---------------------------------------------------------------- fused elementwise + reductions (elementwise.hip)
constexpr int kReduceBlocks = 2048;      // grid of the flat reducing kernels
constexpr int kMaxCand = 16;             // step-size candidates evaluated at once in a later pass
// Candidates of the second of the later passes: a unit's first search climbs from tau0 through 11 to 21 candidates, that is the
// first one and these (ten workloads of 8 000 to 2 M nodes); so many in one pass instead of four and sixteen: 256 M entries 1.17 ms
// for 0.57 and 1.03.
constexpr int kFreshCand = 20;
constexpr int kRestCand = 64;            // most candidates a pass evaluates (in rounds of kMaxCand)
constexpr int kLowRankMax = 16;          // widest next layer for which the Z gradient is kept in low-rank form

// One step-size search ("unit"): a layer's tau, or a (layer, community)'s theta.
struct Unit {
    double step;       // current first candidate / accepted value
    double step0;      // first candidate of this iteration's search (the value the speculative step used)
    double keep;       // value accepted by the previous search (restored if this one takes no step)
    double g;          // squared gradient norm
    double bnorm;      // squared norm of the block that moves
    int32_t done;      // search finished
    int32_t skip;      // step below resolution: block stays
    int32_t ntrials;   // candidates tested this iteration
    int32_t spec;      // the previous search accepted its first candidate: a speculative step with step0 is safe
    int32_t total;     // candidates tested since the counter was cleared (the last-layer solve adds up its steps)
    int32_t fresh;     // the previous search tested no candidate (there has been none, or its step was below resolution)
    double c1, c2;     // the part of the objective's change that is quadratic in 1/step: c1 / step + c2 / step^2
};

// Readout scalars of one layer's base evaluation.
struct LayerScalars {
    double phi;        // phi_l at the base point
    double res2;       // ||Z_L - T_L||^2           (last layer only)
    double dT2;        // ||T_L - T_L(previous)||^2 (last layer only)
    double risk;       // R(Z_L, Y)                 (last layer only)
};

struct SearchParams {
    float nu, rho, eta;
    int32_t max_backtrack;
    int32_t relax;       // 1: a search starts from (last accepted value) / eta, 0: from the last accepted value
};

// phi_l and G_l at T (hidden: G = nu (relu(T)-Z) 1[T>0]; last: G = -(U + rho (Z - T))).
// last != 0 additionally accumulates ||Z-T||^2, ||T-Tprev||^2 (if have_prev) and writes Tprev = T.
// apply_dual (last layer): U += rho (Z - T) is applied first (dual ascent on the iterate just reached).
void launch_phi_G(hipStream_t s, const float* T, const float* Z, float* U, float* G, float* Tprev,
                  int have_prev, int apply_dual, int64_t count, int last, float nu, float rho, double* partials,
                  LayerScalars* out);
// G only (no reduction), same formulas; last layer: the dual step first if apply_dual.
void launch_G_only(hipStream_t s, const float* T, const float* Z, float* U, float* G, int apply_dual, int64_t count,
                   int last, float nu, float rho);
// R(Z_L, Y) summed over labelled rows -> out->risk
void launch_risk(hipStream_t s, const float* ZL, const int32_t* labels, int64_t N, int CL, int risk,
                 double* partials, LayerScalars* out);
// Which layers rest in this iteration.  A W or Z step of a hidden layer that was found below resolution is below resolution
// again, bit for bit, as long as nothing it depends on has changed, and nothing of it is formed anew.  moved[l], l = 1..L-1:
// whether any community of layer l took a Z step in the last iteration (ZTrialArgs::moved).
// launch_rest_w, before the W steps: run_w[l] = 0 where layer l did not step last time and neither Z_l nor Z_{l-1} (and with it T_l
// and H_l) has moved since, unless layer l - 1 may need G_l and it has not been left since the forward pass (left_g).  launch_rest_z, behind them: run_z[l] = 0 where Z_{l-1}, Z_l and Z_{l+1} have not moved and W_l
// and W_{l+1} have not stepped now.  Both are 1 wherever that reaches the last layer, whose Z always moves.
// launch_rest_start, behind a forward pass: Z_l = relu(T_l) to the bit, so that the gradients of the hidden layers are exactly zero
// and none of them would step; moved and the units are left as an iteration that finds that out leaves them (ungated: bit l for a
// layer that has no gate and says that it moved whether it did or not), but no G_l is.  Unless *bad:
// the pre-activations of a hidden layer are not all finite (times zero they would be no numbers).
void launch_rest_start(hipStream_t s, int L, int M, Unit* unitsW, Unit* unitsZ, int32_t* moved, uint64_t ungated, int32_t* left_g,
                       const int32_t* bad);
void launch_rest_w(hipStream_t s, int L, const Unit* unitsW, const int32_t* moved, int32_t* left_g, int32_t* run_w, int32_t* run_z);
void launch_rest_z(hipStream_t s, int L, const Unit* unitsW, int32_t* run_z);
// unit.g = ||gradW||^2, unit.bnorm = ||W||^2 from block sums (pairs), applies the step floor, starts the search.
// gate (may be null): where *gate is 0 the unit stays as it is (launch_rest_w).
void launch_w_begin(hipStream_t s, const double* partials, int n_partials, Unit* unit, SearchParams sp, const int32_t* gate);
// The whole W search of the last layer (its objective is quadratic in T): one pass over memory and the decision.
void launch_w_last_search(hipStream_t s, const float* T0, const float* Q, const float* Z, const float* U, int64_t count,
                          SearchParams sp, Unit* unit, double* partials, int32_t* status);
// One pass of the W search of a hidden layer: the next ncand candidates step*eta^j (1, 4, kFreshCand, or rounds of kMaxCand; the
// pass of four leaves a fresh search to the next one) on
// phi_l(T0 - Q/step).  speculated != 0: T0 already holds the speculative step T0 - Q/step0; the pass rebuilds
// T0 = T0 + Q/step0.
void launch_w_trial(hipStream_t s, const float* T0, const float* Q, const float* Z, int64_t count, int ncand,
                    SearchParams sp, Unit* unit, double* partials, int32_t* status, int speculated = 0);
// Sums n_partials block results of an epilogue-2 product (candidate 0 only) and takes the search decision.
void launch_w_trial_finish(hipStream_t s, double* partials, int n_partials, SearchParams sp, Unit* unit,
                           int32_t* status);
// W -= gradW/step, Wt (C x K, may be null) its transpose, T = T0 - Q/step (count_t entries); no-op if unit.skip.
// speculated != 0: T already holds T0 - Q/step0 and is only repaired if the accepted step differs.
// With Z, Q gets the gradient G = nu (relu(T) - Z) 1[T > 0] of the new T (also if the step is skipped), unless the
// product has left it there (epilogue 2 with leave_g).
void launch_w_step(hipStream_t s, float* W, float* Wt, const float* gradW, int K, int C, float* T, float* Q,
                   int64_t count_t, const Unit* unit, int speculated, const float* Z, float nu);
// The same for the last layer; it also keeps the old T in Tprev (if not null) and leaves G = -(U + rho (Z - T)) of the new
// T (also if the step is skipped).  G may be Q.
void launch_w_step_last(hipStream_t s, float* W, float* Wt, const float* gradW, int K, int C, float* T, const float* Q,
                        int64_t count_t, const Unit* unit, const float* Z, const float* U, float* G, float* Tprev, float rho);

// Z search, layer l (widths Cl, Cn = C_{l+1}).  chunks: (community, kind, begin, end); kind 0 = rows [begin, end) of the
// community, kind 1 = segments [begin, end) of the (community, row) order, grouped by community.
struct ZTrialArgs {
    const int4* chunks;
    int32_t n_chunks;
    const int32_t* unit_chunk_ptr; int32_t M;
    const int32_t* segc_row;
    const float* Zl; const float* gradZ; const float* Tl; int Cl;       // own term, rows of the community ...
    const double* row_sums = nullptr; int sum_tiles = 0; int64_t N = 0; // ... or what the gradient's kernel left of it (RowSums)
    const float* Tn; const float* Zn; const float* P; int Cn;   // next layer, per segment
    const float* Gn = nullptr;   // last next layer: G_L = -(U + rho (Z_L - T_L)), read in place of Tn and Zn
    int next_is_last;
    SearchParams sp;
    // Floor first: the step floor is tested with the rows' sums alone, before anything that only a step needs is formed
    // (grad W_{l+1}, the segment products), and *gate says whether any community takes one.
    int32_t* gate = nullptr;
    int32_t* moved = nullptr;            // without a gate: set to 1, as if one did (may be null)
    const int32_t* run = nullptr;        // with a gate (may be null): where *run is 0, *gate and the searches stay as they are (launch_rest_z)
    Unit* units;           // [M]
    double* partials;      // [n_chunks * kRestCand]
    int32_t* status;
};
// Starts the searches of all communities and applies the step floor (with row_sums and gate).
void launch_z_floor(hipStream_t s, const ZTrialArgs& a);
// Starts the searches of all communities (unless launch_z_floor has) and judges the first candidate, or the first four where
// the previous search did not accept its first; with a last next layer, all of them.
void launch_z_first(hipStream_t s, const ZTrialArgs& a);
// The next ncand candidates (4, or rounds of kMaxCand) where the next layer is hidden.
void launch_z_more(hipStream_t s, const ZTrialArgs& a, int ncand);
// Z_l[i,:] -= gradZ[i,:] / theta[comm(i)]
void launch_z_step(hipStream_t s, float* Zl, const float* gradZ, const int32_t* row_comm, int64_t N, int Cl,
                   const Unit* units, int M, const int32_t* gate);
// the same step with the gradient in its low-rank form nu (Zl - relu(Tl)) + SG Wt (SG: N x Cn, Wt: Cn x Cl)
void launch_z_step_lowrank(hipStream_t s, float* Zl, const float* Tl, const float* SG, const float* Wt, float nu,
                           const int32_t* row_comm, int64_t N, int Cl, int Cn, const Unit* units, int M, const int32_t* gate);
// Tn[i,:] -= sum over the segments (i,c) of row i of P[(i,c),:] / theta_c  (communities whose step was skipped
// contribute nothing): the pre-activation of the next layer after the Z step, without a new aggregation.
struct CarryArgs {
    const float* P = nullptr;
    const int64_t* row_seg_ptr = nullptr; const int32_t* seg_comm = nullptr; const int32_t* seg_pos = nullptr;
    const Unit* units = nullptr; int M = 0;
    const int32_t* gate = nullptr;       // may be null; where *gate is 0 no community took a step (ZTrialArgs)
};
void launch_t_carry(hipStream_t s, float* Tn, const CarryArgs& k, int64_t N, int Cn);
// Last layer (Appendix A, Eq. 5) by J FISTA steps per row, fused with the dual step (Eq. 2):
//   U_new = U + rho (Z_L - T_L),  Z_L_new = FISTA(start Z_L; c = T_L, U, rho)
// update_u = 0 leaves U alone (the dual step is then taken on the new iterates by the next base evaluation).
// carry: T_L is then brought to the new Z_{L-1}, and G (if not null; needs update_u) gets -(U_new + rho (Z_L_new - T_L_new)).
void launch_last_layer(hipStream_t s, float* ZL, float* U, float* TL, const int32_t* labels, int64_t N,
                       int CL, int risk, float rho, int J, int update_u, const CarryArgs* carry, float* G);
// Last layer by FISTA with backtracking on the block subproblem of Z_{L,m} (Appendix A, Eq. 5): one L per community
// and step, found by the device-side search over the rows of the community (chunk tables of the graph, kind 0).
// Stage `stage` of `J` steps: stage 0 evaluates 16 candidates L = rho eta^q at y_0 = Z_L; stage j = 1..J-1 takes step
// j-1 with the L found (x_j = y_{j-1} - grad / L, y_j = x_j + mom (x_j - x_{j-1})) and evaluates the current L at
// y_j; stage J takes the last step, writes Z_L (rows without label: their exact minimiser) and, with update_u, the dual
// step of Eq. 2 with the old Z_L.  more = 1 launches a pass of ncand further candidates for the searches not yet done
// (it returns at once otherwise).  Every stage is followed by the finishing kernel that takes the decisions.
struct FistaArgs {
    float* ZL; float* U; const float* TL; float* Xb; float* Yb;      // Xb, Yb: N x CL scratch (x_j and y_j)
    const int32_t* labels;
    const int4* chunks; int32_t n_chunks; const int32_t* unit_chunk_ptr; int32_t M;      // as in ZTrialArgs
    int CL, risk, J, update_u;
    float rho;
    SearchParams sp;
    Unit* units;           // [M]
    double* partials;      // [n_chunks * kRestCand]
    int32_t* status;
};
void launch_fista_stage(hipStream_t s, const FistaArgs& a, int stage, int more, int ncand, float mom);
void launch_relu(hipStream_t s, const float* T, float* Z, int64_t count, int apply_relu);
// pred[perm[r]] = class of internal row r (its largest entry, the first one on equal values); hits[b], b < kArgmaxBlocks:
// labelled rows of workgroup b whose class is their label
constexpr int kArgmaxBlocks = 512;
void launch_argmax_rows(hipStream_t s, const float* T, int32_t* pred, const int32_t* perm, const int32_t* labels, int32_t* hits,
                        int64_t N, int C);
void launch_fill_units(hipStream_t s, Unit* units, int n, double step);
// *note (pinned host memory) = *flag, at this point of the stream
void launch_note_flag(hipStream_t s, const int32_t* flag, int32_t* note);
// gather / scatter rows between caller order and internal order: dst[r,:] = src[idx[r],:] or dst[idx[r],:] = src[r,:]
void launch_permute_rows(hipStream_t s, const float* src, float* dst, const int32_t* idx, int64_t N, int C,
                         int scatter);

}  // namespace cadmm

// Fused elementwise kernels and reductions of the ADMM sweep (gfx950): subproblem values phi / psi and
// their pre-activation gradients, the step-size searches for tau_l (Section 3.1) and theta_{l,m}
// (Appendix A) run entirely on the device, the last-layer solver fused with the dual step (Eq. 5, Eq. 2).
//
// All of these are bound by HBM traffic.  State is fp32; every sum and every quantity that decides a
// step-size test is formed in fp64 from the fp32 inputs (the fp64 vector rate of the chip is far above
// what these memory-bound passes need).  Reductions are two-stage and order-fixed: each block writes its
// partial sums, a finishing kernel adds them in index order, so results are reproducible run to run.
//
// A step-size search is a sequence of passes enqueued by the host without reading anything back: a pass
// evaluates one, four or up to kRestCand candidates step*eta^j (kMaxCand of them per sweep over memory; all
// of them by two sums where the change is quadratic in 1/step), the finishing kernel picks the first that
// passes the test  value(step) - value(0) <= -||grad||^2 / (2 step)  and marks the search done; later passes
// see the flag and return at once.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace cadmm {

namespace {

constexpr double kStepFloor = 1e-12;   // a step that moves the block by less than this fraction is not taken

// Four consecutive floats per lane at any dword (the chip takes 16-byte global accesses there).
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void ldv4(float (&d)[4], const float* p) {
    const float4u v = *reinterpret_cast<const float4u*>(p);
    d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
}
__device__ __forceinline__ void stv4(float* p, const float (&d)[4]) {
    float4u v = {d[0], d[1], d[2], d[3]};
    *reinterpret_cast<float4u*>(p) = v;
}

// Flat kernels: a matrix as one array, f(i, WHOLE) for every four consecutive entries from i on; WHOLE = std::false_type for
// the last one to three, which one lane handles apart (ldq reads zeros for what is missing, which adds nothing to any sum).
template <class F>
__device__ __forceinline__ void for_quads(int64_t count, F f) {
    const int64_t whole = count & ~(int64_t)3;
    const int64_t first = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x * 4;
    for (int64_t i = first; i < whole; i += stride) f(i, std::true_type{});
    if (first == 0 && whole < count) f(whole, std::false_type{});
}
template <class WHOLE>
__device__ __forceinline__ void ldq(float (&d)[4], const float* p, int64_t left, WHOLE) {
    if constexpr (WHOLE::value) ldv4(d, p);
    else {
        d[0] = p[0];
        d[1] = left > 1 ? p[1] : 0.f;
        d[2] = left > 2 ? p[2] : 0.f;
        d[3] = 0.f;
    }
}
template <class WHOLE>
__device__ __forceinline__ void stq(float* p, const float (&d)[4], int64_t left, WHOLE) {
    if constexpr (WHOLE::value) stv4(p, d);
    else {
        p[0] = d[0];
        if (left > 1) p[1] = d[1];
        if (left > 2) p[2] = d[2];
    }
}

// Row kernels: columns c .. c+3 (c < width) of a row of `width` floats, zeros past its end, by the width's kind:
// kFull: a multiple of four; kTail: another width of four and more, the last quad is read so that it ends with the row and
// moved into place; kNarrow: one to three.  No branches: a load under a condition that differs between lanes makes the
// compiler wait for one load before it issues the next.
enum RowMode { kFull = 0, kTail = 1, kNarrow = 2 };
template <int MODE>
__device__ __forceinline__ void ldr(float (&d)[4], const float* row, int c, int width) {
    if constexpr (MODE == kFull) {
        ldv4(d, row + c);
    } else if constexpr (MODE == kTail) {
        const int off = c + 4 <= width ? 0 : c + 4 - width;
        float q[4];
        ldv4(q, row + c - off);
        const bool o2 = (off & 2) != 0, o1 = (off & 1) != 0;
        const float a0 = o2 ? q[2] : q[0], a1 = o2 ? q[3] : q[1], a2 = o2 ? 0.f : q[2], a3 = o2 ? 0.f : q[3];
        d[0] = o1 ? a1 : a0;
        d[1] = o1 ? a2 : a1;
        d[2] = o1 ? a3 : a2;
        d[3] = o1 ? 0.f : a3;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = row[c + e < width ? c + e : width - 1];
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = c + e < width ? d[e] : 0.f;
    }
}
template <int MODE>
__device__ __forceinline__ void str(float* row, int c, int width, const float (&d)[4]) {
    if (MODE == kFull || c + 4 <= width) stv4(row + c, d);
    else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (c + e < width) row[c + e] = d[e];
    }
}

__device__ __forceinline__ double block_sum(double v, double* sm) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) t += sm[w];
    return t;
}

// Sums of NV values over a workgroup of 256 threads, written to out[0..NV) by its first NV threads: one pass through LDS
// for all of them (sm: NV * 4 doubles).
template <int NV>
__device__ __forceinline__ void block_sums_to(const double (&v)[NV], double* sm, double* out) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        double t = v[j];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) t += __shfl_down(t, o, 64);
        if ((threadIdx.x & 63) == 0) sm[j * 4 + (threadIdx.x >> 6)] = t;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        const double* s = sm + threadIdx.x * 4;
        out[threadIdx.x] = (s[0] + s[1]) + (s[2] + s[3]);
    }
}

// Judges up to ncand candidates of a search, step, step eta, ...  The change of the objective under candidate j is
// D[j] + c1 / step_j + c2 / step_j^2: the part that is exactly quadratic in 1/step is carried by its two coefficients,
// summed once per search (u->c1, u->c2); D (null: nothing) is what has to be evaluated candidate by candidate.
// slack: the test accepts up to this much above the bound (0 for the tau and theta searches).
__device__ __forceinline__ void decide(Unit* u, const double* D, int ncand, SearchParams sp, int32_t* status,
                                       double slack = 0.0) {
    double step = u->step;
    const double g = u->g, c1 = u->c1, c2 = u->c2;
    int nt = u->ntrials;
    for (int j = 0; j < ncand; ++j) {
        ++nt;
        const double inv = 1.0 / step;
        const double d = (D ? D[j] : 0.0) + inv * (c1 + c2 * inv);
        if (!(d == d) || fabs(d) > 1.7e308) atomicOr(status, 2);
        if (d <= -g / (2.0 * step) + slack) { u->step = step; u->ntrials = nt; u->done = 1; return; }
        if (nt > sp.max_backtrack) {
            u->step = step; u->ntrials = nt; u->done = 1;
            atomicOr(status, 1);
            return;
        }
        step *= (double)sp.eta;
    }
    u->step = step;
    u->ntrials = nt;
}

// First candidate of the next search: the last accepted value, or that divided by eta if the parameters may shrink again.
__device__ __forceinline__ double first_candidate(const Unit* u, SearchParams sp) {
    return sp.relax ? u->step / (double)sp.eta : u->step;
}

// Start of a search, before its first decision.
__device__ __forceinline__ void begin_search(Unit* u, SearchParams sp) {
    u->spec = (u->ntrials == 1) ? 1 : 0;     // last search: first candidate accepted
    u->fresh = (u->ntrials == 0) ? 1 : 0;
    u->ntrials = 0;
    u->keep = u->step;
    u->step = first_candidate(u, sp);
    u->step0 = u->step;
    u->done = 0;
    u->skip = 0;
    u->c1 = 0.0;
    u->c2 = 0.0;
}

// A step below resolution is not taken: the block and its step parameter stay as they were.
__device__ __forceinline__ void floor_test(Unit* u, double g, double bnorm) {
    u->g = g;
    u->bnorm = bnorm;
    const double lim = kStepFloor * u->step;
    if (g <= lim * lim * bnorm) { u->done = 1; u->skip = 1; u->step = u->keep; }
}

// ------------------------------------------------------------------------------------------ phi and G
// hidden layer:  e = relu(t) - z,  phi += e^2 (scaled nu/2 at the end),  G = nu e 1[t>0]
// last layer:    r = z - t,        phi += u r + rho/2 r^2,               G = -(u + rho r)
// apply_dual (last layer only): first take the dual ascent step U += rho (Z_L - T) on the iterate just
// reached, then evaluate phi and G with the new U.
// The flat kernels walk a matrix as one array, four floats per lane and trip; the last quad may be partial.
template <int LAST>
__global__ __launch_bounds__(256) void phi_G_kernel(const float* __restrict__ T, const float* __restrict__ Z,
                                                    float* __restrict__ U, float* __restrict__ G,
                                                    float* __restrict__ Tprev, int have_prev, int apply_dual,
                                                    int64_t count, float nu, float rho,
                                                    double* __restrict__ partials) {
    __shared__ double sm[3 * 4];
    double s[3] = {0.0, 0.0, 0.0};          // phi, ||Z - T||^2, ||T - Tprev||^2
    for_quads(count, [&](int64_t i, auto w) {
        const int64_t nv = count - i;
        float t[4], z[4], g[4];
        ldq(t, T + i, nv, w);
        ldq(z, Z + i, nv, w);
        if (LAST) {
            float u[4], tp[4] = {0.f, 0.f, 0.f, 0.f};
            ldq(u, U + i, nv, w);
            if (have_prev) ldq(tp, Tprev + i, nv, w);
            if (apply_dual) {
#pragma unroll
                for (int v = 0; v < 4; ++v) u[v] = u[v] + rho * (z[v] - t[v]);
                stq(U + i, u, nv, w);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double r = (double)z[v] - (double)t[v];
                s[0] += (double)u[v] * r + 0.5 * (double)rho * r * r;
                s[1] += r * r;
                g[v] = -(u[v] + rho * (z[v] - t[v]));
                if (have_prev) { const double d = (double)t[v] - (double)tp[v]; s[2] += d * d; }
            }
            stq(Tprev + i, t, nv, w);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double e = (double)fmaxf(t[v], 0.f) - (double)z[v];
                s[0] += e * e;
                g[v] = (t[v] > 0.f) ? nu * (float)e : 0.f;
            }
        }
        if (G) stq(G + i, g, nv, w);
    });
    block_sums_to<3>(s, sm, partials + (int64_t)blockIdx.x * 3);
}

__global__ __launch_bounds__(256) void phi_G_finish_kernel(const double* __restrict__ partials, int nblocks, int last,
                                                           float nu, LayerScalars* out) {
    __shared__ double sm[4];
    double a = 0.0, b = 0.0, c = 0.0;
    for (int i = threadIdx.x; i < nblocks; i += blockDim.x) {
        a += partials[i * 3 + 0];
        b += partials[i * 3 + 1];
        c += partials[i * 3 + 2];
    }
    a = block_sum(a, sm);
    b = block_sum(b, sm);
    c = block_sum(c, sm);
    if (threadIdx.x == 0) {
        out->phi = last ? a : 0.5 * (double)nu * a;
        out->res2 = b;
        out->dT2 = c;
    }
}

// G without the sums; last layer: the dual step first if asked for (apply_dual).
template <int LAST>
__global__ __launch_bounds__(256) void G_only_kernel(const float* __restrict__ T, const float* __restrict__ Z,
                                                     float* __restrict__ U, float* __restrict__ G, int apply_dual,
                                                     int64_t count, float nu, float rho) {
    for_quads(count, [&](int64_t i, auto w) {
        const int64_t nv = count - i;
        float t[4], z[4], g[4];
        ldq(t, T + i, nv, w);
        ldq(z, Z + i, nv, w);
        if (LAST) {
            float u[4];
            ldq(u, U + i, nv, w);
            if (apply_dual) {
#pragma unroll
                for (int v = 0; v < 4; ++v) u[v] = u[v] + rho * (z[v] - t[v]);
                stq(U + i, u, nv, w);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) g[v] = -(u[v] + rho * (z[v] - t[v]));
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) g[v] = (t[v] > 0.f) ? nu * (float)((double)t[v] - (double)z[v]) : 0.f;
        }
        stq(G + i, g, nv, w);
    });
}

// ------------------------------------------------------------------------------------------ risk
__global__ __launch_bounds__(256) void risk_kernel(const float* __restrict__ ZL, const int32_t* __restrict__ labels,
                                                   int64_t N, int CL, int risk, double* __restrict__ partials) {
    __shared__ double sm[4];
    double s = 0.0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
        const int y = labels[i];
        if (y < 0) continue;
        const float* z = ZL + i * CL;
        if (risk == 0) {
            double mx = (double)z[0];
            for (int c = 1; c < CL; ++c) mx = fmax(mx, (double)z[c]);
            double se = 0.0;
            for (int c = 0; c < CL; ++c) se += exp((double)z[c] - mx);
            s += mx + log(se) - (double)z[y];
        } else {
            for (int c = 0; c < CL; ++c) {
                const double d = (double)z[c] - (c == y ? 1.0 : 0.0);
                s += 0.5 * d * d;
            }
        }
    }
    s = block_sum(s, sm);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ __launch_bounds__(256) void risk_finish_kernel(const double* __restrict__ partials, int nblocks,
                                                          LayerScalars* out) {
    __shared__ double sm[4];
    double a = 0.0;
    for (int i = threadIdx.x; i < nblocks; i += blockDim.x) a += partials[i];
    a = block_sum(a, sm);
    if (threadIdx.x == 0) out->risk = a;
}

// ------------------------------------------------------------------------------------------ W search
// Adds the block sums of ||gradW||^2 and ||W||^2 (left by the reduction of the W-gradient product) in order and starts
// the search.
template <bool GATED>
__global__ __launch_bounds__(256) void w_begin_kernel(const double* __restrict__ partials, int nblocks, Unit* unit,
                                                      SearchParams sp, const int32_t* __restrict__ gate) {
    __shared__ double sm[4];
    if constexpr (GATED) {
        if (*gate == 0) return;
    }
    double g = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < nblocks; i += 256) { g += partials[2 * i]; b += partials[2 * i + 1]; }
    g = block_sum(g, sm);
    b = block_sum(b, sm);
    if (threadIdx.x == 0) {
        begin_search(unit, sp);
        floor_test(unit, g, b);
    }
}

// See launch_rest_w, launch_rest_z; thread l - 1 takes layer l (at most 64 of them).
__global__ __launch_bounds__(64) void rest_w_kernel(int L, const Unit* __restrict__ unitsW, const int32_t* __restrict__ moved,
                                                    int32_t* __restrict__ left_g, int32_t* __restrict__ run_w, int32_t* __restrict__ run_z) {
    const int l = (int)threadIdx.x + 1;
    if (l > L) return;
    const bool here = l == L || moved[l] != 0, before = l > 1 && moved[l - 1] != 0, after = l + 1 >= L || moved[l + 1] != 0;
    // G_l is not there yet, and layer l - 1 may form its gradient
    const bool wanted = l > 1 && !left_g[l] && ((l > 2 && moved[l - 2] != 0) || !unitsW[l - 2].skip);
    const bool run = here || before || !unitsW[l - 1].skip || wanted;
    run_w[l] = run;
    if (run) left_g[l] = 1;
    run_z[l] = here || before || after;
}
__global__ __launch_bounds__(256) void rest_start_kernel(int L, int M, Unit* __restrict__ unitsW, Unit* __restrict__ unitsZ,
                                                         int32_t* __restrict__ moved, uint64_t ungated, int32_t* __restrict__ left_g,
                                                         const int32_t* __restrict__ bad) {
    const int rest = *bad == 0;
    for (int i = threadIdx.x; i < L - 1; i += 256) {
        moved[i + 1] = !rest || (ungated >> (i + 1) & 1) != 0;
        left_g[i + 1] = 0;
        unitsW[i].done = unitsW[i].skip = rest;
    }
    for (int i = threadIdx.x; i < (L - 1) * M; i += 256) unitsZ[i].done = unitsZ[i].skip = rest;
}
__global__ __launch_bounds__(64) void rest_z_kernel(int L, const Unit* __restrict__ unitsW, int32_t* __restrict__ run_z) {
    const int l = (int)threadIdx.x + 1;
    if (l < L && (!unitsW[l - 1].skip || !unitsW[l].skip)) run_z[l] = 1;
}

// Last layer: under T -> T - Q/tau the penalty <U, Z - T> + rho/2 ||Z - T||^2 changes by
// S1/tau + rho/2 S2/tau^2 with S1 = sum q (u + rho (z - t)), S2 = sum q^2, whatever tau is: one pass over memory decides
// the whole search.
__global__ __launch_bounds__(256) void w_last_sums_kernel(const float* __restrict__ T0, const float* __restrict__ Q,
                                                          const float* __restrict__ Z, const float* __restrict__ U,
                                                          int64_t count, float rho, const Unit* unit,
                                                          double* __restrict__ partials) {
    __shared__ double sm[2 * 4];
    if (unit->done) return;
    double s[2] = {0.0, 0.0};
    for_quads(count, [&](int64_t i, auto w) {
        const int64_t nv = count - i;
        float t[4], q[4], z[4], u[4];
        ldq(t, T0 + i, nv, w);
        ldq(q, Q + i, nv, w);
        ldq(z, Z + i, nv, w);
        ldq(u, U + i, nv, w);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double qd = (double)q[v];
            s[0] += qd * ((double)u[v] + (double)rho * ((double)z[v] - (double)t[v]));
            s[1] += qd * qd;
        }
    });
    block_sums_to<2>(s, sm, partials + (int64_t)blockIdx.x * 2);
}

__global__ __launch_bounds__(256) void w_last_finish_kernel(const double* __restrict__ partials, int nblocks,
                                                            SearchParams sp, Unit* unit, int32_t* status) {
    __shared__ double sm[4];
    if (unit->done) return;
    double a = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < nblocks; i += 256) { a += partials[2 * i]; b += partials[2 * i + 1]; }
    a = block_sum(a, sm);
    b = block_sum(b, sm);
    if (threadIdx.x == 0) {
        unit->c1 = a;
        unit->c2 = 0.5 * (double)sp.rho * b;
        decide(unit, nullptr, sp.max_backtrack + 1, sp, status);
    }
}

// Hidden layer: the ReLU makes the change of phi_l piecewise quadratic, so the candidates are evaluated one by one,
// NC at a time and `rounds` times NC per launch (partials: NC * rounds per block).
template <int NC>
__global__ __launch_bounds__(256) void w_trial_kernel(const float* __restrict__ T0, const float* __restrict__ Q,
                                                      const float* __restrict__ Z, int64_t count, SearchParams sp,
                                                      int rounds, const Unit* unit, double* __restrict__ partials,
                                                      int speculated, int leave_fresh) {
    __shared__ double sm[NC * 4];
    if (unit->done || (leave_fresh && unit->fresh)) return;
    const double spec_inv = (speculated && unit->spec) ? 1.0 / unit->step0 : 0.0;      // T0 holds T0 - Q/step0: undo
    double step = unit->step;
    for (int j = 0; j < (int)blockIdx.y * NC; ++j) step *= (double)sp.eta;
    for (int r = blockIdx.y; r < rounds; r += gridDim.y) {          // (side by side or one after the other: launch_w_trial)
        double inv[NC], D[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) { inv[j] = 1.0 / step; step *= (double)sp.eta; D[j] = 0.0; }
        for_quads(count, [&](int64_t i, auto w) {
            const int64_t nv = count - i;
            float t0v[4], qv[4], zv[4];
            ldq(t0v, T0 + i, nv, w);
            ldq(qv, Q + i, nv, w);
            ldq(zv, Z + i, nv, w);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double q = (double)qv[v], z = (double)zv[v];
                const double t0 = (double)t0v[v] + q * spec_inv;
                const double r0 = fmax(t0, 0.0), e2 = 2.0 * (r0 - z);
#pragma unroll
                for (int j = 0; j < NC; ++j) {           // (e1 - e0) (e1 + e0) with e = relu(t) - z
                    const double d = fmax(t0 - q * inv[j], 0.0) - r0;
                    D[j] += d * (d + e2);
                }
            }
        });
        const double hnu = 0.5 * (double)sp.nu;
#pragma unroll
        for (int j = 0; j < NC; ++j) D[j] *= hnu;
        block_sums_to<NC>(D, sm, partials + ((int64_t)blockIdx.x * rounds + r) * NC);
        for (int j = 0; j < ((int)gridDim.y - 1) * NC; ++j) step *= (double)sp.eta;
    }
}

// D[q] = sum of partials[i * stride + q] over the blocks i0 <= i < i1 for q < count, by 256 threads (the caller synchronises).  A
// wavefront takes four values at a time, their loads in flight together (five iterations on 2000 nodes: 46 us in these kernels
// with one value at a time, 37 so).
__device__ __forceinline__ void sum_candidates(const double* __restrict__ partials, int i0, int i1, int stride, int count, double* D) {
    const int lane = threadIdx.x & 63;
    for (int q0 = (threadIdx.x >> 6) * 4; q0 < count; q0 += 16) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
        for (int i = i0 + lane; i < i1; i += 64)
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += partials[(int64_t)i * stride + (q0 + e < count ? q0 + e : q0)];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) s[e] += __shfl_down(s[e], o, 64);
            if (lane == 0 && q0 + e < count) D[q0 + e] = s[e];
        }
    }
}

// Sums the ncand block results (stride per block) of a pass and takes the decision.
__global__ __launch_bounds__(256) void w_trial_finish_kernel(const double* __restrict__ partials, int nblocks, int ncand,
                                                             SearchParams sp, Unit* unit, int32_t* status, int leave_fresh) {
    __shared__ double sm[4];
    __shared__ double D[kRestCand];
    if (unit->done || (leave_fresh && unit->fresh)) return;
    if (ncand == 1) {                                  // many blocks (a product's workgroups), one candidate
        double a = 0.0, b = 0.0, c = 0.0, d = 0.0;     // four independent loads in flight per thread
        int i = threadIdx.x;
        for (; i + 768 < nblocks; i += 1024) {
            a += partials[i];
            b += partials[i + 256];
            c += partials[i + 512];
            d += partials[i + 768];
        }
        for (; i < nblocks; i += 256) a += partials[i];
        a = block_sum((a + b) + (c + d), sm);
        if (threadIdx.x == 0) D[0] = a;
    } else {
        sum_candidates(partials, 0, nblocks, ncand, ncand, D);
    }
    __syncthreads();
    if (threadIdx.x == 0) decide(unit, D, ncand, sp, status);
}

// W <- W - gradW/tau with its transpose beside it, T <- T - Q/tau.  LAST: also keeps the old T (Tprev).  The gradient
// of the new T is left for the Z step of the layer before (G may be the same array as Q): LAST G = -(U + rho (Z - T)), else,
// if there is a G, nu (relu(T) - Z) 1[T > 0].
template <int LAST>
__global__ __launch_bounds__(256) void w_step_kernel(float* __restrict__ W, float* __restrict__ Wt,
                                                     const float* __restrict__ gradW, int K, int C,
                                                     float* __restrict__ T, const float* Q, int64_t count_t,
                                                     const Unit* unit, int speculated, const float* __restrict__ Z,
                                                     const float* __restrict__ U, float* G, float* __restrict__ Tprev,
                                                     float nu, float rho) {
    const bool skip = unit->skip != 0;
    const bool leave = LAST || G != nullptr;
    if (skip && (!leave || speculated)) return;
    const double inv = 1.0 / unit->step;
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
    // T already holds T0 - Q/step0 when the step was taken speculatively: nothing to do if step0 was accepted,
    // otherwise T0 - Q/step = T + Q (1/step0 - 1/step)
    const bool spec = speculated && unit->spec;
    const double tinv = spec ? inv - 1.0 / unit->step0 : inv;
    const bool t_done = spec && !skip && unit->step == unit->step0;
    if (LAST || !t_done) {
        for_quads(count_t, [&](int64_t i, auto w) {
            const int64_t nv = count_t - i;
            float t[4], q[4];
            ldq(t, T + i, nv, w);
            if (!skip) ldq(q, Q + i, nv, w);
            float z[4], u[4], g[4];
            if (leave) ldq(z, Z + i, nv, w);
            if (LAST) {
                ldq(u, U + i, nv, w);
                if (Tprev) stq(Tprev + i, t, nv, w);
            }
            if (!skip) {
#pragma unroll
                for (int v = 0; v < 4; ++v) t[v] = (float)((double)t[v] - (double)q[v] * tinv);
                stq(T + i, t, nv, w);
            }
            if (leave) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if (LAST) g[v] = -(u[v] + rho * (z[v] - t[v]));
                    else g[v] = t[v] > 0.f ? nu * (float)((double)t[v] - (double)z[v]) : 0.f;
                }
                stq(G + i, g, nv, w);
            }
        });
    }
    if (skip) return;
    const int64_t count_w = (int64_t)K * C;
    for (int64_t i = gtid; i < count_w; i += nthreads) {
        const float w = (float)((double)W[i] - (double)gradW[i] * inv);
        W[i] = w;
        if (Wt) {
            const int k = (int)(i / C), cc = (int)(i - (int64_t)k * C);
            Wt[(int64_t)cc * K + k] = w;
        }
    }
}

// ------------------------------------------------------------------------------------------ Z search
// How a workgroup walks rows of `width` floats: 2^shift lanes per row, four columns per lane and trip.
struct RowWalk {
    int wv, shift, c_first, r_first, r_step;
    __device__ __forceinline__ explicit RowWalk(int width) {
        wv = (width + 3) >> 2;
        shift = 0;
        while ((1 << shift) < wv && shift < 8) ++shift;
        c_first = threadIdx.x & ((1 << shift) - 1);
        r_first = threadIdx.x >> shift;
        r_step = 256 >> shift;
    }
};

// First pass of the search for theta_{l,m}, all communities of layer l at once, one workgroup per chunk (a chunk belongs
// to one community).  What is summed decides every candidate of what is quadratic in 1/theta:
//   rows (kind 0): nu/2 ||Z - relu(T_l)||^2 under Z -> Z - g/theta changes by nu/2 (-2 A/theta + B/theta^2) with
//     A = sum e g, e = Z - relu(T_l), and B = ||g||^2; ||Z||^2 for the step floor.
//   segments (kind 1), next layer the last one: <U, Z_L - T> + rho/2 ||Z_L - T||^2 under T -> T - P/theta changes by
//     -S1/theta + rho/2 S2/theta^2 with S1 = sum p G_L (G_L = -(u + rho (z - t)) is at hand) and S2 = sum p^2.
//   segments, next layer hidden (HID): its ReLU makes the term piecewise quadratic; the first candidate is evaluated.
//     Where the previous search did not accept its first candidate this one will hardly either (a layer's first search takes
//     three or four): the first four are evaluated then, for a tenth more than for one and in place of a second pass
//     (500000 rows, 512 columns: 1.32 ms for one, 1.49 for four).
// So with a last next layer this one pass over memory is the whole search, and with a hidden one the later passes read
// the segments alone.  Per chunk: A, B, ||Z||^2, S1 or the candidates' changes, S2.  Bound by HBM traffic.
// SM: kind of the width Cn.
// With a gate the search comes in two parts, the rows (launch_z_floor) and, where any community takes a step, the segments:
// for the rows alone two more launches, for the segments nothing that nobody needs.  PART says which chunks a launch takes.
// PART and GATED (here and below) are template parameters since a branch at a kernel's start, taken or not, keeps the other
// arguments from being loaded beside what it looks at: with them and gemm_nn_narrow_kernel's the iterations of a small run that has no
// gate take 191.0 us, without them 192.1 (20000 nodes, 500-128-3).
constexpr int kFirstCand = 4;
template <int HID> constexpr int kFirstValues = HID ? 3 + kFirstCand : 5;
enum FirstPart { kBoth = 0, kRowsOnly = 1, kSegmentsOnly = 2 };
template <int RM, int V>
__device__ __forceinline__ void z_first_rows(const ZTrialArgs& a, int begin, int end, double (&s)[V]) {
    const RowWalk w(a.Cl);
    for (int r = begin + w.r_first; r < end; r += w.r_step) {
        const int64_t base = (int64_t)r * a.Cl;
        for (int cv = w.c_first; cv < w.wv; cv += 1 << w.shift) {
            float zv[4], gv[4], tv[4];
            ldr<RM>(zv, a.Zl + base, 4 * cv, a.Cl);
            ldr<RM>(tv, a.Tl + base, 4 * cv, a.Cl);
            ldr<RM>(gv, a.gradZ + base, 4 * cv, a.Cl);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const double z = (double)zv[v], gz = (double)gv[v];
                s[0] += (z - fmax((double)tv[v], 0.0)) * gz;
                s[1] += gz * gz;
                s[2] += z * z;
            }
        }
    }
}

template <int HID, int SM, int PART>
__global__ __launch_bounds__(256) void z_first_kernel(ZTrialArgs a) {
    constexpr int kFirstVals = kFirstValues<HID>;
    __shared__ double sm[kFirstVals * 4];
    if (PART == kRowsOnly && a.run && *a.run == 0) return;
    if (PART == kRowsOnly && blockIdx.x == 0 && threadIdx.x == 0) *a.gate = 0;
    if (PART == kSegmentsOnly && *a.gate == 0) return;
    const int4 ck = a.chunks[blockIdx.x];               // community, kind, first row / segment, one past the last
    if ((PART == kRowsOnly && ck.y != 0) || (PART == kSegmentsOnly && ck.y == 0)) return;
    double s[kFirstVals] = {};
    if (ck.y == 0) {
        if (a.row_sums) {                               // the kernel that formed the gradient left the rows' sums
            const int64_t n = 3 * (int64_t)(ck.w - ck.z);
            for (int t = 0; t < a.sum_tiles; ++t) {
                const double* const p = a.row_sums + 3 * ((int64_t)t * a.N + ck.z);
                for (int64_t i = 3 * (int64_t)threadIdx.x; i < n; i += 3 * 256) { s[0] += p[i]; s[1] += p[i + 1]; s[2] += p[i + 2]; }
            }
        } else if (a.Cl % 4 == 0) z_first_rows<kFull>(a, ck.z, ck.w, s);
        else if (a.Cl >= 4) z_first_rows<kTail>(a, ck.z, ck.w, s);
        else z_first_rows<kNarrow>(a, ck.z, ck.w, s);
    } else {
        const RowWalk w(a.Cn);
        const Unit* const u = a.units + ck.x;           // (launch_z_floor has started the search, or the finishing kernel will)
        if (PART == kSegmentsOnly && u->done) return;
        // (f: what a quad of a segment's row adds)
        auto walk = [&](auto f) {
            for (int q = ck.z + w.r_first; q < ck.w; q += w.r_step) {
                const int64_t base = (int64_t)a.segc_row[q] * a.Cn, pbase = (int64_t)q * a.Cn;
                for (int cv = w.c_first; cv < w.wv; cv += 1 << w.shift) {
                    float pv[4], tv[4], zv[4];
                    ldr<SM>(pv, a.P + pbase, 4 * cv, a.Cn);
                    if constexpr (HID) {
                        ldr<SM>(tv, a.Tn + base, 4 * cv, a.Cn);
                        ldr<SM>(zv, a.Zn + base, 4 * cv, a.Cn);
                    } else {
                        ldr<SM>(tv, a.Gn + base, 4 * cv, a.Cn);
                    }
                    f(pv, tv, zv);
                }
            }
        };
        if constexpr (HID) {
            // (r0 = relu(t), d its change: (e1 - e0) (e1 + e0) = d (d + 2 e0) with e = relu(t) - z)
            auto candidates = [&](auto NC) {
                constexpr int kC = decltype(NC)::value;
                double inv[kC], step = PART == kSegmentsOnly ? u->step0 : first_candidate(u, a.sp);
#pragma unroll
                for (int j = 0; j < kC; ++j) { inv[j] = 1.0 / step; step *= (double)a.sp.eta; }
                walk([&](const float (&pv)[4], const float (&tv)[4], const float (&zv)[4]) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const double t = (double)tv[v], p = (double)pv[v], r0 = fmax(t, 0.0), e2 = 2.0 * (r0 - (double)zv[v]);
#pragma unroll
                        for (int j = 0; j < kC; ++j) {
                            const double d = fmax(t - p * inv[j], 0.0) - r0;
                            s[3 + j] += d * (d + e2);
                        }
                    }
                });
            };
            if (PART == kSegmentsOnly ? u->spec : u->ntrials == 1) candidates(std::integral_constant<int, 1>{});
            else candidates(std::integral_constant<int, kFirstCand>{});
        } else {
            walk([&](const float (&pv)[4], const float (&tv)[4], const float (&)[4]) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    s[3] += (double)pv[v] * (double)tv[v];
                    s[4] += (double)pv[v] * (double)pv[v];
                }
            });
        }
    }
    block_sums_to<kFirstVals>(s, sm, a.partials + (int64_t)blockIdx.x * kFirstVals);
}

// One workgroup per community: adds its chunks' sums in order, applies the step floor and takes the decision (all of
// them if the whole change is quadratic).
template <int HID, int PART>
__global__ __launch_bounds__(256) void z_first_finish_kernel(ZTrialArgs a) {
    constexpr int kFirstVals = kFirstValues<HID>;
    __shared__ double sm[kFirstVals * 4];
    __shared__ double S[kFirstVals];
    const int unit = blockIdx.x;
    Unit* u = a.units + unit;
    if (PART == kRowsOnly && a.run && *a.run == 0) return;
    if (PART == kSegmentsOnly && u->done) return;
    if (PART == kBoth && a.moved && unit == 0 && threadIdx.x == 0) *a.moved = 1;
    const int c0 = a.unit_chunk_ptr[unit], c1 = a.unit_chunk_ptr[unit + 1];
    double s[kFirstVals] = {};
    for (int i = c0 + threadIdx.x; i < c1; i += 256) {
        if (PART != kBoth && (a.chunks[i].y == 0) != (PART == kRowsOnly)) continue;
#pragma unroll
        for (int q = 0; q < kFirstVals; ++q) s[q] += a.partials[(int64_t)i * kFirstVals + q];
    }
    block_sums_to<kFirstVals>(s, sm, S);
    __syncthreads();
    if (threadIdx.x == 0) {
        const double hnu = 0.5 * (double)a.sp.nu;
        if (PART != kSegmentsOnly) {
            begin_search(u, a.sp);
            floor_test(u, S[1], S[2]);
            if (u->done) return;
            u->c1 = -2.0 * hnu * S[0];
            u->c2 = hnu * S[1];
        }
        if (PART == kRowsOnly) {
            atomicOr(a.gate, 1);
        } else if (HID) {
            double D[kFirstCand];
            for (int j = 0; j < kFirstCand; ++j) D[j] = hnu * S[3 + j];
            decide(u, D, u->spec ? 1 : kFirstCand, a.sp, a.status);
        } else {
            u->c1 -= S[3];
            u->c2 += 0.5 * (double)a.sp.rho * S[4];
            decide(u, nullptr, a.sp.max_backtrack + 1, a.sp, a.status);
        }
    }
}

// Later passes over the segments (hidden next layer): `rounds` times NC further candidates for the communities still
// searching.  Usually every community is done: a workgroup looks at all the flags at once and leaves if nothing is pending.
template <int NC, int SM>
__global__ __launch_bounds__(256) void z_more_kernel(ZTrialArgs a, int rounds) {
    __shared__ double sm[NC * 4];
    int pending = 0;
    for (int i = threadIdx.x; i < a.M; i += 256) pending |= (a.units[i].done == 0);
    if (!__syncthreads_or(pending)) return;
    const RowWalk w(a.Cn);
    const double hnu = 0.5 * (double)a.sp.nu;
    for (int ch = blockIdx.x; ch < a.n_chunks; ch += gridDim.x) {
        const int4 ck = a.chunks[ch];
        if (ck.y == 0) continue;
        const Unit* u = a.units + ck.x;
        if (u->done) continue;
        double step = u->step;
        for (int rd = 0; rd < rounds; ++rd) {
            double inv[NC], D[NC];
#pragma unroll
            for (int j = 0; j < NC; ++j) { inv[j] = 1.0 / step; step *= (double)a.sp.eta; D[j] = 0.0; }
            for (int q = ck.z + w.r_first; q < ck.w; q += w.r_step) {
                const int64_t base = (int64_t)a.segc_row[q] * a.Cn, pbase = (int64_t)q * a.Cn;
                for (int cv = w.c_first; cv < w.wv; cv += 1 << w.shift) {
                    float pv[4], tv[4], zv[4];
                    ldr<SM>(pv, a.P + pbase, 4 * cv, a.Cn);
                    ldr<SM>(tv, a.Tn + base, 4 * cv, a.Cn);
                    ldr<SM>(zv, a.Zn + base, 4 * cv, a.Cn);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const double t = (double)tv[v], p = (double)pv[v], r0 = fmax(t, 0.0), e2 = 2.0 * (r0 - (double)zv[v]);
#pragma unroll
                        for (int j = 0; j < NC; ++j) {
                            const double d = fmax(t - p * inv[j], 0.0) - r0;
                            D[j] += d * (d + e2);
                        }
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < NC; ++j) D[j] *= hnu;
            block_sums_to<NC>(D, sm, a.partials + ((int64_t)ch * rounds + rd) * NC);
        }
    }
}

__global__ __launch_bounds__(256) void z_more_finish_kernel(ZTrialArgs a, int ncand) {
    __shared__ double D[kRestCand];
    const int unit = blockIdx.x;
    Unit* u = a.units + unit;
    if (u->done) return;
    const int c0 = a.unit_chunk_ptr[unit], c1 = a.unit_chunk_ptr[unit + 1];
    const int lane = threadIdx.x & 63;
    for (int j = threadIdx.x >> 6; j < ncand; j += 4) {
        double s = 0.0;
        for (int i = c0 + lane; i < c1; i += 64)
            if (a.chunks[i].y != 0) s += a.partials[(int64_t)i * ncand + j];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
        if (lane == 0) D[j] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) decide(u, D, ncand, a.sp, a.status);
}

// 1/theta of every community in LDS (0 where no step is taken): kernels that need the step parameter of a row's or a
// segment's community then do not wait for it in a chain of dependent loads (row -> community -> unit).
constexpr int kStepUnits = 1024;
__device__ __forceinline__ double unit_inv(const Unit* u) { return u->skip ? 0.0 : 1.0 / u->step; }
template <bool LDSU>
__device__ __forceinline__ void load_inv(double* s_inv, const Unit* __restrict__ units, int M) {
    if constexpr (LDSU) {
        for (int i = threadIdx.x; i < M; i += 256) s_inv[i] = unit_inv(units + i);
        __syncthreads();
    }
}

// Z_{l,m} <- Z_{l,m} - grad / theta_{l,m}; the loads of a row are issued before its community is known.
template <bool LDSU, int RM, bool GATED>
__global__ __launch_bounds__(256) void z_step_kernel(float* __restrict__ Zl, const float* __restrict__ gradZ,
                                                     const int32_t* __restrict__ row_comm, int64_t N, int Cl,
                                                     const Unit* __restrict__ units, int M, const int32_t* __restrict__ gate) {
    __shared__ double s_inv[LDSU ? kStepUnits : 1];
    if constexpr (GATED) {
        if (*gate == 0) return;
    }
    load_inv<LDSU>(s_inv, units, M);
    const RowWalk w(Cl);
    const int64_t r_step = (int64_t)gridDim.x * w.r_step;
    for (int64_t r = (int64_t)blockIdx.x * w.r_step + w.r_first; r < N; r += r_step) {
        const int cm = row_comm[r];
        const int64_t base = r * Cl;
        for (int cv = w.c_first; cv < w.wv; cv += 1 << w.shift) {
            float z[4], g[4];
            ldr<RM>(z, Zl + base, 4 * cv, Cl);
            ldr<RM>(g, gradZ + base, 4 * cv, Cl);
            const double inv = LDSU ? s_inv[cm] : unit_inv(units + cm);
            if (inv == 0.0) break;                   // no step for this row's community
#pragma unroll
            for (int v = 0; v < 4; ++v) z[v] = (float)((double)z[v] - (double)g[v] * inv);
            str<RM>(Zl + base, 4 * cv, Cl, z);
        }
    }
}

// The same step with the gradient rebuilt from its low-rank form, nu (z - relu(t)) + sum_k sg[k] wt[k] with the operations in
// the order in which gemm_nn_gradz_kernel formed it for the search; a lane group handles two rows per trip with every load issued before the first use.  The rows of W_{l+1}^T
// live in LDS, not in 64 registers per lane: the kernel is a plain in-place update of Z_l and needs the wavefronts in
// flight that a small register footprint allows (5 TB/s against 4.4 with the rows in registers).
// SM: kind of the width Cn.
template <bool LDSU, int SM, bool GATED>
__global__ __launch_bounds__(256) void z_step_lowrank_kernel(float* __restrict__ Zl, const float* __restrict__ Tl,
                                                             const float* __restrict__ SG, const float* __restrict__ Wt,
                                                             float nu, const int32_t* __restrict__ row_comm, int64_t N,
                                                             int Cl, int Cn, const Unit* __restrict__ units, int M,
                                                             const int32_t* __restrict__ gate) {
    __shared__ double s_inv[LDSU ? kStepUnits : 1];
    extern __shared__ __align__(16) float s_wt[];        // [Cn][Cl]
    if constexpr (GATED) {
        if (*gate == 0) return;
    }
    if constexpr (LDSU) {
        for (int i = threadIdx.x; i < M; i += 256) s_inv[i] = unit_inv(units + i);
    }
    for (int i = threadIdx.x; i < Cn * Cl; i += 256) s_wt[i] = Wt[i];
    __syncthreads();
    const int wv = Cl / 4;
    int cshift = 0;
    while ((1 << cshift) < wv && cshift < 8) ++cshift;
    const int c_first = threadIdx.x & ((1 << cshift) - 1);
    if (c_first >= wv) return;                       // (after the barrier)
    const float4* const wcol = reinterpret_cast<const float4*>(s_wt) + c_first;      // row k: wcol[k * wv]
    constexpr int R = 2;
    const int64_t rows_per_block = 256 >> cshift;
    const int64_t r_step = (int64_t)gridDim.x * rows_per_block * R;
    for (int64_t r0 = ((int64_t)blockIdx.x * R) * rows_per_block + (threadIdx.x >> cshift); r0 < N; r0 += r_step) {
        int cm[R];
        float z[R][4], t[R][4], sg[R][kLowRankMax];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int64_t r = r0 + q * rows_per_block;
            const int64_t rr = r < N ? r : N - 1;    // a row past the end repeats the last one and is not stored
            cm[q] = row_comm[rr];
            const int64_t o = rr * Cl + c_first * 4;
            ldv4(z[q], Zl + o);
            ldv4(t[q], Tl + o);
#pragma unroll
            for (int k4 = 0; k4 < kLowRankMax / 4; ++k4) {
                float v[4] = {0.f, 0.f, 0.f, 0.f};
                if (4 * k4 < Cn) ldr<SM>(v, SG + rr * Cn, 4 * k4, Cn);
                sg[q][4 * k4] = v[0]; sg[q][4 * k4 + 1] = v[1]; sg[q][4 * k4 + 2] = v[2]; sg[q][4 * k4 + 3] = v[3];
            }
        }
        float g[R][4];
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) g[q][v] = nu * (z[q][v] - fmaxf(t[q][v], 0.f));
#pragma unroll
        for (int k = 0; k < kLowRankMax; ++k) {
            if (k < Cn) {
                const float4 w4 = wcol[k * wv];
                const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
                for (int q = 0; q < R; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) g[q][v] = fmaf(sg[q][k], w[v], g[q][v]);
            }
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int64_t r = r0 + q * rows_per_block;
            double inv;
            if constexpr (LDSU) inv = s_inv[cm[q]];
            else inv = unit_inv(units + cm[q]);
            if (r >= N || inv == 0.0) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) z[q][v] = (float)((double)z[q][v] - (double)g[q][v] * inv);
            stv4(Zl + r * Cl + c_first * 4, z[q]);
        }
    }
}

// After Z_{l,m} <- Z_{l,m} - grad/theta_{l,m} the next layer's pre-activation A~ Z_l W_{l+1} of row i changes by
// - sum over the segments (i, c) of P_{(i,c)} / theta_{l,c}  (P = A~_{., c} grad W_{l+1}, already formed for the
// search).  Applying that keeps T_{l+1} valid for the next iteration without a new aggregation and product.
constexpr int kCarryBatch = 4;
// acc += that sum for columns 4 cv .. of row r; returns whether any of the row's communities took a step.
// kCarryBatch segments at a time: their index, unit and row loads do not depend on each other, so they are in flight
// together; the sums are still taken in segment order.  s_inv: 1/theta of the communities in LDS, or null if there are too many.
template <int SM>
__device__ __forceinline__ bool carry_sum(double (&acc)[4], const CarryArgs& k, const double* s_inv, int64_t r, int Cn,
                                          int cv) {
    const int64_t s0 = k.row_seg_ptr[r], s1 = k.row_seg_ptr[r + 1];
    bool any = false;
    for (int64_t sgm = s0; sgm < s1; sgm += kCarryBatch) {
        int cm[kCarryBatch], ps[kCarryBatch];
#pragma unroll
        for (int j = 0; j < kCarryBatch; ++j) {
            const int64_t sj = sgm + j < s1 ? sgm + j : s1 - 1;
            cm[j] = k.seg_comm[sj];
            ps[j] = k.seg_pos[sj];
        }
        double inv[kCarryBatch];
        float p[kCarryBatch][4];
#pragma unroll
        for (int j = 0; j < kCarryBatch; ++j) ldr<SM>(p[j], k.P + (int64_t)ps[j] * Cn, 4 * cv, Cn);
        if (s_inv) {
#pragma unroll
            for (int j = 0; j < kCarryBatch; ++j) inv[j] = s_inv[cm[j]];
        } else {
#pragma unroll
            for (int j = 0; j < kCarryBatch; ++j) inv[j] = unit_inv(k.units + cm[j]);
        }
#pragma unroll
        for (int j = 0; j < kCarryBatch; ++j) {
            if (sgm + j >= s1 || inv[j] == 0.0) continue;          // past the row's end, or a step that was not taken
            any = true;
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] += (double)p[j][v] * inv[j];
        }
    }
    return any;
}
__device__ __forceinline__ const double* carry_inv(double* s_inv, const CarryArgs& k) {
    if (k.M > kStepUnits) return nullptr;
    load_inv<true>(s_inv, k.units, k.M);
    return s_inv;
}

template <int SM, bool GATED>
__global__ __launch_bounds__(256) void t_carry_kernel(float* __restrict__ Tn, CarryArgs k, int64_t N, int Cn) {
    __shared__ double s_buf[kStepUnits];
    if constexpr (GATED) {
        if (*k.gate == 0) return;
    }
    const double* const s_inv = carry_inv(s_buf, k);
    const RowWalk w(Cn);
    const int64_t r_step = (int64_t)gridDim.x * w.r_step;
    for (int64_t r = (int64_t)blockIdx.x * w.r_step + w.r_first; r < N; r += r_step) {
        for (int cv = w.c_first; cv < w.wv; cv += 1 << w.shift) {
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            if (!carry_sum<SM>(acc, k, s_inv, r, Cn, cv)) continue;
            float t[4];
            ldr<SM>(t, Tn + r * Cn, 4 * cv, Cn);
#pragma unroll
            for (int v = 0; v < 4; ++v) t[v] = (float)((double)t[v] - acc[v]);
            str<SM>(Tn + r * Cn, 4 * cv, Cn, t);
        }
    }
}

// ------------------------------------------------------------------------------------------ last layer + dual
// 2^LPLOG lanes share one node row, four classes per lane, so a wavefront reads whole 64-byte-aligned
// pieces of consecutive rows with 16-byte accesses; the row maximum and the softmax denominator are
// formed by xor-shuffles inside the lane group.  FISTA on
//   R(z, y_i) + <u, z - c> + rho/2 ||z - c||^2,   c = row of A~ Z_{L-1}^k W_L^{k+1},
// whose smooth part is the whole objective: x_j = y_j - grad(y_j)/Lip, Lip = rho + (1/2 | 1).
// CARRY: T_L is then brought to the new Z_{L-1} (carry_sum) and, with G, the gradient G_L = -(U + rho (Z_L - T_L)) of the
// next iteration is left, all while the row is in registers: one launch and no second pass over Z_L, U and T_L.
template <int LPLOG, int CARRY, int SM, bool GATED>
__global__ __launch_bounds__(256) void last_layer_kernel(float* __restrict__ ZL, float* __restrict__ U, float* __restrict__ TL,
                                                         const int32_t* __restrict__ labels, int64_t N, int CL,
                                                         int risk, float rho, int J, int update_u, CarryArgs k,
                                                         float* __restrict__ G) {
    __shared__ double s_buf[CARRY ? kStepUnits : 1];
    const double* s_inv = nullptr;
    bool carries = CARRY;
    if constexpr (GATED) carries = *k.gate != 0;
    if constexpr (CARRY) {
        if (carries) s_inv = carry_inv(s_buf, k);
    }
    constexpr int LP = 1 << LPLOG;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t row = t >> LPLOG;
    const int j0 = (int)(t & (LP - 1)) * 4;
    const bool act = row < N;                       // uniform over the lane group of a row
    const int64_t base = (act ? row : 0) * CL;
    const int nv = act ? CL - j0 : 0;               // columns of this lane (none, or one to four)
    bool ok[4];
    float c[4] = {0.f, 0.f, 0.f, 0.f}, u[4] = {0.f, 0.f, 0.f, 0.f}, xp[4] = {0.f, 0.f, 0.f, 0.f}, y[4], x[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) ok[v] = v < nv;
    if (nv > 0) {
        ldr<SM>(c, TL + base, j0, CL);
        ldr<SM>(u, U + base, j0, CL);
        ldr<SM>(xp, ZL + base, j0, CL);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) { y[v] = xp[v]; x[v] = xp[v]; }
    // dual step with the iterates as printed in Eq. 2: Z_L^k and the aggregation with W_L^{k+1}
    float un[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) un[v] = u[v] + rho * (xp[v] - c[v]);
    const int lab = act ? labels[row] : -1;
    if (lab < 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = c[v] - u[v] / rho;       // exact minimiser of the quadratic
    } else {
        const float inv_lip = 1.0f / (rho + (risk == 0 ? 0.5f : 1.0f));
        float tk = 1.0f;
        for (int it = 0; it < J; ++it) {
            float g[4];
            if (risk == 0) {
                float mx = -3.0e38f;
#pragma unroll
                for (int v = 0; v < 4; ++v) mx = ok[v] ? fmaxf(mx, y[v]) : mx;
#pragma unroll
                for (int o = 1; o < LP; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
                float se = 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) { g[v] = ok[v] ? __expf(y[v] - mx) : 0.f; se += g[v]; }
#pragma unroll
                for (int o = 1; o < LP; o <<= 1) se += __shfl_xor(se, o, 64);
                const float inv_se = 1.0f / se;
#pragma unroll
                for (int v = 0; v < 4; ++v) g[v] = g[v] * inv_se - ((j0 + v) == lab ? 1.f : 0.f);
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) g[v] = y[v] - ((j0 + v) == lab ? 1.f : 0.f);
            }
            const float tn = 0.5f * (1.0f + sqrtf(1.0f + 4.0f * tk * tk));
            const float mom = (tk - 1.0f) / tn;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float grad = g[v] + u[v] + rho * (y[v] - c[v]);
                x[v] = y[v] - grad * inv_lip;
                y[v] = x[v] + mom * (x[v] - xp[v]);
                xp[v] = x[v];
            }
            tk = tn;
        }
    }
    if (nv <= 0) return;
    if (update_u) str<SM>(U + base, j0, CL, un);
    str<SM>(ZL + base, j0, CL, x);
    if constexpr (CARRY) {
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        if (carries && carry_sum<SM>(acc, k, s_inv, row, CL, j0 >> 2)) {
#pragma unroll
            for (int v = 0; v < 4; ++v) c[v] = (float)((double)c[v] - acc[v]);
            str<SM>(TL + base, j0, CL, c);
        }
        if (G) {
            float g[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) g[v] = -(un[v] + rho * (x[v] - c[v]));
            str<SM>(G + base, j0, CL, g);
        }
    }
}

// relu (or a plain copy) of a matrix
__global__ __launch_bounds__(256) void relu_kernel(const float* __restrict__ T, float* __restrict__ Z, int64_t count,
                                                   int apply_relu) {
    for_quads(count, [&](int64_t i, auto w) {
        const int64_t nv = count - i;
        float t[4];
        ldq(t, T + i, nv, w);
        if (apply_relu) {
#pragma unroll
            for (int v = 0; v < 4; ++v) t[v] = fmaxf(t[v], 0.f);
        }
        stq(Z + i, t, nv, w);
    });
}

// class of every node, see launch_argmax_rows
__global__ __launch_bounds__(256) void argmax_rows_kernel(const float* __restrict__ T, int32_t* __restrict__ pred,
                                                          const int32_t* __restrict__ perm, const int32_t* __restrict__ labels,
                                                          int32_t* __restrict__ hits, int64_t N, int C) {
    __shared__ int sm[4];
    int hit = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < N; i += (int64_t)kArgmaxBlocks * 256) {
        const float* t = T + i * C;
        int best = 0;
        float bv = t[0];
        for (int c = 1; c < C; ++c)
            if (t[c] > bv) { bv = t[c]; best = c; }
        pred[perm[i]] = best;
        hit += best == labels[i];                       // (no class is -1)
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) hit += __shfl_down(hit, o, 64);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = hit;
    __syncthreads();
    if (threadIdx.x == 0) hits[blockIdx.x] = sm[0] + sm[1] + sm[2] + sm[3];
}

// ------------------------------------------------------------------------------------------ last layer, FISTA with backtracking
// See FistaArgs.  2^LPLOG lanes share a node row, four classes per lane, as in last_layer_kernel; a workgroup takes one
// chunk of rows of one community.  Everything that enters a decision is formed in fp64 from the fp32 state: the
// gradient g of F(z) = R(z, y) + <u, z - c> + rho/2 ||z - c||^2 at y, and for a candidate L the difference
// F(y - g/L) - F(y), term by term (the log-sum-exp of both points, the linear and the quadratic terms through
// x - y = -g/L), so that nothing is lost to the cancellation of two nearly equal values of F.
constexpr int kFistaSums = 3;                     // per chunk behind the candidates' differences: ||g||^2, ||y||^2, F(y)
constexpr double kFistaSlack = 1e-12;             // the test accepts up to this relative rounding of F(y)

// The value of the lane that is 2^S away, for the steps of a butterfly over up to sixteen neighbouring lanes: after the steps
// below S the lanes of a group of 2^S hold the same value, so the mirror image of 8 or 16 lanes serves for 4 and 8.  A lane
// exchange inside a row of sixteen is a modifier of a move; __shfl_xor goes through LDS, a hundred cycles per step of a chain of
// dependent reductions.
template <int S>
__device__ __forceinline__ double across(double v) {
    constexpr int ctrl = S == 0 ? 0xB1 : S == 1 ? 0x4E : S == 2 ? 0x141 : 0x140;      // quad 1 0 3 2, quad 2 3 0 1, half mirror, mirror
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
template <int LPLOG>
__device__ __forceinline__ double group_sum(double v) {
    if constexpr (LPLOG > 0) v += across<0>(v);
    if constexpr (LPLOG > 1) v += across<1>(v);
    if constexpr (LPLOG > 2) v += across<2>(v);
    if constexpr (LPLOG > 3) v += across<3>(v);
    return v;
}
template <int LPLOG>
__device__ __forceinline__ double group_max(double v) {
    if constexpr (LPLOG > 0) v = fmax(v, across<0>(v));
    if constexpr (LPLOG > 1) v = fmax(v, across<1>(v));
    if constexpr (LPLOG > 2) v = fmax(v, across<2>(v));
    if constexpr (LPLOG > 3) v = fmax(v, across<3>(v));
    return v;
}

// log-sum-exp over the row (the lanes of the group hold four entries each; entries past CL are off)
template <int LPLOG>
__device__ __forceinline__ double row_lse(const double (&z)[4], const bool (&ok)[4], double (&e)[4], double& se) {
    double mx = -1.0e300;
#pragma unroll
    for (int v = 0; v < 4; ++v) mx = ok[v] ? fmax(mx, z[v]) : mx;
    mx = group_max<LPLOG>(mx);
    double s = 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) { e[v] = ok[v] ? exp(z[v] - mx) : 0.0; s += e[v]; }
    se = group_sum<LPLOG>(s);
    return mx + log(se);
}

template <int LPLOG, int NC>
__global__ __launch_bounds__(256) void fista_stage_kernel(FistaArgs a, int stage, int more, int rounds, float mom) {
    __shared__ double sm[(NC + kFistaSums) * 4];
    constexpr int LP = 1 << LPLOG;
    if (more) {                                        // a pass of further candidates: only if some search is pending
        int pending = 0;
        for (int i = threadIdx.x; i < a.M; i += 256) pending |= (a.units[i].done == 0);
        if (!__syncthreads_or(pending)) return;
    }
    for (int ch = blockIdx.x; ch < a.n_chunks; ch += gridDim.x) {
        const int4 ck = a.chunks[ch];
        if (ck.y != 0) continue;                       // only the chunks of rows
        const Unit* u = a.units + ck.x;
        if (more && u->done) continue;
        const double Lcur = (stage == 0 && !more) ? (double)a.rho : u->step;       // every solve starts from L = rho
        const bool skipped = stage > 0 && !more && u->skip;
        const int r0 = ck.z, r1 = ck.w;
        double L_round = more ? u->step : Lcur;        // first candidate of this round
        for (int rd = 0; rd < rounds; ++rd) {
        double D[NC], sgg = 0.0, syy = 0.0, sF = 0.0;
#pragma unroll
        for (int q = 0; q < NC; ++q) D[q] = 0.0;
        for (int rb = r0; rb < r1; rb += 256 >> LPLOG) {
            const int row = rb + (threadIdx.x >> LPLOG);
            const int j0 = (threadIdx.x & (LP - 1)) * 4;
            const bool act = row < r1;
            const int64_t base = (int64_t)(act ? row : r0) * a.CL + j0;
            bool ok[4];
            double c[4], uu[4], y[4], xo[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                ok[v] = act && (j0 + v < a.CL);
                c[v] = ok[v] ? (double)a.TL[base + v] : 0.0;
                uu[v] = ok[v] ? (double)a.U[base + v] : 0.0;
                // y_{stage-1} and x_{stage-1}; both are Z_L before the first step
                y[v] = ok[v] ? (double)((stage <= 1 && !more) || stage == 0 ? a.ZL[base + v] : a.Yb[base + v]) : 0.0;
                xo[v] = ok[v] ? (double)(stage <= 1 ? a.ZL[base + v] : a.Xb[base + v]) : 0.0;
            }
            const int lab = act ? a.labels[row] : -1;
            const bool on = lab >= 0;                  // uniform over the lane group; rows without label are no part of F
            double e[4], se, g[4];
            auto gradient = [&](const double (&z)[4], double& lse) {
                lse = 0.0;
                if (a.risk == 0) {
                    lse = row_lse<LPLOG>(z, ok, e, se);
#pragma unroll
                    for (int v = 0; v < 4; ++v) g[v] = ok[v] ? e[v] / se - ((j0 + v) == lab ? 1.0 : 0.0) : 0.0;
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) g[v] = ok[v] ? z[v] - ((j0 + v) == lab ? 1.0 : 0.0) : 0.0;
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) g[v] = ok[v] ? g[v] + uu[v] + (double)a.rho * (z[v] - c[v]) : 0.0;
            };
            double lse_y;
            if (stage > 0 && !more) {
                // take step stage-1 from y with the L its search ended with, then the momentum point
                gradient(y, lse_y);
                const double invL = skipped ? 0.0 : 1.0 / Lcur;
                float xn[4], yn[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    xn[v] = (float)(y[v] - g[v] * invL);
                    yn[v] = xn[v] + mom * (xn[v] - (float)xo[v]);
                }
                if (stage < a.J) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (ok[v]) { a.Xb[base + v] = xn[v]; a.Yb[base + v] = yn[v]; }
                } else {
                    // last stage: the result, and the dual step of Eq. 2 with the old Z_L
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (ok[v]) {
                            const float zold = a.ZL[base + v];
                            a.ZL[base + v] = on ? xn[v] : (float)c[v] - (float)uu[v] / a.rho;
                            if (a.update_u) a.U[base + v] = (float)uu[v] + a.rho * (zold - (float)c[v]);
                        }
                    continue;
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) y[v] = (double)yn[v];
            }
            // the search at y: ||g||^2, ||y||^2, F(y), and F(y - g/L) - F(y) for the candidates L = Lcur eta^q
            gradient(y, lse_y);
            if (!on) continue;                         // (its lanes still took part in the group reductions above)
            double gg = 0.0, yy = 0.0, Fy = 0.0, ug = 0.0, gd = 0.0;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                gg += g[v] * g[v];
                yy += y[v] * y[v];
                ug += uu[v] * g[v];
                gd += g[v] * (y[v] - c[v]);
                const double lin = (j0 + v) == lab ? 1.0 : 0.0;
                Fy += ok[v] ? uu[v] * (y[v] - c[v]) + 0.5 * (double)a.rho * (y[v] - c[v]) * (y[v] - c[v]) +
                                  (a.risk == 0 ? -lin * y[v] : 0.5 * (y[v] - lin) * (y[v] - lin)) : 0.0;
            }
            const bool lead = (threadIdx.x & (LP - 1)) == 0;
            if (a.risk == 0 && lead) Fy += lse_y;
            double gl = 0.0;
#pragma unroll
            for (int v = 0; v < 4; ++v) gl += (j0 + v) == lab ? g[v] : 0.0;
            const double glab = group_sum<LPLOG>(gl);
            const double gg_row = group_sum<LPLOG>(gg), ug_row = group_sum<LPLOG>(ug), gd_row = group_sum<LPLOG>(gd);
            sgg += gg; syy += yy; sF += Fy;
            double Lq = L_round;
#pragma unroll
            for (int q = 0; q < NC; ++q) {
                const double inv = 1.0 / Lq;
                // x - y = -g/L:  <u, x - y> + rho/2 (||x - c||^2 - ||y - c||^2)
                double d = -inv * ug_row + 0.5 * (double)a.rho * (-2.0 * inv * gd_row + inv * inv * gg_row);
                if (a.risk == 0) {
                    double x[4], e2[4], se2;
#pragma unroll
                    for (int v = 0; v < 4; ++v) x[v] = y[v] - g[v] * inv;
                    const double lse_x = row_lse<LPLOG>(x, ok, e2, se2);
                    d += (lse_x - lse_y) + inv * glab;     // R(x) - R(y), with -(x - y)_label = g_label / L
                } else {
                    // 1/2 (||x - e||^2 - ||y - e||^2) = sum (x - y) (y - e) + 1/2 ||x - y||^2
                    double t = 0.0;
#pragma unroll
                    for (int v = 0; v < 4; ++v) t += ok[v] ? g[v] * (y[v] - ((j0 + v) == lab ? 1.0 : 0.0)) : 0.0;
                    d += -inv * group_sum<LPLOG>(t) + 0.5 * inv * inv * gg_row;
                }
                if (lead) D[q] += d;
                Lq *= (double)a.sp.eta;
            }
        }
        if (stage == a.J && !more) continue;
        if (more) {
            block_sums_to<NC>(D, sm, a.partials + ((int64_t)ch * rounds + rd) * NC);
            for (int q = 0; q < NC; ++q) L_round *= (double)a.sp.eta;
        } else {
            double all[NC + kFistaSums];
#pragma unroll
            for (int q = 0; q < NC; ++q) all[q] = D[q];
            all[NC] = sgg; all[NC + 1] = syy; all[NC + 2] = sF;
            block_sums_to<NC + kFistaSums>(all, sm, a.partials + (int64_t)ch * (NC + kFistaSums));
        }
        }
    }
}

// Takes the decisions of a pass.  first_pass: the searches of stage `stage` begin here (the counters of the finished
// stage are added up, every solve starts from L = rho), the step floor is applied, then the first candidates are judged.
__global__ __launch_bounds__(256) void fista_finish_kernel(FistaArgs a, int ncand, int first_pass, int stage) {
    __shared__ double D[kRestCand];               // (a first pass has sixteen candidates at most)
    const int unit = blockIdx.x;
    Unit* u = a.units + unit;
    if (!first_pass && u->done) return;
    const int c0 = a.unit_chunk_ptr[unit], c1 = a.unit_chunk_ptr[unit + 1];
    const int n_val = first_pass ? ncand + kFistaSums : ncand;       // (the chunks are all of rows)
    sum_candidates(a.partials, c0, c1, n_val, n_val, D);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (first_pass) {
            if (stage == 0) { u->step = (double)a.rho; u->total = 0; }
            else u->total += u->ntrials;
            u->ntrials = 0; u->done = 0; u->skip = 0; u->keep = u->step;
            floor_test(u, D[ncand], D[ncand + 1]);
            u->step0 = kFistaSlack * fabs(D[ncand + 2]);       // kept for the passes of further candidates
            if (u->done) return;
        }
        decide(u, D, ncand, a.sp, a.status, u->step0);
    }
}

__global__ void note_flag_kernel(const int32_t* flag, int32_t* note) { *note = *flag; }

__global__ void fill_units_kernel(Unit* units, int n, double step) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Unit u;
    u.step = step; u.step0 = step; u.keep = step; u.g = 0.0; u.bnorm = 0.0; u.done = 0; u.skip = 0; u.ntrials = 0;
    u.spec = 0; u.total = 0; u.fresh = 0; u.c1 = 0.0; u.c2 = 0.0;
    units[i] = u;
}

// rows between the caller's and the internal order, 16 bytes per lane
template <int RM>
__global__ __launch_bounds__(256) void permute_rows_kernel(const float* __restrict__ src, float* __restrict__ dst,
                                                           const int32_t* __restrict__ idx, int64_t N, int C,
                                                           int scatter) {
    const RowWalk w(C);
    const int64_t r_step = (int64_t)gridDim.x * w.r_step;
    for (int64_t r = (int64_t)blockIdx.x * w.r_step + w.r_first; r < N; r += r_step) {
        const int64_t o = idx[r];
        const float* const from = src + (scatter ? r : o) * C;
        float* const to = dst + (scatter ? o : r) * C;
        for (int cv = w.c_first; cv < w.wv; cv += 1 << w.shift) {
            float v[4];
            ldr<RM>(v, from, 4 * cv, C);
            str<RM>(to, 4 * cv, C, v);
        }
    }
}

inline int flat_grid(int64_t count) {
    int64_t nb = (count + 1023) / 1024;     // about four elements per thread at least
    if (nb < 1) nb = 1;
    if (nb > kReduceBlocks) nb = kReduceBlocks;
    return (int)nb;
}

}  // namespace

void launch_phi_G(hipStream_t s, const float* T, const float* Z, float* U, float* G, float* Tprev,
                  int have_prev, int apply_dual, int64_t count, int last, float nu, float rho, double* partials,
                  LayerScalars* out) {
    const int nb = flat_grid(count);
    if (last) hipLaunchKernelGGL((phi_G_kernel<1>), dim3(nb), dim3(256), 0, s, T, Z, U, G, Tprev, have_prev, apply_dual, count, nu, rho, partials);
    else hipLaunchKernelGGL((phi_G_kernel<0>), dim3(nb), dim3(256), 0, s, T, Z, U, G, Tprev, have_prev, apply_dual, count, nu, rho, partials);
    hipLaunchKernelGGL(phi_G_finish_kernel, dim3(1), dim3(256), 0, s, partials, nb, last, nu, out);
}

void launch_G_only(hipStream_t s, const float* T, const float* Z, float* U, float* G, int apply_dual, int64_t count,
                   int last, float nu, float rho) {
    const int nb = flat_grid(count);
    if (last) hipLaunchKernelGGL((G_only_kernel<1>), dim3(nb), dim3(256), 0, s, T, Z, U, G, apply_dual, count, nu, rho);
    else hipLaunchKernelGGL((G_only_kernel<0>), dim3(nb), dim3(256), 0, s, T, Z, U, G, apply_dual, count, nu, rho);
}

void launch_risk(hipStream_t s, const float* ZL, const int32_t* labels, int64_t N, int CL, int risk,
                 double* partials, LayerScalars* out) {
    const int nb = flat_grid(N * 4);
    hipLaunchKernelGGL(risk_kernel, dim3(nb), dim3(256), 0, s, ZL, labels, N, CL, risk, partials);
    hipLaunchKernelGGL(risk_finish_kernel, dim3(1), dim3(256), 0, s, partials, nb, out);
}

void launch_w_begin(hipStream_t s, const double* partials, int n_partials, Unit* unit, SearchParams sp, const int32_t* gate) {
    if (gate) hipLaunchKernelGGL((w_begin_kernel<true>), dim3(1), dim3(256), 0, s, partials, n_partials, unit, sp, gate);
    else hipLaunchKernelGGL((w_begin_kernel<false>), dim3(1), dim3(256), 0, s, partials, n_partials, unit, sp, gate);
}

void launch_rest_start(hipStream_t s, int L, int M, Unit* unitsW, Unit* unitsZ, int32_t* moved, uint64_t ungated, int32_t* left_g,
                       const int32_t* bad) {
    hipLaunchKernelGGL(rest_start_kernel, dim3(1), dim3(256), 0, s, L, M, unitsW, unitsZ, moved, ungated, left_g, bad);
}

void launch_rest_w(hipStream_t s, int L, const Unit* unitsW, const int32_t* moved, int32_t* left_g, int32_t* run_w, int32_t* run_z) {
    hipLaunchKernelGGL(rest_w_kernel, dim3(1), dim3(64), 0, s, L, unitsW, moved, left_g, run_w, run_z);
}

void launch_rest_z(hipStream_t s, int L, const Unit* unitsW, int32_t* run_z) {
    hipLaunchKernelGGL(rest_z_kernel, dim3(1), dim3(64), 0, s, L, unitsW, run_z);
}

void launch_w_trial_finish(hipStream_t s, double* partials, int n_partials, SearchParams sp, Unit* unit,
                           int32_t* status) {
    hipLaunchKernelGGL(w_trial_finish_kernel, dim3(1), dim3(256), 0, s, partials, n_partials, 1, sp, unit, status, 0);
}

void launch_w_last_search(hipStream_t s, const float* T0, const float* Q, const float* Z, const float* U, int64_t count,
                          SearchParams sp, Unit* unit, double* partials, int32_t* status) {
    const int nb = flat_grid(count);
    hipLaunchKernelGGL(w_last_sums_kernel, dim3(nb), dim3(256), 0, s, T0, Q, Z, U, count, sp.rho, unit, partials);
    hipLaunchKernelGGL(w_last_finish_kernel, dim3(1), dim3(256), 0, s, partials, nb, sp, unit, status);
}

void launch_w_trial(hipStream_t s, const float* T0, const float* Q, const float* Z, int64_t count, int ncand,
                    SearchParams sp, Unit* unit, double* partials, int32_t* status, int speculated) {
    int nb = flat_grid(count);
    // a fresh search needs more than four candidates: the pass after this one starts it, if the passes then still hold them all
    const int leave_fresh = ncand == 4 && (sp.max_backtrack > 4 + kFreshCand || (sp.max_backtrack > 4 && sp.max_backtrack <= kFreshCand));
    if (ncand == 1)
        hipLaunchKernelGGL((w_trial_kernel<1>), dim3(nb), dim3(256), 0, s, T0, Q, Z, count, sp, 1, unit, partials, speculated, 0);
    else if (ncand <= 4)
        hipLaunchKernelGGL((w_trial_kernel<4>), dim3(nb), dim3(256), 0, s, T0, Q, Z, count, sp, 1, unit, partials, speculated, leave_fresh);
    else if (ncand == kFreshCand)
        hipLaunchKernelGGL((w_trial_kernel<kFreshCand>), dim3(nb), dim3(256), 0, s, T0, Q, Z, count, sp, 1, unit, partials, speculated, 0);
    else {
        // The rounds of a small matrix share the chip (2000 x 64, four rounds: 31 us in one after the other, 5 so), up to as many
        // workgroups as a large one has in a single round.  Those of a large one follow each other: each round fills the chip by
        // itself, and where the search is over, as it mostly is in this pass, 2048 workgroups that leave at once and the
        // launch behind them take 3.1 us, 4 x 2048 4.4.
        const int rounds = (ncand + kMaxCand - 1) / kMaxCand;
        const int side_by_side = std::max(1, std::min(rounds, kReduceBlocks / nb));
        hipLaunchKernelGGL((w_trial_kernel<kMaxCand>), dim3(nb, side_by_side), dim3(256), 0, s, T0, Q, Z, count, sp, rounds, unit,
                           partials, speculated, 0);
    }
    const int nc = ncand == 1 ? 1 : ncand <= 4 ? 4 : ncand == kFreshCand ? kFreshCand : (ncand + kMaxCand - 1) / kMaxCand * kMaxCand;
    hipLaunchKernelGGL(w_trial_finish_kernel, dim3(1), dim3(256), 0, s, partials, nb, nc, sp, unit, status, leave_fresh);
}

void launch_w_step(hipStream_t s, float* W, float* Wt, const float* gradW, int K, int C, float* T, float* Q,
                   int64_t count_t, const Unit* unit, int speculated, const float* Z, float nu) {
    const int64_t cw = (int64_t)K * C;
    const int nb = flat_grid(count_t > cw ? count_t : cw);
    hipLaunchKernelGGL((w_step_kernel<0>), dim3(nb), dim3(256), 0, s, W, Wt, gradW, K, C, T, Q, count_t, unit, speculated,
                       Z, nullptr, Z ? Q : nullptr, nullptr, nu, 0.f);
}

void launch_w_step_last(hipStream_t s, float* W, float* Wt, const float* gradW, int K, int C, float* T, const float* Q,
                        int64_t count_t, const Unit* unit, const float* Z, const float* U, float* G, float* Tprev, float rho) {
    const int64_t cw = (int64_t)K * C;
    const int nb = flat_grid(count_t > cw ? count_t : cw);
    hipLaunchKernelGGL((w_step_kernel<1>), dim3(nb), dim3(256), 0, s, W, Wt, gradW, K, C, T, Q, count_t, unit, 0, Z, U, G,
                       Tprev, 0.f, rho);
}

// calls f with the width's kind as an integral constant
template <class F>
static void with_mode(int width, F f) {
    if (width % 4 == 0) f(std::integral_constant<int, kFull>{});
    else if (width >= 4) f(std::integral_constant<int, kTail>{});
    else f(std::integral_constant<int, kNarrow>{});
}
// calls f with a condition as an integral constant
template <class F>
static void with_flag(bool is, F f) {
    if (is) f(std::true_type{});
    else f(std::false_type{});
}

template <int PART>
static void launch_first_part(hipStream_t s, const ZTrialArgs& a) {
    const dim3 grid(a.n_chunks), block(256);
    const auto go = [&](auto hid, auto sm) {
        constexpr int HID = decltype(hid)::value, SM = decltype(sm)::value;
        if (a.n_chunks > 0) hipLaunchKernelGGL((z_first_kernel<HID, SM, PART>), grid, block, 0, s, a);
        hipLaunchKernelGGL((z_first_finish_kernel<HID, PART>), dim3(a.M), block, 0, s, a);
    };
    const std::integral_constant<int, 0> last;
    const std::integral_constant<int, 1> hidden;
    if constexpr (PART == kRowsOnly) go(last, std::integral_constant<int, kFull>{});        // (the rows know nothing of the next layer)
    else with_mode(a.Cn, [&](auto sm) { a.next_is_last ? go(last, sm) : go(hidden, sm); });
}
void launch_z_floor(hipStream_t s, const ZTrialArgs& a) { launch_first_part<kRowsOnly>(s, a); }
void launch_z_first(hipStream_t s, const ZTrialArgs& a) {
    if (a.gate) launch_first_part<kSegmentsOnly>(s, a);
    else launch_first_part<kBoth>(s, a);
}

void launch_z_more(hipStream_t s, const ZTrialArgs& a, int ncand) {
    // the pass of four is often needed and takes a grid that fills the chip, the others hardly ever
    const int cap = ncand <= 4 ? kReduceBlocks : kReduceBlocks / 4;
    const dim3 grid(a.n_chunks < cap ? a.n_chunks : cap), block(256);
    const int rounds = (ncand + kMaxCand - 1) / kMaxCand;
    if (a.n_chunks > 0)
        with_mode(a.Cn, [&](auto sm) {
            constexpr int SM = decltype(sm)::value;
            if (ncand <= 4) hipLaunchKernelGGL((z_more_kernel<4, SM>), grid, block, 0, s, a, 1);
            else hipLaunchKernelGGL((z_more_kernel<kMaxCand, SM>), grid, block, 0, s, a, rounds);
        });
    hipLaunchKernelGGL(z_more_finish_kernel, dim3(a.M), dim3(256), 0, s, a, ncand <= 4 ? 4 : rounds * kMaxCand);
}

void launch_z_step(hipStream_t s, float* Zl, const float* gradZ, const int32_t* row_comm, int64_t N, int Cl,
                   const Unit* units, int M, const int32_t* gate) {
    const int nb = flat_grid(N * (int64_t)Cl);
    with_mode(Cl, [&](auto rm) {
        constexpr int RM = decltype(rm)::value;
        with_flag(gate != nullptr, [&](auto gated) {
            constexpr bool GATED = decltype(gated)::value;
            if (M <= kStepUnits) hipLaunchKernelGGL((z_step_kernel<true, RM, GATED>), dim3(nb), dim3(256), 0, s, Zl, gradZ, row_comm, N, Cl, units, M, gate);
            else hipLaunchKernelGGL((z_step_kernel<false, RM, GATED>), dim3(nb), dim3(256), 0, s, Zl, gradZ, row_comm, N, Cl, units, M, gate);
        });
    });
}

void launch_z_step_lowrank(hipStream_t s, float* Zl, const float* Tl, const float* SG, const float* Wt, float nu,
                           const int32_t* row_comm, int64_t N, int Cl, int Cn, const Unit* units, int M, const int32_t* gate) {
    // more and smaller workgroups than the reducing kernels use: nothing is reduced here
    int64_t nb = (N * (int64_t)Cl + 2047) / 2048;
    nb = nb < 1 ? 1 : (nb > 4 * kReduceBlocks ? 4 * kReduceBlocks : nb);
    const size_t lds = (size_t)Cn * Cl * sizeof(float);                 // at most 16 x 1024 floats (the low-rank limit)
    with_mode(Cn, [&](auto sm) {
        constexpr int SM = decltype(sm)::value;
        with_flag(gate != nullptr, [&](auto gated) {
            constexpr bool GATED = decltype(gated)::value;
            if (M <= kStepUnits) hipLaunchKernelGGL((z_step_lowrank_kernel<true, SM, GATED>), dim3((unsigned)nb), dim3(256), lds, s, Zl, Tl, SG, Wt, nu, row_comm, N, Cl, Cn, units, M, gate);
            else hipLaunchKernelGGL((z_step_lowrank_kernel<false, SM, GATED>), dim3((unsigned)nb), dim3(256), lds, s, Zl, Tl, SG, Wt, nu, row_comm, N, Cl, Cn, units, M, gate);
        });
    });
}

void launch_t_carry(hipStream_t s, float* Tn, const CarryArgs& k, int64_t N, int Cn) {
    const int nb = flat_grid(N * (int64_t)Cn * 4);
    with_mode(Cn, [&](auto sm) {
        with_flag(k.gate != nullptr, [&](auto gated) {
            hipLaunchKernelGGL((t_carry_kernel<decltype(sm)::value, decltype(gated)::value>), dim3(nb), dim3(256), 0, s, Tn, k, N, Cn);
        });
    });
}

void launch_last_layer(hipStream_t s, float* ZL, float* U, float* TL, const int32_t* labels, int64_t N,
                       int CL, int risk, float rho, int J, int update_u, const CarryArgs* carry, float* G) {
    const CarryArgs k = carry ? *carry : CarryArgs();
    with_mode(CL, [&](auto sm) {
        constexpr int SM = decltype(sm)::value;
        auto go = [&](auto lg) {
            constexpr int LG = decltype(lg)::value;
            const dim3 grid((unsigned)(((N << LG) + 255) / 256));
            if (carry && k.gate) hipLaunchKernelGGL((last_layer_kernel<LG, 1, SM, true>), grid, dim3(256), 0, s, ZL, U, TL, labels, N, CL, risk, rho, J, update_u, k, G);
            else if (carry) hipLaunchKernelGGL((last_layer_kernel<LG, 1, SM, false>), grid, dim3(256), 0, s, ZL, U, TL, labels, N, CL, risk, rho, J, update_u, k, G);
            else hipLaunchKernelGGL((last_layer_kernel<LG, 0, SM, false>), grid, dim3(256), 0, s, ZL, U, TL, labels, N, CL, risk, rho, J, update_u, k, nullptr);
        };
        if constexpr (SM == kNarrow) {
            go(std::integral_constant<int, 0>{});
        } else {
            if (CL <= 4) go(std::integral_constant<int, 0>{});
            else if (CL <= 8) go(std::integral_constant<int, 1>{});
            else if (CL <= 16) go(std::integral_constant<int, 2>{});
            else if (CL <= 32) go(std::integral_constant<int, 3>{});
            else go(std::integral_constant<int, 4>{});
        }
    });
}

void launch_relu(hipStream_t s, const float* T, float* Z, int64_t count, int apply_relu) {
    hipLaunchKernelGGL(relu_kernel, dim3(flat_grid(count)), dim3(256), 0, s, T, Z, count, apply_relu);
}

void launch_argmax_rows(hipStream_t s, const float* T, int32_t* pred, const int32_t* perm, const int32_t* labels, int32_t* hits,
                        int64_t N, int C) {
    hipLaunchKernelGGL(argmax_rows_kernel, dim3(kArgmaxBlocks), dim3(256), 0, s, T, pred, perm, labels, hits, N, C);
}

void launch_fista_stage(hipStream_t s, const FistaArgs& a, int stage, int more, int ncand, float mom) {
    if (a.n_chunks <= 0) return;
    // more = 0: the pass that takes the step and tries the first candidates; more = 1: ncand further candidates, four on a
    // grid that fills the chip (a step usually needs one or two doublings, in many communities at once), more of them on a
    // small grid, which usually finds nothing pending
    const int nc = ncand <= 1 ? 1 : ncand <= 4 ? 4 : kMaxCand;
    const int rounds = (ncand + nc - 1) / nc;
    const int cap = more == 0 ? a.n_chunks : (nc == 4 ? kReduceBlocks : kReduceBlocks / 4);
    const int nb = a.n_chunks < cap ? a.n_chunks : cap;
#define CADMM_FISTA(LG_) do { \
        if (nc == kMaxCand) hipLaunchKernelGGL((fista_stage_kernel<LG_, kMaxCand>), dim3(nb), dim3(256), 0, s, a, stage, more, rounds, mom); \
        else if (nc == 4) hipLaunchKernelGGL((fista_stage_kernel<LG_, 4>), dim3(nb), dim3(256), 0, s, a, stage, more, rounds, mom); \
        else hipLaunchKernelGGL((fista_stage_kernel<LG_, 1>), dim3(nb), dim3(256), 0, s, a, stage, more, rounds, mom); } while (0)
    if (a.CL <= 4) CADMM_FISTA(0);
    else if (a.CL <= 8) CADMM_FISTA(1);
    else if (a.CL <= 16) CADMM_FISTA(2);
    else if (a.CL <= 32) CADMM_FISTA(3);
    else CADMM_FISTA(4);
#undef CADMM_FISTA
    if (stage < a.J) hipLaunchKernelGGL(fista_finish_kernel, dim3(a.M), dim3(256), 0, s, a, nc * rounds, more ? 0 : 1, stage);
}

void launch_note_flag(hipStream_t s, const int32_t* flag, int32_t* note) {
    hipLaunchKernelGGL(note_flag_kernel, dim3(1), dim3(1), 0, s, flag, note);
}

void launch_fill_units(hipStream_t s, Unit* units, int n, double step) {
    hipLaunchKernelGGL(fill_units_kernel, dim3((n + 255) / 256), dim3(256), 0, s, units, n, step);
}

void launch_permute_rows(hipStream_t s, const float* src, float* dst, const int32_t* idx, int64_t N, int C,
                         int scatter) {
    with_mode(C, [&](auto rm) {
        hipLaunchKernelGGL((permute_rows_kernel<decltype(rm)::value>), dim3(flat_grid(N * (int64_t)((C + 3) & ~3))), dim3(256), 0, s, src,
                           dst, idx, N, C, scatter);
    });
}

}  // namespace cadmm

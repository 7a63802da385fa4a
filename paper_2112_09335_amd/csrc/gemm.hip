// Dense fp32 contractions of the sweep on the gfx950 matrix cores: v_mfma_f32_32x32x2_f32, or (default for results
// wider than 32 columns, the *_split_kernel variants) v_mfma_f32_32x32x16_bf16 on operands split exactly into
// three bf16 parts each, or (large products inside the sweep, the *_pair_kernel variants) v_mfma_f32_32x32x16_f16 on
// scaled operands of two fp16 parts each, half as many instructions again, where that gives the fp32 kernels' accuracy too,
// at a fraction of the matrix-core time:
//   gemm_nn : out[n x C] = A[n x K] B[K x C]     (T_l = H_l W_l, Q = H_l gradW, G W^T, gradZ W;
//                                                 paper Section 3.1 and Appendix A)
//   gemm_tn : out[K x C] = A[n x K]^T G[n x C]   (gradient of phi with respect to W_l: a sum over all
//                                                 nodes of all communities, Section 3.1)
// n is the number of nodes (up to millions), K and C are layer widths (1..4096).
//
// Tiling: 256 threads = 4 wavefronts per workgroup, operands staged through LDS, the next steps prefetched into registers
// while the current one feeds the MFMAs.
//   split products and fp32 products wider than 32 columns: 2 x 2 wavefronts, 128 x 128 results and 16 of the contraction
//   per step; split products with few tiles 64 x 64 (kFewTiles);
//   products on pairs: 128 x 256 results; W gradients whose rows fill them: 256 x 128; see there;
//   results of at most 32 columns: a wavefront forms 32 rows by 32 columns, 32 of the contraction per step.
// MFMA operand layout for 32x32x2 (64 lanes): lane holds A[i = lane%32][k = lane/32] and B[k = lane/32][j = lane%32];
// accumulator register r of a lane is C[8*(r/4) + 4*(lane/32) + r%4][lane%32].
// gemm_tn splits n into chunks, each block reduces one chunk for one result tile (128 or 64 rows of K) into a partial
// matrix; a second kernel adds the partials in chunk order in fp64 (deterministic).
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace cadmm {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int BM = 128;
constexpr int BK = 16;

// Four consecutive columns c .. c+3 of a row of `width` floats; entries past the row's end read as zero.  Every variant is
// free of branches: a load under a condition that differs between lanes makes the compiler wait for one load before it
// issues the next.  The chip takes 16-byte global accesses at any dword, so rows of any width are read in quads:
//   width a multiple of four (kFull): the quad is there or not at all;
//   other widths of four and more (kTail): the last quad is moved back to end with the row, and its entries into place;
//   one to three columns (kNarrow): dwords.
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
enum RowMode { kFull = 0, kTail = 1, kNarrow = 2 };
__device__ __forceinline__ int row_mode(int width) { return width % 4 == 0 ? kFull : width >= 4 ? kTail : kNarrow; }
// Loading and putting the quad right are two steps, so that a kernel that fetches ahead does the second where it uses the
// quad: anything done to a loaded value right away makes the fetch wait for it.
template <int MODE>
__device__ __forceinline__ float4 ld_quad_raw(const float* row, int c, int width) {
    if constexpr (MODE == kNarrow) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = row[c + e < width ? c + e : width - 1];
        return make_float4(v[0], v[1], v[2], v[3]);
    } else {
        const int cc = MODE == kFull ? (c < width ? c : 0) : (c + 4 <= width ? c : width - 4);
        const float4u q = *reinterpret_cast<const float4u*>(row + cc);
        return make_float4(q.x, q.y, q.z, q.w);
    }
}
template <int MODE>
__device__ __forceinline__ float4 fix_quad(float4 q, int c, int width) {
    if constexpr (MODE == kFull) {
        const bool in = c < width;
        return make_float4(in ? q.x : 0.f, in ? q.y : 0.f, in ? q.z : 0.f, in ? q.w : 0.f);
    } else if constexpr (MODE == kTail) {
        const int off = c + 4 <= width ? 0 : c + 4 - width;     // how many entries of the quad come before column c
        const bool o2 = (off & 2) != 0, o1 = (off & 1) != 0, none = off >= 4;
        const float a0 = o2 ? q.z : q.x, a1 = o2 ? q.w : q.y, a2 = o2 ? 0.f : q.z, a3 = o2 ? 0.f : q.w;
        const float b0 = o1 ? a1 : a0, b1 = o1 ? a2 : a1, b2 = o1 ? a3 : a2, b3 = o1 ? 0.f : a3;
        return make_float4(none ? 0.f : b0, none ? 0.f : b1, none ? 0.f : b2, none ? 0.f : b3);
    } else {
        return make_float4(c < width ? q.x : 0.f, c + 1 < width ? q.y : 0.f, c + 2 < width ? q.z : 0.f, c + 3 < width ? q.w : 0.f);
    }
}
template <int MODE>
__device__ __forceinline__ float4 ld_quad(const float* row, int c, int width) {
    return fix_quad<MODE>(ld_quad_raw<MODE>(row, c, width), c, width);
}
__device__ __forceinline__ float4 ld_quad_raw(int mode, const float* row, int c, int width) {        // mode: uniform
    if (mode == kFull) return ld_quad_raw<kFull>(row, c, width);
    if (mode == kTail) return ld_quad_raw<kTail>(row, c, width);
    return ld_quad_raw<kNarrow>(row, c, width);
}
__device__ __forceinline__ float4 fix_quad(int mode, float4 q, int c, int width) {
    if (mode == kFull) return fix_quad<kFull>(q, c, width);
    if (mode == kTail) return fix_quad<kTail>(q, c, width);
    return fix_quad<kNarrow>(q, c, width);
}
// stores up to four entries of a flat array of which `valid` (one to four) exist
__device__ __forceinline__ void st4u(float* p, const float (&d)[4], int valid) {
    if (valid >= 4) {
        float4u v = {d[0], d[1], d[2], d[3]};
        *reinterpret_cast<float4u*>(p) = v;
    } else {
        p[0] = d[0];
        if (valid > 1) p[1] = d[1];
        if (valid > 2) p[2] = d[2];
    }
}
// Consecutive workgroups go round-robin to the eight XCDs, each with an L2 of its own.  Workgroups that read the
// same operand tile (the `inner` column tiles of one row tile, the tiles of one row chunk) are therefore given
// indices 8 apart, so that they run at about the same time on ONE XCD and the shared tile comes from its L2.
// The last, incomplete set of 8 * inner workgroups keeps the plain order.  (outer, in) is a bijection of blockIdx.
__device__ __forceinline__ void xcd_group(unsigned b, unsigned nb, unsigned inner, int64_t& outer, int& in) {
    const unsigned set = 8u * inner;
    if (b < nb / set * set) {
        const unsigned w = b % set;
        outer = (int64_t)(b / set) * 8 + (w & 7u);
        in = (int)(w >> 3);
    } else {
        outer = b / inner;
        in = (int)(b % inner);
    }
}

// What an epilogue does with one quad of results (EPI as below): v the product's, z and t the rows of Zl and of Tl (Tio), o the
// quad's place in the result matrix, nv how many of its columns exist there.
struct EpilogueArgs {
    float* out;
    const float* Zl;
    const float* tin;
    float nu;
    float* Tio;
    double inv0;             // EPI 2, 4: 1 / first candidate
    bool take, hold;         // EPI 2, 4: the step is taken ahead; EPI 4: no step at all
};
template <int EPI, int MODE>
__device__ __forceinline__ void epilogue_quad(float (&v)[4], float4 z4, float4 t4, int64_t o, int nv, const EpilogueArgs& a,
                                              double& dsum) {
    float t[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (EPI == 1 || EPI == 2 || EPI == 4) {
        const float z[4] = {z4.x, z4.y, z4.z, z4.w};
        t[0] = t4.x; t[1] = t4.y; t[2] = t4.z; t[3] = t4.w;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // (columns past C hold a copy of the last one; with z and t zero there a zero adds nothing)
            if constexpr (MODE != kFull) v[e] = e < nv ? v[e] : 0.f;
            if constexpr (EPI == 1) v[e] = a.nu * (z[e] - fmaxf(t[e], 0.f)) + v[e];
            if constexpr (EPI == 2 || EPI == 4) {
                const double t0 = (double)t[e], zd = (double)z[e];
                const double t1 = t0 - (double)v[e] * a.inv0;
                const double e0 = fmax(t0, 0.0) - zd, e1 = fmax(t1, 0.0) - zd;
                dsum += (e1 - e0) * (e1 + e0);
                t[e] = (float)t1;
            }
        }
    }
    if constexpr (EPI == 2) {
        if (a.take) st4u(a.Tio + o, t, nv);
        else st4u(a.out + o, v, nv);
    } else if constexpr (EPI == 4) {
        if (a.take) st4u(a.Tio + o, t, nv);
        if (a.take || a.hold) {                                  // (as launch_G_only forms it)
            const float z[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = t[e] > 0.f ? a.nu * (float)((double)t[e] - (double)z[e]) : 0.f;
        }
        st4u(a.out + o, v, nv);
    } else if constexpr (EPI == 3) {
        // (a finite number times zero is zero, any other is no number; entries past the row's end repeat finite ones or not)
        dsum += (double)((v[0] * 0.f + v[1] * 0.f) + (v[2] * 0.f + v[3] * 0.f));
        if (a.out) st4u(a.out + o, v, nv);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
        st4u(a.Tio + o, v, nv);
    } else {
        st4u(a.out + o, v, nv);
    }
}
// EPI 1: RowSums of a quad of columns c .. c + 3 (of C), over 16 or 32 neighbouring lanes (LANES); every one of them gets the sums.
template <int LANES>
__device__ __forceinline__ void quad_row_sums(double (&rs)[3], const float (&v)[4], float4 z4, float4 t4, int c, int C, float nu) {
    const float z[4] = {z4.x, z4.y, z4.z, z4.w}, tt[4] = {t4.x, t4.y, t4.z, t4.w};
    rs[0] = rs[1] = rs[2] = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool in = c + e < C;
        const float g = nu * (z[e] - fmaxf(tt[e], 0.f)) + v[e];
        const double zd = in ? (double)z[e] : 0.0, gd = in ? (double)g : 0.0;
        rs[0] += (zd - fmax((double)tt[e], 0.0)) * gd;
        rs[1] += gd * gd;
        rs[2] += zd * zd;
    }
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1)
#pragma unroll
        for (int s = 0; s < 3; ++s) rs[s] += __shfl_xor(rs[s], o, 64);
}

// Epilogue of a result tile of 64 T x 64 T held as T x T accumulators per wavefront (2 x 2 wavefronts).
// The accumulators hold 32 consecutive columns per row and lane group; passing each 32-row slab of the tile
// through LDS (Cs: 32 x (64 T + 4) floats, the operand buffer reused) turns every global access of the epilogue into
// 16-byte pieces of a row of 256 T bytes.
// EPI 0: out = acc.  EPI 1: out = nu (Zl - relu(Tl)) + acc.  EPI 2: first candidate of the W search and the step
// on Tio ahead of the decision, see GemmEpilogue.  EPI 3: out (if there is one) = acc, Tio = relu(acc).
// EPI 4: 2 that leaves G (GemmEpilogue::leave_g); an epilogue of its own, since its registers made the product of 2 spill
// (2M x 128 x 256: 1444 us without it, 1681 with).
template <int EPI, int T, int MODE>
__device__ __forceinline__ void tile_epilogue_mode(floatx16 (&acc)[T][T], float* Cs, int64_t m0, int c0, int64_t n, int C,
                                                   const EpilogueArgs& args, double& dsum, double* __restrict__ row_sums) {
    constexpr int BN = 64 * T;
    constexpr int LDC = BN + 4;
    constexpr int Q = BN / 4;                            // quads per row
    constexpr int PER_T = 32 * Q / 256;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, lk = lane >> 5;
#pragma unroll
    for (int q = 0; q < 2 * T; ++q) {
        __syncthreads();
        if (wm == q / T) {
#pragma unroll
            for (int j = 0; j < T; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    Cs[(8 * (r >> 2) + 4 * lk + (r & 3)) * LDC + wn * 32 * T + j * 32 + li] = acc[q % T][j][r];
        }
        __syncthreads();
        // two 16-byte pieces of a lane at a time, their loads before either is used (more would cost the product registers)
#pragma unroll
        for (int u0 = 0; u0 < PER_T; u0 += 2) {
            float4 z4[2], t4[2];
            if constexpr (EPI == 1 || EPI == 2 || EPI == 4) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int f = tid + 256 * (u0 + u);
                    const int64_t row = m0 + 32 * q + f / Q;
                    const int64_t ro = (row < n ? row : n - 1) * (int64_t)C;
                    z4[u] = ld_quad<MODE>(args.Zl + ro, c0 + 4 * (f % Q), C);
                    t4[u] = ld_quad<MODE>(args.tin + ro, c0 + 4 * (f % Q), C);
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int f = tid + 256 * (u0 + u);
                const int rl = f / Q, cq = f % Q;
                const int64_t row = m0 + 32 * q + rl;
                const int c = c0 + 4 * cq;
                const float4 v4 = *reinterpret_cast<const float4*>(Cs + rl * LDC + 4 * cq);
                float v[4] = {v4.x, v4.y, v4.z, v4.w};
                if constexpr (EPI == 1) {
                    if (row_sums) {                              // (uniform) the row's sums over this tile's columns
                        double rs[3];
                        quad_row_sums<Q>(rs, v, z4[u], t4[u], c, C, args.nu);
                        if (cq < 3 && row < n) row_sums[((int64_t)(c0 / BN) * n + row) * 3 + cq] = cq == 0 ? rs[0] : cq == 1 ? rs[1] : rs[2];
                    }
                }
                if (row >= n || c >= C) continue;
                // columns of this lane: four, or the row's last few
                epilogue_quad<EPI, MODE>(v, z4[u], t4[u], row * C + c, MODE == kFull ? 4 : C - c, args, dsum);
            }
        }
    }
}

// EPI 3: *bad = 1 if a result was not finite; s: what epilogue_quad has added up (bad: null if nobody asks).
__device__ __forceinline__ void note_bad(double s, int32_t* bad) {
    if (bad && __any(!(s == 0.0)) && (threadIdx.x & 63) == 0) atomicOr(bad, 1);
}

template <int EPI, int T>
__device__ __forceinline__ void tile_epilogue(floatx16 (&acc)[T][T], float* Cs, int64_t m0, int c0, int64_t n, int C,
                                              float* __restrict__ out, const float* __restrict__ Zl,
                                              const float* __restrict__ Tl, float nu, float* __restrict__ Tio,
                                              const Unit* unit, double* __restrict__ partials) {
    // (epilogue 1 has no partials: the argument then carries the row sums)
    double* const row_sums = EPI == 1 ? partials : nullptr;
    double inv0 = 0.0, dsum = 0.0;
    bool take = false, hold = false;
    if constexpr (EPI == 2 || EPI == 4) {
        hold = EPI == 4 && unit->skip != 0;
        inv0 = unit->skip ? 0.0 : 1.0 / unit->step0;
        take = unit->spec != 0 && !unit->skip;
    }
    const EpilogueArgs args{out, Zl, (EPI == 2 || EPI == 4) ? Tio : Tl, nu, Tio, inv0, take, hold};
    if (C % 4 == 0) tile_epilogue_mode<EPI, T, kFull>(acc, Cs, m0, c0, n, C, args, dsum, row_sums);
    else tile_epilogue_mode<EPI, T, kTail>(acc, Cs, m0, c0, n, C, args, dsum, row_sums);   // (C > 32)
    // (nor has epilogue 3: it carries the flag)
    if constexpr (EPI == 3) note_bad(dsum, reinterpret_cast<int32_t*>(partials));
    if constexpr (EPI == 2 || EPI == 4) {
        __shared__ double red[4];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = dsum;
        __syncthreads();
        if (threadIdx.x == 0) partials[blockIdx.x] = 0.5 * (double)nu * (red[0] + red[1] + red[2] + red[3]);
    }
}

// ------------------------------------------------------------------------------------------------ NN
// EPI 1: out = nu * (Zl - relu(Tl)) + A B   (gradient of the Z subproblem, Appendix A)
// EPI 2: out = Q = A B; first candidate of the W search and speculative step on Tio (Section 3.1), see kernels.h
// EPI 3: Tio = relu(A B), and out = A B if there is an out;  EPI 4: 2, and G where the step is taken ahead or not at all
template <int EPI>
__global__ __launch_bounds__(256) void gemm_nn_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                      float* __restrict__ out, int64_t n, int K, int C,
                                                      const float* __restrict__ Zl, const float* __restrict__ Tl,
                                                      float nu, float* __restrict__ Tio, const Unit* unit,
                                                      double* __restrict__ partials, const int32_t* __restrict__ gate) {
    constexpr int BN = 128;
    constexpr int LDA = BK + 1;
    constexpr int LDB = BN + 4;

    // one buffer: the operand tiles during the product, a 32-row slab of the result tile afterwards
    __shared__ __align__(16) float smem[BM * LDA + BK * LDB];
    float* const As = smem;
    float* const Bs = smem + BM * LDA;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int ctiles = (C + BN - 1) / BN;
    if constexpr (EPI == 0) {
        if (gate && *gate == 0) return;
        // gated plain product: Q again for a W search whose speculative step (epilogue 2, Q not stored) was rejected
        if (unit != nullptr && (!unit->spec || unit->skip || (unit->done && unit->step == unit->step0))) return;
    }
    int64_t mtile;
    int ctile;
    xcd_group(blockIdx.x, gridDim.x, (unsigned)ctiles, mtile, ctile);
    const int64_t m0 = mtile * BM;
    const int c0 = ctile * BN;

    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    float4 ra[2], rb[2];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int f = tid + 256 * i;
            const int64_t gr = m0 + (f >> 2) < n ? m0 + (f >> 2) : n - 1;
            const int k = k0 + (f >> 5) < K ? k0 + (f >> 5) : K - 1;
            const float* ar = A + gr * K;
            const float* br = B + (int64_t)k * C;
            if (K % 4 == 0) ra[i] = ld_quad<kFull>(ar, k0 + 4 * (f & 3), K);
            else if (K >= 4) ra[i] = ld_quad<kTail>(ar, k0 + 4 * (f & 3), K);
            else ra[i] = ld_quad<kNarrow>(ar, k0 + 4 * (f & 3), K);
            // (both operands are zero past K: a zero times an infinity would not be)
            const float4 b = C % 4 == 0 ? ld_quad<kFull>(br, c0 + 4 * (f & 31), C) : ld_quad<kTail>(br, c0 + 4 * (f & 31), C);
            rb[i] = k0 + (f >> 5) < K ? b : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int f = tid + 256 * i;
            float* d = As + (f >> 2) * LDA + 4 * (f & 3);
            d[0] = ra[i].x; d[1] = ra[i].y; d[2] = ra[i].z; d[3] = ra[i].w;
            *reinterpret_cast<float4*>(Bs + (f >> 5) * LDB + 4 * (f & 31)) = rb[i];
        }
    };

    int nk = (K + BK - 1) / BK;
    if constexpr (EPI == 2 || EPI == 4) {
        if (unit->skip) {           // no step is taken: nothing reads Q; epilogue 4 leaves G of the T that stays
            if (EPI == 2) return;
            nk = 0;
        }
    }
    fetch(0);
    for (int kt = 0; kt < nk; ++kt) {
        __syncthreads();            // previous tile fully consumed
        stash();
        __syncthreads();
        if (kt + 1 < nk) fetch((kt + 1) * BK);
        const int li = lane & 31, lk = lane >> 5;
#pragma unroll
        for (int kk = 0; kk < BK; kk += 2) {
            float a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = As[(wm * 64 + i * 32 + li) * LDA + kk + lk];
#pragma unroll
            for (int j = 0; j < 2; ++j) b[j] = Bs[(kk + lk) * LDB + wn * 64 + j * 32 + li];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
    static_assert(32 * (BN + 4) <= BM * LDA + BK * LDB, "result slab must fit the operand buffer");
    tile_epilogue<EPI, 2>(acc, smem, m0, c0, n, C, out, Zl, Tl, nu, Tio, unit, partials);
}

// Results of at most 32 columns: bound by reading A, so a step takes 32 columns of it (a whole 128-byte line of every
// row; no half line has to survive in the L2 until the next step).  A wavefront forms 32 rows.
//   SPLIT 0: four wavefronts share a workgroup's 128 rows and its tile of B.
//   SPLIT 1: they share 32 rows and take a quarter of the K steps each, added up in LDS at the end.  For few rows: a
//   workgroup per 128 rows leaves most of the chip idle and its K steps are one chain of memory latencies
//   (13752 x 1000 by 10 columns: 77 us in 108 workgroups, 17 us in 430).
// EPI kGated: 0 behind a gate (GemmEpilogue::gate), an instance of its own: a branch on the gate's pointer, null or not, keeps the
// other arguments from being loaded beside it, a twentieth of a small product (20000 x 128 by 3 columns: 6.7 us without, 7.15 with).
constexpr int kGated = 5;
template <int EPI, int SPLIT>
__global__ __launch_bounds__(256) void gemm_nn_narrow_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                             float* __restrict__ out, int64_t n, int K, int C,
                                                             const float* __restrict__ Zl, const float* __restrict__ Tl,
                                                             float nu, float* __restrict__ relu_out, const int32_t* __restrict__ gate) {
    if constexpr (EPI == kGated) {
        if (*gate == 0) return;
    }
    constexpr int KS = 32;
    constexpr int LDA = KS + 1;
    constexpr int LDB = 32 + 4;
    constexpr int A_TILE = 32 * LDA, B_TILE = KS * LDB;
    constexpr int B_PER_T = SPLIT ? 4 : 1;
    __shared__ __align__(16) float As[4 * A_TILE];                       // 32 rows per wavefront
    __shared__ __align__(16) float Bs[(SPLIT ? 4 : 1) * B_TILE];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t m0 = (int64_t)blockIdx.x * (SPLIT ? 32 : 128) + (SPLIT ? 0 : 32 * wave);   // this wavefront's rows
    const int li = lane & 31, lk = lane >> 5;
    float* const Aw = As + wave * A_TILE;
    float* const Bw = Bs + (SPLIT ? wave * B_TILE : 0);
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    // A: lane takes quad lane % 8 of rows lane / 8 + 8 i; B: rows of the K step, columns past C are never stored
    int64_t arow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t r = m0 + (lane >> 3) + 8 * i;
        arow[i] = (r < n ? r : n - 1) * K;
    }
    float4 ra[4], rb[B_PER_T];
    auto fetch_mode = [&](int k0, auto am, auto bm) {
#pragma unroll
        for (int i = 0; i < 4; ++i) ra[i] = ld_quad_raw<decltype(am)::value>(A + arow[i], k0 + 4 * (lane & 7), K);
#pragma unroll
        for (int i = 0; i < B_PER_T; ++i) {
            const int f = SPLIT ? lane + 64 * i : tid;
            const int k = k0 + (f >> 3);
            rb[i] = ld_quad_raw<decltype(bm)::value>(B + (int64_t)(k < K ? k : K - 1) * C, 4 * (f & 7), C);
        }
    };
    auto fetch = [&](int k0) {
        using full = std::integral_constant<int, kFull>;
        using tail = std::integral_constant<int, kTail>;
        using narrow = std::integral_constant<int, kNarrow>;
        if (K % 4 == 0) {
            if (C % 4 == 0) fetch_mode(k0, full{}, full{});
            else if (C >= 4) fetch_mode(k0, full{}, tail{});
            else fetch_mode(k0, full{}, narrow{});
        } else if (K >= 4) {
            if (C >= 4) fetch_mode(k0, tail{}, tail{});
            else fetch_mode(k0, tail{}, narrow{});
        } else {
            if (C >= 4) fetch_mode(k0, narrow{}, tail{});
            else fetch_mode(k0, narrow{}, narrow{});
        }
    };
    const int amode = row_mode(K), bmode = row_mode(C);
    auto stash = [&](int k0) {
        if (amode != kFull || k0 + KS > K)
#pragma unroll
            for (int i = 0; i < 4; ++i) ra[i] = fix_quad(amode, ra[i], k0 + 4 * (lane & 7), K);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float* d = Aw + ((lane >> 3) + 8 * i) * LDA + 4 * (lane & 7);
            d[0] = ra[i].x; d[1] = ra[i].y; d[2] = ra[i].z; d[3] = ra[i].w;
        }
#pragma unroll
        for (int i = 0; i < B_PER_T; ++i) {
            const int f = SPLIT ? lane + 64 * i : tid;
            float4 b = fix_quad(bmode, rb[i], 4 * (f & 7), C);
            if (k0 + (f >> 3) >= K) b = make_float4(0.f, 0.f, 0.f, 0.f);       // (as A: zero times infinity is no zero)
            *reinterpret_cast<float4*>(Bw + (f >> 3) * LDB + 4 * (f & 7)) = b;
        }
    };
    // SPLIT: wavefront w takes the K steps w, w + 4, ...; a step past the end is all zeros
    const int nk = (K + KS - 1) / KS;
    const int stride = SPLIT ? 4 : 1, trips = SPLIT ? (nk + 3) / 4 : nk;
    int ks = SPLIT ? wave : 0;
    fetch(ks * KS);
    for (int kt = 0; kt < trips; ++kt) {
        __syncthreads();
        stash(ks * KS);
        __syncthreads();
        ks += stride;
        if (kt + 1 < trips) fetch(ks * KS);
#pragma unroll
        for (int kk = 0; kk < KS; kk += 2) {
            const float a = Aw[li * LDA + kk + lk];
            const float b = Bw[(kk + lk) * LDB + li];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
        }
    }
    auto store = [&](int row_in_tile, float v) {
        const int64_t row = m0 + row_in_tile;
        if (row < n && li < C) {
            if constexpr (EPI == 1) v = nu * (Zl[row * C + li] - fmaxf(Tl[row * C + li], 0.f)) + v;
            if constexpr (EPI == 3) relu_out[row * C + li] = fmaxf(v, 0.f);
            if (EPI != 3 || out) out[row * C + li] = v;
        }
    };
    if constexpr (SPLIT == 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) store(8 * (r >> 2) + 4 * lk + (r & 3), acc[r]);
    } else {
        static_assert(4 * 16 * 64 <= 4 * A_TILE, "the four partial tiles must fit the operand buffer");
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) As[(wave * 16 + r) * 64 + lane] = acc[r];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {                        // wavefront w finishes accumulator registers 4 w .. 4 w + 3
            const int r = 4 * wave + q;
            float v = As[r * 64 + lane];
            for (int w = 1; w < 4; ++w) v += As[(w * 16 + r) * 64 + lane];
            store(8 * (r >> 2) + 4 * lk + (r & 3), v);
        }
    }
}

// The same product out[n x C] = A[n x K] B[K x C] on the bf16 matrix cores, fp32-exact in its inputs: an fp32 number is the
// exact sum of three bf16 numbers (8 + 8 + 8 significand bits, each part the truncated remainder of the one before), and of the
// nine cross products the six largest are accumulated in fp32 (hi*hi, hi*mid, mid*hi, mid*mid, hi*lo, lo*hi; the three
// that are left out are below 2^-24 of |a||b|).  Six v_mfma_f32_32x32x16_bf16 per 16 columns of K replace 32
// v_mfma_f32_32x32x2_f32, at a sixteenth of the cycles per flop.  Operand layout of 32x32x16 (64 lanes): a lane holds
// A[i = lane%32][k = 8*(lane/32) .. +7] and B[k = 8*(lane/32) .. +7][j = lane%32]; the accumulator as for 32x32x2.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int intx4 __attribute__((ext_vector_type(4)));        // eight bf16 carried as plain bits

// two fp32 numbers -> their three bf16 parts, each pair packed into one dword (low half = first number)
__device__ __forceinline__ void split3_pair(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
    const unsigned u0 = __float_as_uint(x0), u1 = __float_as_uint(x1);
    h = __builtin_amdgcn_perm(u1, u0, 0x07060302u);             // upper halves of u1 and u0
    const float r0 = x0 - __uint_as_float(u0 & 0xFFFF0000u);    // exact
    const float r1 = x1 - __uint_as_float(u1 & 0xFFFF0000u);
    const unsigned v0 = __float_as_uint(r0), v1 = __float_as_uint(r1);
    m = __builtin_amdgcn_perm(v1, v0, 0x07060302u);
    const float s0 = r0 - __uint_as_float(v0 & 0xFFFF0000u);    // exact, at most 8 significant bits left
    const float s1 = r1 - __uint_as_float(v1 & 0xFFFF0000u);
    l = __builtin_amdgcn_perm(__float_as_uint(s1), __float_as_uint(s0), 0x07060302u);
}

// The six products of one K step, smallest terms first, for T x T accumulators per wavefront; As / Bs: three planes of
// 64 T rows (columns of B) by 16 k.
template <int T, int LDH>
__device__ __forceinline__ void multiply_split(floatx16 (&acc)[T][T], const unsigned short* As, const unsigned short* Bs,
                                               int a_row, int b_row, int lk) {
    constexpr int PLANE = 64 * T * LDH;
    bf16x8 a[3][T];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < T; ++i)
            a[p][i] = *reinterpret_cast<const bf16x8*>(As + p * PLANE + (a_row + i * 32) * LDH + 8 * lk);
#pragma unroll
    for (int j = 0; j < T; ++j) {
        bf16x8 b[3];                             // one column tile's parts at a time keeps the register count down
#pragma unroll
        for (int p = 0; p < 3; ++p)
            b[p] = *reinterpret_cast<const bf16x8*>(Bs + p * PLANE + (b_row + j * 32) * LDH + 8 * lk);
#pragma unroll
        for (int i = 0; i < T; ++i) {
            floatx16 c = acc[i][j];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2][i], b[0], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][i], b[2], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1][i], b[1], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1][i], b[0], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][i], b[1], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][i], b[0], c, 0, 0, 0);
            acc[i][j] = c;
        }
    }
}
// NE consecutive k of one tile row, split and stored into the three planes at element o (NE = 4 or 8)
template <int NE>
__device__ __forceinline__ void stash_split(unsigned short* S, int plane, int o, const float (&x)[NE]) {
    unsigned h[NE / 2], m[NE / 2], l[NE / 2];
#pragma unroll
    for (int e = 0; e < NE / 2; ++e) split3_pair(x[2 * e], x[2 * e + 1], h[e], m[e], l[e]);
    if constexpr (NE == 8) {
        *reinterpret_cast<uint4*>(S + o) = make_uint4(h[0], h[1], h[2], h[3]);
        *reinterpret_cast<uint4*>(S + plane + o) = make_uint4(m[0], m[1], m[2], m[3]);
        *reinterpret_cast<uint4*>(S + 2 * plane + o) = make_uint4(l[0], l[1], l[2], l[3]);
    } else {
        *reinterpret_cast<uint2*>(S + o) = make_uint2(h[0], h[1]);
        *reinterpret_cast<uint2*>(S + plane + o) = make_uint2(m[0], m[1]);
        *reinterpret_cast<uint2*>(S + 2 * plane + o) = make_uint2(l[0], l[1]);
    }
}

// T: 32 x 32 accumulators per wavefront and direction; the workgroup's tile is 64 T x 64 T.  PF: K steps fetched ahead.
// T = 2, PF = 1 for many tiles (four wavefronts per SIMD are asked for: the few registers that spill cost less than the
// fourth wavefront gains, and a second step in flight costs more occupancy than the latency it hides).  T = 1, PF = 4
// where 128 x 128 tiles would not give every compute unit two: a workgroup is then alone on its compute unit and waits
// for memory once per step.
// The vector ALU is the scarce unit here (the split of both operands): every address is a uniform base, advanced by
// scalar instructions, plus an offset that a thread computes once.
template <int EPI, int T, int PF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(T == 2 ? 4 : 1, T == 2 ? 4 : 8))) void gemm_nn_split_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ out, int64_t n, int K, int C,
    const float* __restrict__ Zl, const float* __restrict__ Tl, float nu, float* __restrict__ Tio, const Unit* unit,
    double* __restrict__ partials, const int32_t* __restrict__ gate) {
    if ((EPI == 0 || (T == 2 && EPI != 3)) && gate && *gate == 0) return;
    if constexpr (EPI == 0) {
        // gated plain product, as in gemm_nn_kernel
        if (unit != nullptr && (!unit->spec || unit->skip || (unit->done && unit->step == unit->step0))) return;
    }
    constexpr int BT = 64 * T;                    // rows and columns of the tile
    constexpr int LDH = BK + 8;                   // bf16 per tile row: rows start 16-byte aligned
    constexpr int PLANE = BT * LDH;
    constexpr int NB = 4 * T;                     // k per thread of the B tile
    constexpr int kSlab = 32 * (BT + 4) * 4;      // bytes of the result slab, which reuses the operand buffer
    constexpr int kBytes = 6 * PLANE * 2 > kSlab ? 6 * PLANE * 2 : kSlab;
    __shared__ __align__(16) unsigned short smem[kBytes / 2];
    unsigned short* const As = smem;              // [3][BT][LDH]: A tile, k contiguous per row
    unsigned short* const Bs = smem + 3 * PLANE;  // [3][BT][LDH]: B tile transposed, k contiguous per column
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, lk = lane >> 5;
    const int ctiles = (C + BT - 1) / BT;
    int64_t mtile;
    int ctile;
    xcd_group(blockIdx.x, gridDim.x, (unsigned)ctiles, mtile, ctile);
    const int64_t m0 = mtile * BT;
    const int c0 = ctile * BT;

    floatx16 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // A: thread takes 4 consecutive k of T rows; B: NB consecutive k of one column (coalesced across the columns).  Rows
    // past n and columns past C repeat the last one: their results are never stored.
    const float* const At = A + m0 * K;
    const int rows = (int)(n - m0 < BT ? n - m0 : BT);
    int aoff[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int r = (tid >> 2) + 64 * i;
        aoff[i] = (r < rows ? r : rows - 1) * K + 4 * (tid & 3);
    }
    const int bc = tid & (BT - 1);
    const int bkg = __builtin_amdgcn_readfirstlane(tid / BT);
    const int boff = c0 + bc < C ? c0 + bc : C - 1;
    float ra[PF][T][4], rb[PF][NB];
    auto fetch = [&](int s, int k0) {
        if (k0 + BK <= K) {
#pragma unroll
            for (int i = 0; i < T; ++i) {
                const float4u q = *reinterpret_cast<const float4u*>(At + k0 + aoff[i]);
                ra[s][i][0] = q.x; ra[s][i][1] = q.y; ra[s][i][2] = q.z; ra[s][i][3] = q.w;
            }
#pragma unroll
            for (int e = 0; e < NB; ++e) rb[s][e] = (B + (int64_t)(k0 + NB * bkg + e) * C)[boff];
        } else {                                  // the last, partial step: A is zero past K, B repeats its last row
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = k0 + 4 * (tid & 3) + e;
                    const float v = At[aoff[i] - 4 * (tid & 3) + (k < K ? k : K - 1)];
                    ra[s][i][e] = k < K ? v : 0.f;
                }
#pragma unroll
            for (int e = 0; e < NB; ++e) {
                const int k = k0 + NB * bkg + e;
                rb[s][e] = (B + (int64_t)(k < K ? k : K - 1) * C)[boff];
            }
        }
    };
    int nk = (K + BK - 1) / BK;
    if constexpr (EPI == 2 || EPI == 4) {
        if (unit->skip) {                         // as in gemm_nn_kernel
            if (EPI == 2) return;
            nk = 0;
        }
    }
#pragma unroll
    for (int s = 0; s < PF; ++s)
        if (s < nk) fetch(s, s * BK);
    for (int kt0 = 0; kt0 < nk; kt0 += PF) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            const int kt = kt0 + s;
            if (PF > 1 && kt >= nk) break;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < T; ++i) stash_split<4>(As, PLANE, ((tid >> 2) + 64 * i) * LDH + 4 * (tid & 3), ra[s][i]);
            stash_split<NB>(Bs, PLANE, bc * LDH + NB * bkg, rb[s]);
            __syncthreads();
            if (kt + PF < nk) fetch(s, (kt + PF) * BK);
            multiply_split<T, LDH>(acc, As, Bs, wm * 32 * T + li, wn * 32 * T + li, lk);
        }
    }
    tile_epilogue<EPI, T>(acc, reinterpret_cast<float*>(smem), m0, c0, n, C, out, Zl, Tl, nu, Tio, unit, partials);
}

// ------------------------------------------------------------------------------------------------ NN, pairs of fp16
// The same product with half the matrix instructions: an operand scaled by a power of two so that its largest entry lies in
// [2^14, 2^15) is the sum of two fp16 numbers, x = hi + lo, hi = fp16(x) and lo = fp16(x - hi) rounded to nearest, to 2^-24 of
// itself or 2^-25, whichever is more, and hi*hi, hi*lo and lo*hi are accumulated in fp32; lo*lo is below 2^-24 of |a||b|.  A row of A
// has a scale of its own (from RowRange, left by whatever formed A), so has a column of B; results are scaled back by ldexp.
// Entries far below the largest of their row or column are not held to 24 bits of themselves.  That is of no account where enough
// of a row's largest entries meet large ones of the column, and a tile of results is formed on pairs only if that is certain for
// each of them, by counting alone: if of the n entries of a row that are not zero l are near the largest, and of a column s are not
// near its largest (zeros among them), at least l - s products have two near factors.  Near: at least 2^-6 (2^-7 in a column) of the
// power of two in the largest, scaled 2^8 and 2^7.  With l - s >= n / 16 the sum |a||b| is at least n / 16 * 2^15, what the 2^-25
// add up to at most 2 n 2^15 2^-25, and a result is within 3 * 2^-24 + 2^-20 of |a||b|, usually a tenth of that and less.  A tile for
// which the counts do not say so (features of some columns 1e6 times the others', one-hot weights, rows with few entries) is formed
// from bf16 triples like the products of gemm_nn_split_kernel, to the bit.
// What bounds wide products is the power the matrix instructions take (the chip runs them at 1.55 to 1.65 GHz, by GRBM_GUI_ACTIVE over
// time), and the fp32 roundings are half as many: against 64 bits the error of 512-long sums is 2.6e-7 of the result where the
// three-way split of bf16 has 3.5e-7 (Gaussian operands; at 16 it would be 1.2 times, from 64 on it is 0.75 to 0.95 times that of the
// bf16 split, also for positive ones and for rows and columns scaled by 1e-8 to 1e8).
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

// two fp32 numbers times s -> their two fp16 parts, each pair packed into one dword (low half = first number)
__device__ __forceinline__ void split2_pair(float x0, float x1, float s, unsigned& h, unsigned& l) {
    const float2v y = {x0 * s, x1 * s};
    const half2v hi = __builtin_convertvector(y, half2v);
    const float2v r = {fmaf(x0, s, -(float)hi.x), fmaf(x1, s, -(float)hi.y)};             // exact
    h = __builtin_bit_cast(unsigned, hi);
    l = __builtin_bit_cast(unsigned, __builtin_convertvector(r, half2v));
}
// The scale of numbers of largest magnitude m is 2^(141 - e) with the exponent field e of m (15 and more, so that it is a number).
__device__ __forceinline__ int pair_exponent(float m) {
    const int e = (int)(__float_as_uint(m) >> 23) & 255;
    return (e < 15 ? 15 : e) - 141;                              // what results are scaled back by
}
__device__ __forceinline__ float pair_scale(int back) { return __uint_as_float((unsigned)(127 - back) << 23); }

constexpr int kPairK = 32;                                       // contraction per step
constexpr int kPairTM = 4, kPairTN = 2;                          // 32 x 32 accumulators of a wavefront: 128 x 64
constexpr int kPairWaves = 4;                                    // side by side
constexpr int kPairRows = 32 * kPairTM, kPairCols = 32 * kPairTN * kPairWaves;
constexpr int kPairLeast = 129;                                  // columns: half a tile and less go by other kernels
constexpr int kPairSub = 2 * 2 * 512;                            // fp16 of 32 rows (columns of B) and one step: 16-k halves, parts, lanes of eight
constexpr int kTripleSub = 2 * 3 * 512;                          // bf16 likewise
// Near entries (range_word): of a column; of a wavefront's 64 columns of a result row, which are parts of a tile's, as tiles are of
// the row's.  In all a row's are within 3 + 1 + 2 binades, as those of an aggregation's tile are within 4 + 2.
constexpr int kNearColumn = 7, kNearSlab = 3, kSlabBinades = 1, kTileBinades = 2;
constexpr int kUnlike = -(1 << 30);                              // reach of a row that is not for pairs

// B (K x C) in the matrix cores' own operand layout, [32 columns][step][16-k half][part][lane][8], zeros past K, and what the
// columns' results are scaled back by; behind the C of them, how many entries of a column are not near its largest.  A workgroup
// takes 32 columns; entries are read twice, the second time from the L2.
__global__ __launch_bounds__(1024) void pair_weights_kernel(const float* __restrict__ B, int K, int C, unsigned short* __restrict__ planes,
                                                            int* __restrict__ columns, const int32_t* __restrict__ gate) {
    __shared__ float s_max[32][32];
    __shared__ int s_small[32][32];
    __shared__ float s_top[32];
    if (gate && *gate == 0) return;
    const int li = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int c = blockIdx.x * 32 + li;
    const float* const col = B + (c < C ? c : C - 1);
    auto load8 = [&](int k0, float (&x)[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v = col[(int64_t)(k0 + e < K ? k0 + e : K - 1) * C];
            x[e] = k0 + e < K ? v : 0.f;
        }
    };
    float m = 0.f;
    for (int k0 = 8 * g; k0 < K; k0 += 256) {
        float x[8];
        load8(k0, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(x[e]));
    }
    s_max[g][li] = m;
    __syncthreads();
    if (g == 0) {
        for (int i = 1; i < 32; ++i) m = fmaxf(m, s_max[i][li]);
        s_top[li] = m;
        if (c < C) columns[c] = pair_exponent(m);
    }
    __syncthreads();
    m = s_top[li];
    const float s = pair_scale(pair_exponent(m)), near = range_near(m, kNearColumn);
    int small = 0;
    const int steps = (K + kPairK - 1) / kPairK;
    for (int k0 = 8 * g; k0 < steps * kPairK; k0 += 256) {
        float x[8];
        load8(k0, x);
        uint4v h, l;
#pragma unroll
        for (int e = 0; e < 8; ++e) small += k0 + e < K && fabsf(x[e]) < near ? 1 : 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            unsigned a, b;
            split2_pair(x[2 * e], x[2 * e + 1], s, a, b);
            h[e] = a;
            l[e] = b;
        }
        unsigned short* const o = planes + ((int64_t)blockIdx.x * steps + k0 / kPairK) * kPairSub + (k0 & 16 ? 1024 : 0) +
                                  ((k0 & 8 ? 32 : 0) + li) * 8;
        *reinterpret_cast<uint4v*>(o) = h;
        *reinterpret_cast<uint4v*>(o + 512) = l;
    }
    s_small[g][li] = small;
    __syncthreads();
    if (g == 0 && c < C) {
        for (int i = 1; i < 32; ++i) small += s_small[i][li];
        // nothing but zeros asks for nothing; a largest entry that cannot be scaled to 2^14 (or is no number) for more than there is
        const uint32_t e = magnitude_exponent(m);
        columns[C + c] = m == 0.f ? kUnlike : e < 15 || e == 255 ? K + 1 : small;
    }
}

// A wavefront's 128 x 64 results, 32 rows at a time through a slab of LDS of its own (no barrier) so that every global access
// is a 16-byte piece of 256 consecutive bytes.  EPI as in tile_epilogue.  s_rs / s_rm: EPI 1, where this wavefront's share of its
// rows' sums and its RowRange words go (null: nobody asks).
constexpr int kPairLd = 64 + 4;
template <int EPI, int MODE>
__device__ __forceinline__ void pair_epilogue(floatx16 (&acc)[kPairTM][kPairTN], float* Cs, const int* s_back, const int (&cb)[kPairTN],
                                              int64_t m0, int c0, int64_t n, int C, const EpilogueArgs& args, double& dsum,
                                              double* s_rs, uint32_t* s_rm) {
    const int lane = threadIdx.x & 63;
    const int li = lane & 31, lk = lane >> 5;
    const int c = c0 + 4 * (lane & 15);
    constexpr int U = 4;                                 // pieces of a lane at a time, their loads before any is used
#pragma unroll
    for (int q = 0; q < kPairTM; ++q) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int4 rb = *reinterpret_cast<const int4*>(s_back + 32 * q + 8 * r4 + 4 * lk);
            const int b[4] = {rb.x, rb.y, rb.z, rb.w};
#pragma unroll
            for (int j = 0; j < kPairTN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    Cs[(8 * r4 + 4 * lk + e) * kPairLd + j * 32 + li] = ldexpf(acc[q][j][4 * r4 + e], b[e] + cb[j]);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u0 = 0; u0 < 8; u0 += U) {
            float4 z4[U], t4[U];
            if constexpr (EPI == 1 || EPI == 2 || EPI == 4) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t row = m0 + 32 * q + 4 * (u0 + u) + (lane >> 4);
                    const int64_t ro = (row < n ? row : n - 1) * (int64_t)C;
                    z4[u] = ld_quad<MODE>(args.Zl + ro, c, C);
                    t4[u] = ld_quad<MODE>(args.tin + ro, c, C);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int rl = 4 * (u0 + u) + (lane >> 4);
                const int64_t row = m0 + 32 * q + rl;
                const float4 v4 = *reinterpret_cast<const float4*>(Cs + rl * kPairLd + 4 * (lane & 15));
                float v[4] = {v4.x, v4.y, v4.z, v4.w};
                if constexpr (EPI == 1) {
                    if (s_rs) {                          // (uniform)
                        double rs[3];
                        quad_row_sums<16>(rs, v, z4[u], t4[u], c, C, args.nu);
                        const int p = lane & 15;
                        if (p < 3) s_rs[(32 * q + rl) * 3 + p] = p == 0 ? rs[0] : p == 1 ? rs[1] : rs[2];
                    }
                }
                const bool in = row < n && c < C;
                if (in) epilogue_quad<EPI, MODE>(v, z4[u], t4[u], row * C + c, MODE == kFull ? 4 : C - c, args, dsum);
                if constexpr (EPI == 1) {
                    if (s_rm) {
                        float m = in ? fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))) : 0.f;
                        m = __int_as_float(over_lanes<16>(__float_as_int(m), [](int a, int b) { return max(a, b); }));       // (as whole numbers)
                        const float t = range_near(m, kNearSlab);
                        int n = 0;
#pragma unroll
                        for (int e = 0; e < 4; ++e) n += in && c + e < C ? (fabsf(v[e]) >= t ? 1 : 0) + (v[e] != 0.f ? 1 << 16 : 0) : 0;
                        n = over_lanes<16>(n, [](int a, int b) { return a + b; });
                        if ((lane & 15) == 0) s_rm[32 * q + rl] = range_word_of(m, n);
                    }
                }
            }
        }
    }
}

// A workgroup forms 128 rows by 256 columns.  A is split on its way to LDS (three buffers, so that a step's first
// operands are read before the barrier that starts it); B comes from the L2 straight into registers, in operand layout
// (pair_weights_kernel), a half step ahead: no wavefront reads what another does.  Two workgroups of four wavefronts share a
// compute unit, one's epilogue beside the other's products.  Against one workgroup of 256 x 256, both operands in LDS, the large
// product is as fast and the mid-sized one is not cut into three rounds and a bit: us for 500000 x 512 x 512 and 200000 x 256
// x 256, bf16 split 1590 and 182, 256 x 256 946 and 195, 128 x 128 1090 and 186, this one 950 and 122.  The counts of RowRange cost
// them 1 % (its words read, a barrier that is there anyway), 4 % where the result's are left too; tiles on triples take as long as
// those of the bf16 kernel (500000 x 512 x 512 with epilogue 4, all of them 1830 us, the bf16 kernel 1795, on pairs 1210).
template <int EPI>
__global__ __launch_bounds__(64 * kPairWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_nn_pair_kernel(
    const float* __restrict__ A, const float* __restrict__ B, const unsigned short* __restrict__ planes, const int* __restrict__ columns,
    const uint32_t* __restrict__ row_range, int range_tiles, float* __restrict__ out, int64_t n, int K, int C,
    const float* __restrict__ Zl, const float* __restrict__ Tl, float nu, float* __restrict__ Tio, const Unit* unit,
    double* __restrict__ partials, uint32_t* __restrict__ out_range, const int32_t* __restrict__ gate) {
    if (EPI != 3 && gate && *gate == 0) return;
    if constexpr (EPI == 0) {
        // gated plain product, as in gemm_nn_kernel
        if (unit != nullptr && (!unit->spec || unit->skip || (unit->done && unit->step == unit->step0))) return;
    }
    constexpr int WN = kPairWaves, NT = 64 * WN;
    constexpr int AP = kPairRows * 4 / NT;               // pieces of eight k per thread and step
    constexpr int BUF = kPairTM * kPairSub;
    constexpr int kSlabs = WN * 32 * kPairLd * 4;        // bytes: the wavefronts' slabs, then (EPI 1) their rows' sums and words
    constexpr int kSums = WN * kPairRows * 3 * 8, kWords = WN * kPairRows * 4;
    static_assert(kSlabs + kSums + kWords <= 3 * BUF * 2, "the epilogue's share must fit the operand buffers");
    __shared__ __align__(16) unsigned short smem[3 * BUF];
    __shared__ __align__(16) int s_back[kPairRows];
    __shared__ __align__(16) int s_reach[NT / 16], s_small[NT / 16];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lk = lane >> 5;
    const int ctiles = (C + kPairCols - 1) / kPairCols;
    int64_t mtile;
    int ctile;
    xcd_group(blockIdx.x, gridDim.x, (unsigned)ctiles, mtile, ctile);
    const int64_t m0 = mtile * kPairRows;
    const int c0 = ctile * kPairCols + 64 * wave;          // this wavefront's columns
    int steps = (K + kPairK - 1) / kPairK;
    if constexpr (EPI == 2 || EPI == 4) {
        if (unit->skip) {                                // as in gemm_nn_kernel
            if (EPI == 2) return;
            steps = 0;
        }
    }

    // piece: eight k of a row, four pieces per row; rows past n repeat the last one, their results are never stored.  In LDS a
    // piece is the 16 bytes of one lane in operand layout, lanes exchanged so that eight pieces written at once hit different banks.
    const float* const At = A + m0 * K;
    const int rows = (int)(n - m0 < kPairRows ? n - m0 : kPairRows);
    int aoff[AP], aw[AP];
    float scale[AP];
    int reach = -kUnlike;                                // the least of the tile's rows, as far as this thread knows
#pragma unroll
    for (int i = 0; i < AP; ++i) {
        const int r = (tid + NT * i) >> 2, p = tid & 3, rr = r < rows ? r : rows - 1;
        // the four threads of a row share its tiles; sixteen of them and less are read once
        const uint32_t* const words = row_range + m0 + rr;
        uint32_t word[4];
        int top = 0, near = 0;
        auto load = [&](int t0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) word[u] = t0 + 4 * u < range_tiles ? words[(int64_t)(t0 + 4 * u) * n] : 0u;
        };
        for (int t0 = p; t0 < range_tiles + p; t0 += 16) {
            load(t0);
#pragma unroll
            for (int u = 0; u < 4; ++u) top = max(top, (int)range_exponent(word[u]));
        }
        top = over_lanes<4>(top, [](int a, int b) { return max(a, b); });
        for (int t0 = p; t0 < range_tiles + p; t0 += 16) {
            if (range_tiles > 16) load(t0);
#pragma unroll
            for (int u = 0; u < 4; ++u) near += range_share(word[u], (uint32_t)top, kTileBinades, 16);
        }
        near = over_lanes<4>(near, [](int a, int b) { return a + b; });
        if (top != 0) reach = min(reach, top < 15 || top == 255 ? kUnlike + 1 : near);
        const int back = max(top, 15) - 141;
        scale[i] = pair_scale(back);
        if (p == 0) s_back[r] = back;
        aoff[i] = rr * K + 8 * p;
        aw[i] = (r >> 5) * kPairSub + (p >> 1) * 1024 + ((p & 1) * 32 + ((r & 31) ^ (p << 2))) * 8;
    }
    int small = ctile * kPairCols + tid < C ? columns[C + ctile * kPairCols + tid] : kUnlike;        // the most of the tile's columns
    static_assert(NT == kPairCols, "a thread per column");
    reach = over_lanes<16>(reach, [](int a, int b) { return min(a, b); });
    small = over_lanes<16>(small, [](int a, int b) { return max(a, b); });
    if ((lane & 15) == 0) {
        s_reach[tid >> 4] = reach;
        s_small[tid >> 4] = small;
    }
    const int nsub = (C + 31) / 32;
    const half8* Bw[kPairTN];
#pragma unroll
    for (int j = 0; j < kPairTN; ++j) {
        const int sub = c0 / 32 + j < nsub ? c0 / 32 + j : nsub - 1;         // (columns past C: never stored)
        Bw[j] = reinterpret_cast<const half8*>(planes + (int64_t)sub * ((K + kPairK - 1) / kPairK) * kPairSub) + lane;
    }

    floatx16 acc[kPairTM][kPairTN];
#pragma unroll
    for (int i = 0; i < kPairTM; ++i)
#pragma unroll
        for (int j = 0; j < kPairTN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    float4u ra[AP][2];
    auto fetch = [&](int kt, int i) {
        const float* const p = At + kt * kPairK + aoff[i];
        if (kt * kPairK + kPairK <= K) {
            ra[i][0] = *reinterpret_cast<const float4u*>(p);
            ra[i][1] = *reinterpret_cast<const float4u*>(p + 4);
        } else {                                         // the last, partial step: zeros past K
            const int left = K - kt * kPairK - 8 * (tid & 3);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = p[e < left ? e : left - 1];
                ra[i][e >> 2][e & 3] = e < left ? v : 0.f;
            }
        }
    };
    auto stash = [&](unsigned short* D, int i) {
        uint4v h, l;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            unsigned a, b;
            split2_pair(ra[i][e >> 1][2 * (e & 1)], ra[i][e >> 1][2 * (e & 1) + 1], scale[i], a, b);
            h[e] = a;
            l[e] = b;
        }
        *reinterpret_cast<uint4v*>(D + aw[i]) = h;
        *reinterpret_cast<uint4v*>(D + aw[i] + 512) = l;
    };
    half8 b[2][kPairTN][2], a[2][2];
    auto load_b = [&](int half) {                        // both parts of this wavefront's columns, 16-k half `half` of the contraction
        const int h = half < 2 * steps ? half : 2 * steps - 1;
#pragma unroll
        for (int j = 0; j < kPairTN; ++j)
#pragma unroll
            for (int p = 0; p < 2; ++p) b[half & 1][j][p] = Bw[j][h * 128 + 64 * p];
    };
    // lane's operand of rows 32 i .., half kc: piece 2 kc + lk, lanes exchanged as they were written
    const int ar0 = (lk * 32 + (li ^ (lk << 2))) * 8, ar1 = 1024 + (lk * 32 + (li ^ ((2 + lk) << 2))) * 8;
    auto load_a = [&](int w, const unsigned short* S, int kc, int i) {
        const unsigned short* const p = S + i * kPairSub + (kc ? ar1 : ar0);
        a[w][0] = *reinterpret_cast<const half8*>(p);
        a[w][1] = *reinterpret_cast<const half8*>(p + 512);
    };
    unsigned short *S0 = smem, *S1 = smem + BUF, *S2 = smem + 2 * BUF;       // this step's tile, the next one's, and where the one after goes
    // STASH, FETCH: whether there are a step after the next and one after that
    auto step = [&](int kt, auto STASH, auto FETCH) {
        __syncthreads();
        constexpr int SUBS = 2 * kPairTM;
#pragma unroll
        for (int st = 0; st < SUBS; ++st) {
            const int kc = st / kPairTM, i = st % kPairTM, w = st & 1;
            if (st + 1 < SUBS) load_a(w ^ 1, S0, (st + 1) / kPairTM, (st + 1) % kPairTM);
            else load_a(w ^ 1, S1, 0, 0);                // (behind the last step: read and not used)
            if (i == 0) load_b(2 * kt + kc + 1);
#pragma unroll
            for (int t = 0; t < 3; ++t)                  // smallest terms first
#pragma unroll
                for (int j = 0; j < kPairTN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[w][t == 0 ? 1 : 0], b[kc][j][t == 1 ? 1 : 0], acc[i][j], 0, 0, 0);
            if constexpr (decltype(STASH)::value) {
                if (st < AP) {
                    stash(S2, st);
                    if constexpr (decltype(FETCH)::value) fetch(kt + 3, st);
                }
            }
            // the operands' reads first, then the split between the matrix instructions
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
            for (int u = 0; u < 3 * kPairTN; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        unsigned short* const t = S0;
        S0 = S1;
        S1 = S2;
        S2 = t;
    };
    using yes = std::true_type;
    using no = std::false_type;
    // The tile from bf16 triples: two buffers of A, one barrier per step, B straight from the matrix.  (Nobody reads the pairs that the
    // buffers hold.)
    auto triples = [&] {
        int boff[kPairTN];
#pragma unroll
        for (int j = 0; j < kPairTN; ++j) boff[j] = 8 * lk * C + (c0 + 32 * j + li < C ? c0 + 32 * j + li : C - 1);
        auto stash3 = [&](unsigned short* D, int i) {
            const int r = (tid + NT * i) >> 2, p = tid & 3;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = ra[i][e >> 2][e & 3];
            stash_split<8>(D, 512, (r >> 5) * kTripleSub + (p >> 1) * 1536 + ((p & 1) * 32 + ((r & 31) ^ (p << 2))) * 8, x);
        };
        float rb[kPairTN][8];
        auto fetch_b = [&](int half, int j) {
            const float* const p = B + (int64_t)half * 16 * C;
            if (half * 16 + 16 <= K) {
#pragma unroll
                for (int e = 0; e < 8; ++e) rb[j][e] = (p + (int64_t)e * C)[boff[j]];
            } else {                                     // past K: the last row again, A is zero there
                const int left = K - half * 16 - 8 * lk;
#pragma unroll
                for (int e = 0; e < 8; ++e) rb[j][e] = p[boff[j] + (int64_t)(e < left ? e : left - 1) * C];
            }
        };
        if (tid < kPairRows) s_back[tid] = 0;
#pragma unroll
        for (int i = 0; i < AP; ++i) fetch(0, i);
#pragma unroll
        for (int j = 0; j < kPairTN; ++j) fetch_b(0, j);
#pragma unroll
        for (int i = 0; i < AP; ++i) stash3(smem, i);
        if (steps > 1)
#pragma unroll
            for (int i = 0; i < AP; ++i) fetch(1, i);
#pragma unroll 1
        for (int kt = 0; kt < steps; ++kt) {
            const unsigned short* const S = smem + (kt & 1) * kPairTM * kTripleSub;
            unsigned short* const D = smem + (~kt & 1) * kPairTM * kTripleSub;
            __syncthreads();
            if (kt + 1 < steps) {
#pragma unroll
                for (int i = 0; i < AP; ++i) stash3(D, i);
                if (kt + 2 < steps)
#pragma unroll
                    for (int i = 0; i < AP; ++i) fetch(kt + 2, i);
            }
#pragma unroll 1
            for (int kc = 0; kc < 2; ++kc) {
                const unsigned short* const p0 = S + kc * 1536 + (lk * 32 + (li ^ ((2 * kc + lk) << 2))) * 8;
#pragma unroll
                for (int j = 0; j < kPairTN; ++j) {      // (a column tile's parts at a time, A's read once for each: nothing spills)
                    intx4 b[3];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        unsigned h, m, l;
                        split3_pair(rb[j][2 * e], rb[j][2 * e + 1], h, m, l);
                        b[0][e] = (int)h;
                        b[1][e] = (int)m;
                        b[2][e] = (int)l;
                    }
                    fetch_b(2 * kt + kc + 1, j);
                    asm volatile("" ::: "memory");     // (A's parts are not kept from one column tile to the next)
#pragma unroll
                    for (int i0 = 0; i0 < kPairTM; i0 += 2) {
                        bf16x8 a3[2][3];
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int q = 0; q < 3; ++q) a3[i][q] = *reinterpret_cast<const bf16x8*>(p0 + (i0 + i) * kTripleSub + 512 * q);
                        constexpr int P[6] = {2, 0, 1, 1, 0, 0}, Q[6] = {0, 2, 1, 0, 1, 0};          // smallest terms first
#pragma unroll
                        for (int t = 0; t < 6; ++t)
#pragma unroll
                            for (int i = 0; i < 2; ++i)
                                acc[i0 + i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a3[i][P[t]], __builtin_bit_cast(bf16x8, b[Q[t]]), acc[i0 + i][j], 0, 0, 0);
                    }
                }
            }
        }
    };
    bool on_pairs = true;
    static_assert(2 * kPairTM * kTripleSub <= 3 * BUF, "two buffers of triples in the three of pairs");
    if (steps > 0) {
        load_b(0);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            if (p >= steps) break;
#pragma unroll
            for (int i = 0; i < AP; ++i) fetch(p, i);
            if (p < 2)
#pragma unroll
                for (int i = 0; i < AP; ++i) stash(smem + p * BUF, i);
        }
        __syncthreads();
        static_assert(NT == 256, "a lane per sixteen threads");
        on_pairs = __builtin_amdgcn_readfirstlane(over_lanes<16>(s_reach[lane & 15], [](int a, int b) { return min(a, b); }) >=
                                                  over_lanes<16>(s_small[lane & 15], [](int a, int b) { return max(a, b); }));
        if (on_pairs) {
            load_a(0, S0, 0, 0);
            int kt = 0;
            for (; kt + 3 < steps; ++kt) step(kt, yes{}, yes{});
            if (kt + 2 < steps) step(kt++, yes{}, no{});
            for (; kt < steps; ++kt) step(kt, no{}, no{});
        } else {
            triples();
        }
    }
    __syncthreads();                                     // every wavefront is through with the operands
    float* const Cs = reinterpret_cast<float*>(smem) + wave * 32 * kPairLd;
    double* const s_sums = reinterpret_cast<double*>(reinterpret_cast<char*>(smem) + kSlabs);
    uint32_t* const s_words = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(smem) + kSlabs + kSums);
    // (epilogue 1 has no partials: the argument then carries the row sums)
    double* const row_sums = EPI == 1 ? partials : nullptr;
    int cb[kPairTN];
#pragma unroll
    for (int j = 0; j < kPairTN; ++j) cb[j] = on_pairs ? columns[c0 + 32 * j + li < C ? c0 + 32 * j + li : C - 1] : 0;
    EpilogueArgs args{out, Zl, (EPI == 2 || EPI == 4) ? Tio : Tl, nu, Tio, 0.0, false, false};
    double dsum = 0.0;
    if constexpr (EPI == 2 || EPI == 4) {
        args.hold = EPI == 4 && unit->skip != 0;
        args.inv0 = unit->skip ? 0.0 : 1.0 / unit->step0;
        args.take = unit->spec != 0 && !unit->skip;
    }
    double* const s_rs = EPI == 1 && row_sums ? s_sums + wave * kPairRows * 3 : nullptr;
    uint32_t* const s_rm = EPI == 1 && out_range ? s_words + wave * kPairRows : nullptr;
    if (C % 4 == 0) pair_epilogue<EPI, kFull>(acc, Cs, s_back, cb, m0, c0, n, C, args, dsum, s_rs, s_rm);
    else pair_epilogue<EPI, kTail>(acc, Cs, s_back, cb, m0, c0, n, C, args, dsum, s_rs, s_rm);
    if constexpr (EPI == 3) note_bad(dsum, reinterpret_cast<int32_t*>(partials));
    if constexpr (EPI == 1) {
        if (row_sums || out_range) {
            __syncthreads();
            for (int r = tid; r < kPairRows; r += NT) {
                const int64_t row = m0 + r;
                if (row >= n) break;
                const int64_t o = (int64_t)ctile * n + row;
                if (row_sums) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        double s = 0.0;
#pragma unroll
                        for (int w = 0; w < WN; ++w) s += s_sums[(w * kPairRows + r) * 3 + q];
                        row_sums[o * 3 + q] = s;
                    }
                }
                if (out_range) {
                    uint32_t top = 0;
                    int near = 0;
#pragma unroll
                    for (int w = 0; w < WN; ++w) top = max(top, range_exponent(s_words[w * kPairRows + r]));
#pragma unroll
                    for (int w = 0; w < WN; ++w) near += range_share(s_words[w * kPairRows + r], top, kSlabBinades, 4);
                    out_range[o] = top ? range_word(top, near) : 0u;
                }
            }
        }
    }
    if constexpr (EPI == 2 || EPI == 4) {
        __shared__ double red[WN];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) dsum += __shfl_down(dsum, o, 64);
        if (lane == 0) red[wave] = dsum;
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < WN; ++w) s += red[w];
            partials[blockIdx.x] = 0.5 * (double)nu * s;
        }
    }
}

// out[n x C] = g W with g = nu (Z - relu(T)) + SG W^T  (W: K1 x C, SG: n x C, C <= 16, K1 a multiple of four).
// This is (grad_Z psi) W without ever storing the gradient: an element of it is formed while its tile is loaded (C fused
// multiply-adds, the rows of W^T and the block's rows of SG from LDS), for the product and for the row sums of the search, which
// then reads neither Z nor T.  The kernel is bound by reading those two, with the vector work and the products behind it: the
// products take v_mfma_f32_16x16x4_f32 (C <= 16: a 32 x 32 instruction's second half would be zeros) and both operands from the tiles
// that the gradient is formed with, W as the columns of W^T.  2000000 x 256 x 16: 985 us with v_mfma_f32_32x32x2_f32 on [W; W^T W],
// which a launch of its own made, 833 so, 5.2 TB/s of Z, T, SG and out.
constexpr int kSgLd = kLowRankMax + 4;            // row stride of SG in LDS: the eight rows a wavefront reads at once hit different banks
template <bool GATED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void gemm_nn_gradz_kernel(const float* __restrict__ Zl, const float* __restrict__ Tl,
                                                            const float* __restrict__ SG,
                                                            const float* __restrict__ Wt, float* __restrict__ out, int64_t n,
                                                            int K1, int C, float nu, double* __restrict__ row_sums,
                                                            const int32_t* __restrict__ gate) {
    if constexpr (GATED) {
        if (*gate == 0) return;
    }
    // 32 columns of Z_l and T_l per step: every row then gives a whole 128-byte line of each matrix to one step.
    // With half lines the second half had left the L2 before its step came (twice the traffic, measured).
    constexpr int GBK = 32;
    constexpr int LD = GBK + 4;                      // 16 rows by 4 columns, a matrix instruction's operand, hit different banks
    __shared__ __align__(16) float As[BM * LD];
    __shared__ __align__(16) float s_sg[BM * kSgLd];
    __shared__ __align__(16) float s_wt[2][kLowRankMax * LD];            // the step's 32 columns of W^T, zeros past its rows and columns
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wm = tid >> 6;
    const int64_t m0 = (int64_t)blockIdx.x * BM;
    floatx4 acc[2];                                  // rows 0 .. 15 and 16 .. 31 of the wavefront's 32
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[0][r] = acc[1][r] = 0.f;
    // threads of the first two wavefronts: quad tid % 8 of row tid / 8 of the tile that starts at column k0; rows past C are zero
    const bool has_w = tid < 8 * kLowRankMax;
    float4 rw = make_float4(0.f, 0.f, 0.f, 0.f);
    auto fetch_w = [&](int k0) {
        const int k = k0 + 4 * (tid & 7);
        rw = make_float4(0.f, 0.f, 0.f, 0.f);
        if (tid >> 3 < C && k < K1) rw = *reinterpret_cast<const float4*>(Wt + (int64_t)(tid >> 3) * K1 + k);
    };
    const int wt_at = (tid >> 3) * LD + 4 * (tid & 7);
    if (has_w) {
        fetch_w(0);
        *reinterpret_cast<float4*>(s_wt[0] + wt_at) = rw;
    }
    if (C % 4 == 0) {
        for (int i = tid; i < BM * (C / 4); i += 256) {
            const int r = i / (C / 4), q = i - r * (C / 4);
            const int64_t gr = m0 + r < n ? m0 + r : n - 1;
            *reinterpret_cast<float4*>(s_sg + r * kSgLd + 4 * q) = *reinterpret_cast<const float4*>(SG + gr * C + 4 * q);
        }
    } else {
        const int q = tid & 15;
        for (int r = tid >> 4; r < BM; r += 16) {
            const int64_t gr = m0 + r < n ? m0 + r : n - 1;
            const float v = SG[gr * C + (q < C ? q : C - 1)];
            s_sg[r * kSgLd + q] = q < C ? v : 0.f;
        }
    }
    // thread: quad tid % 8 of rows tid / 8 + 32 i
    const int kq = tid & 7;
    int64_t grow[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t gr = m0 + (tid >> 3) + 32 * i;
        grow[i] = gr < n ? gr : n - 1;
    }
    double rs[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) rs[i][0] = rs[i][1] = rs[i][2] = 0.0;
    float4 rz[4], rt[4];
    auto fetch = [&](int k0) {
        const int k = k0 + 4 * kq < K1 ? k0 + 4 * kq : 0;                // (quads past K1 are not used)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rz[i] = *reinterpret_cast<const float4*>(Zl + grow[i] * K1 + k);
            rt[i] = *reinterpret_cast<const float4*>(Tl + grow[i] * K1 + k);
        }
    };
    // the gradient of the quads that were fetched, into the tile, and what the search needs of it
    auto stash = [&](int k0, const float* wt) {
        const bool own = k0 + 4 * kq < K1;
        float g[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            g[i][0] = nu * (rz[i].x - fmaxf(rt[i].x, 0.f));
            g[i][1] = nu * (rz[i].y - fmaxf(rt[i].y, 0.f));
            g[i][2] = nu * (rz[i].z - fmaxf(rt[i].z, 0.f));
            g[i][3] = nu * (rz[i].w - fmaxf(rt[i].w, 0.f));
        }
        for (int q4 = 0; q4 < C; q4 += 4) {
            float4 sg[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) sg[i] = *reinterpret_cast<const float4*>(s_sg + ((tid >> 3) + 32 * i) * kSgLd + q4);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 w = *reinterpret_cast<const float4*>(wt + (q4 + q) * LD + 4 * kq);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float f = q == 0 ? sg[i].x : q == 1 ? sg[i].y : q == 2 ? sg[i].z : sg[i].w;
                    g[i][0] = fmaf(f, w.x, g[i][0]);
                    g[i][1] = fmaf(f, w.y, g[i][1]);
                    g[i][2] = fmaf(f, w.z, g[i][2]);
                    g[i][3] = fmaf(f, w.w, g[i][3]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<float4*>(As + ((tid >> 3) + 32 * i) * LD + 4 * kq) =
                own ? make_float4(g[i][0], g[i][1], g[i][2], g[i][3]) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (!own) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float z[4] = {rz[i].x, rz[i].y, rz[i].z, rz[i].w}, t[4] = {rt[i].x, rt[i].y, rt[i].z, rt[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double zd = (double)z[e], gd = (double)g[i][e];
                rs[i][0] += (zd - fmax((double)t[e], 0.0)) * gd;
                rs[i][1] += gd * gd;
                rs[i][2] += zd * zd;
            }
        }
    };
    const int nk = (K1 + GBK - 1) / GBK;
    const int li = lane & 15, lk = lane >> 4;
    fetch(0);
    if (has_w) fetch_w(GBK);
    for (int kt = 0; kt < nk; ++kt) {
        __syncthreads();
        // the tile of W^T is stored a step before it is read: no third barrier
        if (has_w) *reinterpret_cast<float4*>(s_wt[(kt + 1) & 1] + wt_at) = rw;
        stash(kt * GBK, s_wt[kt & 1]);
        __syncthreads();
        if (kt + 1 < nk) {
            fetch((kt + 1) * GBK);
            if (has_w) fetch_w((kt + 2) * GBK);
        }
#pragma unroll
        for (int kk = 0; kk < GBK; kk += 4) {
            const float b = s_wt[kt & 1][li * LD + kk + lk];             // (results past C are not stored)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(As[(wm * 32 + 16 * t + li) * LD + kk + lk], b, acc[t], 0, 0, 0);
        }
    }
    if (li < C) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int64_t row = m0 + wm * 32 + 16 * (r >> 2) + 4 * lk + (r & 3);
            if (row < n) out[row * C + li] = acc[r >> 2][r & 3];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int o = 1; o < 8; o <<= 1)
#pragma unroll
            for (int q = 0; q < 3; ++q) rs[i][q] += __shfl_xor(rs[i][q], o, 64);
        const int64_t row = m0 + (tid >> 3) + 32 * i;
        if (kq < 3 && row < n) row_sums[row * 3 + kq] = kq == 0 ? rs[i][0] : kq == 1 ? rs[i][1] : rs[i][2];
    }
}

// ------------------------------------------------------------------------------------------------ TN
// Block (chunk, ktile, ctile): partial[chunk][k][c] = sum_{rows of chunk} A[row][k] G[row][c].
// PRO 1: the right operand is the hidden-layer pre-activation gradient nu (relu(T) - Z) 1[T > 0], formed from
// T (passed as G) and Z while the tile is loaded, so that it is never stored.
// FULL: both widths are multiples of four.
template <int BN, int PRO, int FULL>
__global__ __launch_bounds__(256) void gemm_tn_kernel(const float* __restrict__ A, const float* __restrict__ G,
                                                      const float* __restrict__ Zl, float nu,
                                                      float* __restrict__ partial, int64_t n, int K, int C,
                                                      int64_t rows_per_chunk) {
    constexpr int WN = (BN == 128) ? 2 : 1;
    constexpr int WM = 4 / WN;
    constexpr int TM = BM / (WM * 32);
    constexpr int TN = BN / (WN * 32);
    constexpr int LDA = BM + 4;
    constexpr int LDG = BN + 4;
    constexpr int G_F4 = BK * BN / 4;
    constexpr int G_PER_T = (G_F4 + 255) / 256;

    __shared__ __align__(16) float As[BK * LDA];
    __shared__ __align__(16) float Gs[BK * LDG];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int ktiles = (K + BM - 1) / BM;
    const int ctiles = (C + BN - 1) / BN;
    int tile;
    int64_t chunk;
    xcd_group(blockIdx.x, gridDim.x, (unsigned)(ktiles * ctiles), chunk, tile);
    const int k0 = (tile / ctiles) * BM;
    const int c0 = (tile % ctiles) * BN;
    const int64_t r_begin = chunk * rows_per_chunk;
    const int64_t r_end = (r_begin + rows_per_chunk < n) ? (r_begin + rows_per_chunk) : n;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    float4 ra[2], rg[G_PER_T], rz[PRO ? G_PER_T : 1];
    const int amode = FULL ? kFull : row_mode(K), gmode = FULL ? kFull : row_mode(C);
    auto fetch = [&](int64_t r0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {              // A tile: 16 rows x 128 k = 512 quads; columns past K are never stored
            const int f = tid + 256 * i;
            const int64_t gr = r0 + (f >> 5);
            ra[i] = ld_quad_raw(amode, A + (gr < r_end ? gr : r_end - 1) * K, k0 + 4 * (f & 31), K);     // rows past the chunk: see stash
        }
#pragma unroll
        for (int i = 0; i < G_PER_T; ++i) {
            const int f = tid + 256 * i;
            if (f < G_F4) {
                const int64_t gr = r0 + f / (BN / 4);
                const int64_t go = (gr < r_end ? gr : r_end - 1) * C;
                const int c = c0 + 4 * (f % (BN / 4));
                rg[i] = ld_quad_raw(gmode, G + go, c, C);
                if constexpr (PRO == 1) rz[i] = ld_quad_raw(gmode, Zl + go, c, C);
            }
        }
    };
    auto stash = [&](int64_t r0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int f = tid + 256 * i;
            float4 a = fix_quad(amode, ra[i], k0 + 4 * (f & 31), K);
            if (r0 + (f >> 5) >= r_end) a = make_float4(0.f, 0.f, 0.f, 0.f);   // both operands are zero there
            *reinterpret_cast<float4*>(As + (f >> 5) * LDA + 4 * (f & 31)) = a;
        }
#pragma unroll
        for (int i = 0; i < G_PER_T; ++i) {
            const int f = tid + 256 * i;
            if (f < G_F4) {
                const int rr = f / (BN / 4), cq = f % (BN / 4);
                float4 g = fix_quad(gmode, rg[i], c0 + 4 * cq, C);
                if constexpr (PRO == 1) {
                    const float4 z = fix_quad(gmode, rz[i], c0 + 4 * cq, C);
                    g.x = (g.x > 0.f) ? nu * (g.x - z.x) : 0.f;
                    g.y = (g.y > 0.f) ? nu * (g.y - z.y) : 0.f;
                    g.z = (g.z > 0.f) ? nu * (g.z - z.z) : 0.f;
                    g.w = (g.w > 0.f) ? nu * (g.w - z.w) : 0.f;
                }
                const bool in = r0 + rr < r_end;
                *reinterpret_cast<float4*>(Gs + rr * LDG + 4 * cq) = make_float4(in ? g.x : 0.f, in ? g.y : 0.f, in ? g.z : 0.f, in ? g.w : 0.f);
            }
        }
    };

    const int li = lane & 31, lk = lane >> 5;
    if (r_begin < r_end) fetch(r_begin);
    for (int64_t r0 = r_begin; r0 < r_end; r0 += BK) {
        __syncthreads();
        stash(r0);
        __syncthreads();
        if (r0 + BK < r_end) fetch(r0 + BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 2) {
            float a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = As[(kk + lk) * LDA + wm * TM * 32 + i * 32 + li];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = Gs[(kk + lk) * LDG + wn * TN * 32 + j * 32 + li];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
    float* dst = partial + chunk * (int64_t)K * C;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int c = c0 + wn * TN * 32 + j * 32 + li;
            if (c >= C) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = k0 + wm * TM * 32 + i * 32 + 8 * (r >> 2) + 4 * lk + (r & 3);
                if (k < K) dst[(int64_t)k * C + c] = acc[i][j][r];
            }
        }
}

// gemm_tn on the bf16 matrix cores, same three-way split as gemm_nn_split_kernel.  Both operands are contracted
// over the rows, so both tiles are stored transposed (8 consecutive rows of one column per lane and MFMA): a thread
// loads 4 T rows of one column, which is coalesced across the threads of a wavefront (consecutive columns).
// PRO 1 forms G = nu (relu(T) - Z) 1[T > 0] from T (passed as G) and Zl while loading.  Tile 64 T x 64 T; T, PF as there.
// A row's address is uniform over a wavefront: scalar instructions form it, a thread adds its column.
// Four wavefronts per SIMD are asked for without the prologue (1.68 -> 1.49 ms for 500000 x 512 x 512); with it that spills
// sixteen registers in the loop and loses more than the fourth wavefront gains.
template <int PRO, int T, int PF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(T == 2 && PRO == 0 ? 4 : 1, T == 2 && PRO == 0 ? 4 : 8))) void gemm_tn_split_kernel(const float* __restrict__ A, const float* __restrict__ G,
                                                            const float* __restrict__ Zl, float nu,
                                                            float* __restrict__ partial, int64_t n, int K, int C,
                                                            int64_t rows_per_chunk, const int32_t* __restrict__ gate) {
    if (PRO == 1 && T == 2 && gate && *gate == 0) return;
    constexpr int BT = 64 * T;
    constexpr int LDH = BK + 8;
    constexpr int PLANE = BT * LDH;
    constexpr int NR = 4 * T;                     // rows per thread
    __shared__ __align__(16) unsigned short smem[6 * PLANE];
    unsigned short* const As = smem;              // [3][BT columns of A][LDH rows]
    unsigned short* const Gs = smem + 3 * PLANE;  // [3][BT columns of G][LDH rows]
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, lk = lane >> 5;
    const int ktiles = (K + BT - 1) / BT;
    const int ctiles = (C + BT - 1) / BT;
    int tile;
    int64_t chunk;
    xcd_group(blockIdx.x, gridDim.x, (unsigned)(ktiles * ctiles), chunk, tile);
    const int k0 = (tile / ctiles) * BT;
    const int c0 = (tile % ctiles) * BT;
    const int64_t r_begin = chunk * rows_per_chunk;
    const int64_t r_end = (r_begin + rows_per_chunk < n) ? (r_begin + rows_per_chunk) : n;

    floatx16 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // this thread: column `col` of both tiles (one past the edge repeats the last: never stored), rows NR rg .. NR rg + NR - 1
    const int col = tid & (BT - 1);
    const int rg = __builtin_amdgcn_readfirstlane(tid / BT);
    const int acol = k0 + col < K ? k0 + col : K - 1, gcol = c0 + col < C ? c0 + col : C - 1;
    float ra[PF][NR], rgv[PF][NR], rz[PRO ? PF : 1][NR];
    auto fetch = [&](int s, int64_t r0) {
#pragma unroll
        for (int e = 0; e < NR; ++e) {
            const int64_t r = r0 + NR * rg + e;
            const int64_t rr = r < r_end ? r : r_end - 1;      // rows past the chunk: G is set to zero there
            ra[s][e] = (A + rr * K)[acol];
            rgv[s][e] = (G + rr * C)[gcol];
            if constexpr (PRO == 1) rz[s][e] = (Zl + rr * C)[gcol];
        }
    };
    auto stash = [&](int s, int64_t r0) {
        stash_split<NR>(As, PLANE, col * LDH + NR * rg, ra[s]);
        if constexpr (PRO == 1)
#pragma unroll
            for (int e = 0; e < NR; ++e) rgv[s][e] = rgv[s][e] > 0.f ? nu * (rgv[s][e] - rz[s][e]) : 0.f;
        if (r0 + BK > r_end)
#pragma unroll
            for (int e = 0; e < NR; ++e) rgv[s][e] = r0 + NR * rg + e < r_end ? rgv[s][e] : 0.f;
        stash_split<NR>(Gs, PLANE, col * LDH + NR * rg, rgv[s]);
    };
    const int steps = r_begin < r_end ? (int)((r_end - r_begin + BK - 1) / BK) : 0;
#pragma unroll
    for (int s = 0; s < PF; ++s)
        if (s < steps) fetch(s, r_begin + s * BK);
    for (int t0 = 0; t0 < steps; t0 += PF) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            const int t = t0 + s;
            if (PF > 1 && t >= steps) break;
            __syncthreads();
            stash(s, r_begin + (int64_t)t * BK);
            __syncthreads();
            if (t + PF < steps) fetch(s, r_begin + (int64_t)(t + PF) * BK);
            multiply_split<T, LDH>(acc, As, Gs, wm * 32 * T + li, wn * 32 * T + li, lk);
        }
    }
    float* dst = partial + chunk * (int64_t)K * C;
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int c = c0 + wn * 32 * T + j * 32 + li;
            if (c >= C) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = k0 + wm * 32 * T + i * 32 + 8 * (r >> 2) + 4 * lk + (r & 3);
                if (k < K) dst[(int64_t)k * C + c] = acc[i][j][r];
            }
        }
}

// gemm_tn_split_kernel<1> in larger tiles, for matrices whose rows fill them.  With the prologue a thread holds three
// operands' numbers in flight, which leaves the 128 x 128 kernel at three wavefronts per SIMD; per step it has two barriers and
// 24 matrix instructions of a wavefront for 16 numbers to split per lane and 12 LDS reads of 16 bytes.  Here a workgroup forms
// 256 x 128, a wavefront 128 x 64 of it (128 accumulator registers, two wavefronts per SIMD): 48 matrix instructions for 24 numbers
// and 18 reads, three quarters as much of either, two buffers and one barrier per step, and the next step's numbers are formed and
// split between the matrix instructions of this one.
// 500000 x 512 x 512 1657 -> 1332 us (in iterations in which eight such layers step 1850 -> 1510), 200000 x 256 x 256 198 -> 162,
// 20000 x 700 x 512 128 -> 100, 30000 x 480 x 200 71 -> 58, 13752 x 767 x 1000 174 -> 159.  The same tile without the prologue
// gains 0 to 6 % (the 128 x 128 kernel then fits four wavefronts), and in out = A B it loses to its longer epilogue what it
// gains: not used there.
// Not on pairs of fp16, which would take half the matrix instructions (1534 -> 1064 us): the sum runs along the rows, whose sizes
// in a column of A and of G have nothing to do with each other, and where the largest entry of a column meets zeros, or large rows of
// the one meet small rows of the other, an entry held to a part of its column's largest is not held to enough of itself (features of
// some nodes 1e7 times the others', those nodes' G zero: 4e-6 of |A||G|; rows of e^(4 N(0,1)) against their inverses: 1e-3).
constexpr int kWideM = 4, kWideN = 2;                        // 32 x 32 accumulators of a wavefront
constexpr int kWideRows = 64 * kWideM, kWideCols = 64 * kWideN;
constexpr int kWideA = kWideRows * BK, kWideB = kWideCols * BK;        // bf16 of one plane: the tile of A, then that of B
constexpr int kWideBuf = 3 * (kWideA + kWideB);
// A tile row's 16 k are two 16-byte halves, swapped in every other group of four rows: the eight lanes that read or write at
// once hit different banks without padding.  Element of the half that holds k (0 or 8) of row r:
__device__ __forceinline__ int wide_at(int r, int half) { return r * BK + ((half ^ ((r >> 2) & 1)) << 3); }
// One step: the products of the tiles in S; after those of accumulator row i, between(i).
template <class F>
__device__ __forceinline__ void wide_step(floatx16 (&acc)[kWideM][kWideN], const unsigned short* S, int ao, int bo, F between) {
    bf16x8 b[kWideN][3], a[2][3];
    auto load_a = [&](bf16x8 (&x)[3], int i) {
#pragma unroll
        for (int p = 0; p < 3; ++p) x[p] = *reinterpret_cast<const bf16x8*>(S + ao + p * kWideA + i * 32 * BK);
    };
#pragma unroll
    for (int j = 0; j < kWideN; ++j)
#pragma unroll
        for (int p = 0; p < 3; ++p) b[j][p] = *reinterpret_cast<const bf16x8*>(S + bo + p * kWideB + j * 32 * BK);
    load_a(a[0], 0);
#pragma unroll
    for (int i = 0; i < kWideM; ++i) {
        if (i + 1 < kWideM) load_a(a[(i + 1) & 1], i + 1);
        constexpr int P[6] = {2, 0, 1, 1, 0, 0}, Q[6] = {0, 2, 1, 0, 1, 0};          // smallest terms first
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int j = 0; j < kWideN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i & 1][P[t]], b[j][Q[t]], acc[i][j], 0, 0, 0);
        between(i);
    }
}

__global__ __launch_bounds__(256, 2) void gemm_tn_wide_kernel(const float* __restrict__ A, const float* __restrict__ G,
                                                              const float* __restrict__ Zl, float nu,
                                                              float* __restrict__ partial, int64_t n, int K, int C,
                                                              int64_t rows_per_chunk, const int32_t* __restrict__ gate) {
    if (gate && *gate == 0) return;
    __shared__ __align__(16) unsigned short smem[2 * kWideBuf];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, lk = lane >> 5;
    const int ktiles = (K + kWideRows - 1) / kWideRows;
    const int ctiles = (C + kWideCols - 1) / kWideCols;
    int tile;
    int64_t chunk;
    xcd_group(blockIdx.x, gridDim.x, (unsigned)(ktiles * ctiles), chunk, tile);
    const int k0 = (tile / ctiles) * kWideRows;
    const int c0 = (tile % ctiles) * kWideCols;
    const int64_t r_begin = chunk * rows_per_chunk;
    const int64_t r_end = (r_begin + rows_per_chunk < n) ? (r_begin + rows_per_chunk) : n;

    floatx16 acc[kWideM][kWideN];
#pragma unroll
    for (int i = 0; i < kWideM; ++i)
#pragma unroll
        for (int j = 0; j < kWideN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // columns past the edge repeat the last one: never stored; rows past the chunk: G is set to zero there
    const int col = tid & (kWideCols - 1);
    const int rg = __builtin_amdgcn_readfirstlane(tid / kWideCols);
    const int acol = k0 + tid < K ? k0 + tid : K - 1, gcol = c0 + col < C ? c0 + col : C - 1;
    float ra[2][8], rgv[8], rz[8];
    auto fetch_a = [&](int64_t r0, int h) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t r = r0 + 8 * h + e;
            ra[h][e] = (A + (r < r_end ? r : r_end - 1) * K)[acol];
        }
    };
    auto fetch_g = [&](int64_t r0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t r = r0 + 8 * rg + e, rr = r < r_end ? r : r_end - 1;
            rgv[e] = (G + rr * C)[gcol];
            rz[e] = (Zl + rr * C)[gcol];
        }
    };
    const int aw = wide_at(tid, 0), aw8 = wide_at(tid, 1), gw = 3 * kWideA + wide_at(col, rg);
    auto stash_a = [&](unsigned short* D, int h) { stash_split<8>(D, kWideA, h ? aw8 : aw, ra[h]); };
    auto stash_g = [&](unsigned short* D, int64_t r0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) rgv[e] = rgv[e] > 0.f ? nu * (rgv[e] - rz[e]) : 0.f;
        if (r0 + BK > r_end)
#pragma unroll
            for (int e = 0; e < 8; ++e) rgv[e] = r0 + 8 * rg + e < r_end ? rgv[e] : 0.f;
        stash_split<8>(D, kWideB, gw, rgv);
    };
    const int ao = wide_at(wm * 32 * kWideM + li, lk), bo = 3 * kWideA + wide_at(wn * 32 * kWideN + li, lk);
    const int steps = r_begin < r_end ? (int)((r_end - r_begin + BK - 1) / BK) : 0;
    if (steps > 0) {
        fetch_a(r_begin, 0);
        fetch_a(r_begin, 1);
        fetch_g(r_begin);
        stash_a(smem, 0);
        stash_a(smem, 1);
        stash_g(smem, r_begin);
        const int64_t r1 = r_begin + BK;
        fetch_a(r1, 0);                           // (past the chunk's end: its last row again, stored nowhere)
        fetch_a(r1, 1);
        fetch_g(r1);
    }
    for (int t = 0; t < steps; ++t) {
        unsigned short* const D = smem + ((t + 1) & 1) * kWideBuf;
        const int64_t r1 = r_begin + (int64_t)(t + 1) * BK, r2 = r1 + BK;
        __syncthreads();
        // (behind the last step the buffer that nobody reads any more is filled once more)
        wide_step(acc, smem + (t & 1) * kWideBuf, ao, bo, [&](int i) {
            if (i == 0) { stash_a(D, 0); fetch_a(r2, 0); }
            if (i == 1) { stash_a(D, 1); fetch_a(r2, 1); }
            if (i == 2) { stash_g(D, r1); fetch_g(r2); }
        });
    }
    float* dst = partial + chunk * (int64_t)K * C;
#pragma unroll
    for (int i = 0; i < kWideM; ++i)
#pragma unroll
        for (int j = 0; j < kWideN; ++j) {
            const int c = c0 + wn * 32 * kWideN + j * 32 + li;
            if (c >= C) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int k = k0 + wm * 32 * kWideM + i * 32 + 8 * (r >> 2) + 4 * lk + (r & 3);
                if (k < K) dst[(int64_t)k * C + c] = acc[i][j][r];
            }
        }
}

// out = sum of the chunks' partial matrices, in fp64 and in a fixed order.  A workgroup takes 4 X entries: X lanes of four
// consecutive entries, 256 / X groups of lanes that take the chunks round-robin, four loads in flight each, and are
// added up in LDS.  X = 16 for large results, 4 for small ones, whose few workgroups would walk many chunks one by one.
// With W, the workgroup also leaves its share of ||out||^2 and ||W||^2 in norms (two doubles per workgroup).
template <int X, bool GATED>
__global__ __launch_bounds__(256) void gemm_tn_reduce_kernel(const float* __restrict__ partial, float* __restrict__ out,
                                                             int64_t count, int nchunks, const float* __restrict__ W,
                                                             double* __restrict__ norms, const int32_t* __restrict__ gate) {
    if constexpr (GATED) {
        if (*gate == 0) return;
    }
    constexpr int G = 256 / X;
    __shared__ double sm[G][4 * X];
    const int x = threadIdx.x & (X - 1), y = threadIdx.x / X;
    double ng = 0.0, nw = 0.0;
    for (int64_t i0 = (int64_t)blockIdx.x * (4 * X); i0 < count; i0 += (int64_t)gridDim.x * (4 * X)) {
        const int64_t i = i0 + 4 * x;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        auto sum = [&](auto whole) {
            for (int c0 = y; c0 < nchunks; c0 += 4 * G) {
                float v[4][4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = c0 + u * G < nchunks ? c0 + u * G : c0;
                    if constexpr (decltype(whole)::value) {
                        const float4u q = *reinterpret_cast<const float4u*>(partial + (int64_t)c * count + i);
                        v[u][0] = q.x; v[u][1] = q.y; v[u][2] = q.z; v[u][3] = q.w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[u][e] = partial[(int64_t)c * count + (i + e < count ? i + e : count - 1)];
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (c0 + u * G < nchunks)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[e] += (double)v[u][e];
            }
        };
        if (i + 4 <= count) sum(std::true_type{});
        else sum(std::false_type{});                     // (entries past the end are not written)
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) sm[y][4 * x + e] = acc[e];
        __syncthreads();
        if (threadIdx.x < 4 * X && i0 + threadIdx.x < count) {
            double t = 0.0;
#pragma unroll 8
            for (int q = 0; q < G; ++q) t += sm[q][threadIdx.x];
            const float g = (float)t;
            out[i0 + threadIdx.x] = g;
            if (W) {
                const double w = (double)W[i0 + threadIdx.x];
                ng += (double)g * (double)g;
                nw += w * w;
            }
        }
    }
    if (W && threadIdx.x < 64) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) { ng += __shfl_down(ng, o, 64); nw += __shfl_down(nw, o, 64); }
        if (threadIdx.x == 0) { norms[2 * blockIdx.x] = ng; norms[2 * blockIdx.x + 1] = nw; }
    }
}

__global__ __launch_bounds__(256) void transpose_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                        int K, int C) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= K * C) return;
    const int k = i / C, c = i % C;
    out[c * K + k] = in[i];
}

// Machine calibration: nothing but dependent chains of fp32 MFMAs on registers, four chains per wavefront.
__global__ __launch_bounds__(256) void mfma_chain_kernel(float* __restrict__ out, int iters, float seed) {
    floatx16 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    const float a = seed + (float)(threadIdx.x & 7), b = 0.5f * seed;
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc[j], 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += acc[j][r];
    out[(int64_t)blockIdx.x * 256 + threadIdx.x] = s;
}

// Machine calibration: chains of bf16 MFMAs (32x32x16) on registers, four chains per wavefront.  With VALU > 0, that
// many independent vector instructions (fused multiply-adds on registers of their own) follow every matrix
// instruction: whether the vector ALU runs beside the matrix cores, and how many instructions fit per matrix instruction.
template <int VALU>
__global__ __launch_bounds__(256) void mfma_bf16_chain_kernel(float* __restrict__ out, int iters, float seed) {
    floatx16 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    intx4 a, b;
    a.x = a.y = a.z = a.w = 0x3F803F80 + (int)(threadIdx.x & 7);      // pairs of bf16 near 1
    b.x = b.y = b.z = b.w = 0x3F003F00;
    float v[VALU > 0 ? VALU : 1];
#pragma unroll
    for (int q = 0; q < (VALU > 0 ? VALU : 1); ++q) v[q] = seed + (float)q;
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc[j],
                                                             0, 0, 0);
#pragma unroll
            for (int q = 0; q < VALU; ++q) v[q] = __builtin_fmaf(v[q], 0.999f, seed);
            if constexpr (VALU > 0) {
                // keep each matrix instruction and its vector instructions together in the schedule
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);        // one MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, VALU, 0);     // VALU instructions
            }
        }
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += acc[j][r];
#pragma unroll
    for (int q = 0; q < (VALU > 0 ? VALU : 1); ++q) s += v[q];
    out[(int64_t)blockIdx.x * 256 + threadIdx.x] = s;
}

// Machine calibration: dst = src, one float4 per thread and step.
__global__ __launch_bounds__(256) void stream_copy_kernel(const float4* __restrict__ src, float4* __restrict__ dst,
                                                          int64_t n4) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) dst[i] = src[i];
}

// Machine calibration: dst = 0.999 dst + src in place, one float4 per thread and step: two arrays read, one of them
// written back to where it was read, the memory mix of the step kernels.
__global__ __launch_bounds__(256) void stream_update_kernel(const float4* __restrict__ src, float4* __restrict__ dst,
                                                            int64_t n4) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
        const float4 a = src[i];
        float4 d = dst[i];
        d.x = 0.999f * d.x + a.x; d.y = 0.999f * d.y + a.y; d.z = 0.999f * d.z + a.z; d.w = 0.999f * d.w + a.w;
        dst[i] = d;
    }
}

// 1: wide products run on the 16-bit matrix cores with split operands (pairs of fp16 or three bf16, by size), 0: fp32 MFMA,
// 2: pairs of fp16 wherever gemm_nn_pair_form allows
int g_split = 1;

// Tiles per wavefront direction of the split product out[n x C]: 128 x 128 tiles where they give every compute unit two, else
// 64 x 64 (see gemm_nn_split_kernel).
constexpr int64_t kFewTiles = 512;
int nn_tile(int64_t n, int C, int split) {
    if (!split) return 2;
    return ((n + 127) / 128) * ((C + 127) / 128) < kFewTiles ? 1 : 2;
}

}  // namespace

// (below 64 long sums the pairs are the less accurate split)
bool gemm_nn_pair_form(int K, int C) { return K >= 64 && C >= kPairLeast; }
// A workgroup's tile is larger than the bf16 kernels' (columns past C cost as much as others), B takes a launch of its own to be split
// (5 us), and both weigh the more the shorter the sums: pairs pay from 3.3e6 results and, for sums shorter than 512, 3.2e11 / K^2 on.  us with
// bf16 and with pairs, that launch with them (forward product): 10000 x 512 x 512 48.9 and 40.7, 24000 x 256 x 256 34.5 and 29.5,
// 20000 x 256 x 256 24.5 and 21.4, 80000 x 128 x 512 90 and 82, 160000 x 256 x 256 148 and 115, 13752 x 767 x 1000 149 and 84; below the line
// 10000 x 449 x 289 31 and 40, 10000 x 800 x 129 38 and 56, 10000 x 128 x 512 19.6 and 24.5, 40000 x 128 x 289 36 and 46, 12000 x 256 x 256
// 17.3 and 20.2.  Of 252 shapes (6000 to 160000 rows, 128 to 800 long sums, 129 to 1000 columns) it sends 140 to pairs, at 0.55 to 1.07 of
// bf16's time, and keeps four from them that would gain a tenth.  (Every tile on pairs; with none of them, 1.1 to 1.7 of bf16's time, the least in
// the largest.)
bool gemm_nn_pair(int64_t n, int K, int C) {
    if (!gemm_nn_pair_form(K, C) || g_split == 0) return false;
    const double results = (double)n * C;
    return g_split == 2 || (K >= 128 && results >= 3.3e6 && results * K * K >= 3.2e11);
}
int gemm_nn_pair_tiles(int C) { return (C + kPairCols - 1) / kPairCols; }
size_t gemm_nn_pair_planes(int K, int C) { return (size_t)((K + kPairK - 1) / kPairK) * ((C + 31) / 32) * kPairSub; }

// Scratch is asked for by shape alone, so that a workspace holds what its shapes need however the library is tuned later.
// The base is that of chunks of at least 256 rows, about 1024 workgroups of 128-row tiles; callers are refused by it.  Small
// shapes get up to five times that, so that they can be cut into chunks of 64 rows (four times the chunks, and one more for
// what rounding adds): 2000 x 256 x 64 18.0 us in the base's scratch, 12.6 in three times and 11.6 in five to eight times
// that; 5000 x 100 x 20 18.3, 12.9 and 12.1 us.  32 MiB are as much as they get by it: limits of 8 to 64 MiB measured the
// same, since shapes that would need more have workgroups enough at the base.
constexpr size_t kTnSmallScratch = (size_t)8 << 20;
size_t gemm_tn_base_floats(int64_t n, int K, int C) {
    const int64_t bn = C > 32 ? 128 : 32, tiles = ((K + BM - 1) / BM) * ((C + bn - 1) / bn);
    const int64_t nch = std::max<int64_t>(1, std::min<int64_t>((1024 + tiles - 1) / tiles, (n + 255) / 256));
    const int64_t rpc = std::max<int64_t>(BK, ((n + nch - 1) / nch + BK - 1) / BK * BK);
    return (size_t)std::max<int64_t>(1, (n + rpc - 1) / rpc) * K * C;
}
size_t gemm_tn_reserve(size_t base) { return std::max(base, std::min(kTnSmallScratch, 5 * base)); }
size_t gemm_tn_scratch_floats(int64_t n, int K, int C) { return gemm_tn_reserve(gemm_tn_base_floats(n, K, C)); }

namespace {

struct TnPlan {
    int nchunks;
    int64_t rows_per_chunk;
    int bn;              // columns per tile: 128, 64 (split product with few workgroups) or 32
    int tiles;
    bool wide;           // 256 rows of K per tile: gemm_tn_wide_kernel
};

// The rows are cut into chunks so that about 1024 workgroups share the product, four per compute unit.  A chunk has at
// least 64 rows, and beyond 32 chunks the partial matrices stay below half the size of the operands.  The sums over a
// chunk's rows are in fp32, their error grows with its length: whatever the tile and these limits ask for, there are no
// fewer chunks than at the base (128-row tiles, 256 rows).  Longer chunks would be faster with the prologue, whose
// registers let the chip hold 768 workgroups and not 1024, but not as accurate: with 128 x 128 tiles 13752 x 767 x 1000 in
// 864 rows 157 us and 4.6e-7 of the 64-bit product, in 640 rows 182 us and 3.9e-7; 16956 x 476 x 347 in 784 rows 83 us and 4.4e-7,
// in 256 rows 76 us and 2.6e-7.  They fit the scratch of the shape (gemm_tn_scratch_floats) whatever tile and operand path is chosen.
constexpr int kTnBlocks = 1024;
// prologue: the right operand is formed on the way.
TnPlan tn_plan(int64_t n, int K, int C, bool prologue) {
    TnPlan p;
    const int64_t base_chunks = (int64_t)gemm_tn_base_floats(n, K, C) / ((int64_t)K * C);
    auto plan = [&](int bm, int bn, int blocks = kTnBlocks) {
        p.bn = bn;
        p.wide = bm == kWideRows;
        p.tiles = ((K + bm - 1) / bm) * ((C + bn - 1) / bn);
        int64_t nch = (blocks + p.tiles - 1) / p.tiles;
        nch = std::min(nch, (n + 63) / 64);
        nch = std::min(nch, std::max<int64_t>(32, n * (K + C) / (2 * (int64_t)K * C)));
        nch = std::min(nch, (int64_t)gemm_tn_scratch_floats(n, K, C) / ((int64_t)K * C));
        nch = std::max(nch, base_chunks);
        int64_t rpc = (n + nch - 1) / nch;
        rpc = (rpc + BK - 1) / BK * BK;
        p.rows_per_chunk = rpc;
        p.nchunks = (int)std::max<int64_t>(1, (n + rpc - 1) / rpc);
    };
    if (C <= 32) { plan(BM, 32); return p; }
    plan(BM, 128);
    if (g_split && (int64_t)p.nchunks * p.tiles < kFewTiles) plan(64, 64);
    // (where the last 256 rows would be half empty the tiles cost more than they gain: 384 x 256 138 -> 188 us)
    else if (g_split && prologue && (K + kWideRows - 1) / kWideRows * 2 == (K + 127) / 128) plan(kWideRows, 128, kTnBlocks / 2);
    return p;
}

}  // namespace

void set_gemm_split(int mode) { g_split = mode == 0 || mode == 2 ? mode : 1; }
int get_gemm_split() { return g_split; }

void launch_gemm_nn(hipStream_t s, const float* A, const float* B, float* out, int64_t n, int K, int C,
                    const GemmEpilogue& epi) {
    if (n <= 0 || C <= 0) return;
    const dim3 block(256);
    if (epi.pair.planes && gemm_nn_pair(n, K, C)) {
        const PairOperands& p = epi.pair;
        if (!p.ready) hipLaunchKernelGGL(pair_weights_kernel, dim3((unsigned)((C + 31) / 32)), dim3(1024), 0, s, B, K, C, p.planes, p.columns, epi.gate);
        const dim3 grid((unsigned)gemm_nn_blocks(n, C, true));
#define CADMM_PAIR(E_, Tl_, unit_, partials_, out_max_, gate_) \
        hipLaunchKernelGGL(gemm_nn_pair_kernel<E_>, grid, dim3(64 * kPairWaves), 0, s, A, B, p.planes, p.columns, p.row_range, p.range_tiles, out, \
                           n, K, C, epi.Zl, Tl_, epi.nu, epi.Tio, unit_, partials_, out_max_, gate_)
        double* const bad = reinterpret_cast<double*>(epi.bad);
        if (epi.kind == 3) CADMM_PAIR(3, nullptr, nullptr, bad, nullptr, nullptr);
        else if (epi.kind == 2 && epi.leave_g) CADMM_PAIR(4, nullptr, epi.unit, epi.partials, nullptr, epi.gate);
        else if (epi.kind == 2) CADMM_PAIR(2, nullptr, epi.unit, epi.partials, nullptr, epi.gate);
        else if (epi.kind == 1) CADMM_PAIR(1, epi.Tl, nullptr, epi.row_sums, epi.out_range, epi.gate);
        else CADMM_PAIR(0, nullptr, epi.unit, nullptr, nullptr, epi.gate);
#undef CADMM_PAIR
        return;
    }
    if (C > 32) {
        const int t = nn_tile(n, C, g_split);
        const dim3 grid((unsigned)gemm_nn_blocks(n, C, false));
#define CADMM_NN(K4_, K3_, K2_, K1_, K0_) \
        if (epi.kind == 3) \
            hipLaunchKernelGGL(K3_, grid, block, 0, s, A, B, out, n, K, C, nullptr, nullptr, 0.f, epi.Tio, nullptr, \
                               reinterpret_cast<double*>(epi.bad), nullptr); \
        else if (epi.kind == 2 && epi.leave_g) \
            hipLaunchKernelGGL(K4_, grid, block, 0, s, A, B, out, n, K, C, epi.Zl, nullptr, epi.nu, epi.Tio, epi.unit, \
                               epi.partials, epi.gate); \
        else if (epi.kind == 2) \
            hipLaunchKernelGGL(K2_, grid, block, 0, s, A, B, out, n, K, C, epi.Zl, nullptr, epi.nu, epi.Tio, epi.unit, \
                               epi.partials, epi.gate); \
        else if (epi.kind == 1) \
            hipLaunchKernelGGL(K1_, grid, block, 0, s, A, B, out, n, K, C, epi.Zl, epi.Tl, epi.nu, nullptr, nullptr, \
                               epi.row_sums, epi.gate); \
        else \
            hipLaunchKernelGGL(K0_, grid, block, 0, s, A, B, out, n, K, C, nullptr, nullptr, 0.f, nullptr, epi.unit, \
                               nullptr, epi.gate)
        if (!g_split) {
            CADMM_NN((gemm_nn_kernel<4>), (gemm_nn_kernel<3>), (gemm_nn_kernel<2>), (gemm_nn_kernel<1>), (gemm_nn_kernel<0>));
        } else if (t == 2) {
            CADMM_NN((gemm_nn_split_kernel<4, 2, 1>), (gemm_nn_split_kernel<3, 2, 1>), (gemm_nn_split_kernel<2, 2, 1>), (gemm_nn_split_kernel<1, 2, 1>), (gemm_nn_split_kernel<0, 2, 1>));
        } else {
            CADMM_NN((gemm_nn_split_kernel<4, 1, 4>), (gemm_nn_split_kernel<3, 1, 4>), (gemm_nn_split_kernel<2, 1, 4>), (gemm_nn_split_kernel<1, 1, 4>), (gemm_nn_split_kernel<0, 1, 4>));
        }
#undef CADMM_NN
    } else {
        // (two workgroups per compute unit, as for the wide products; the rows are the only tiles here)
        const bool few = (n + 127) / 128 < kFewTiles;
        const dim3 grid((unsigned)(few ? (n + 31) / 32 : (n + 127) / 128));
#define CADMM_NARROW(E_) \
        if (few) hipLaunchKernelGGL((gemm_nn_narrow_kernel<E_, 1>), grid, block, 0, s, A, B, out, n, K, C, epi.Zl, epi.Tl, epi.nu, epi.Tio, epi.gate); \
        else hipLaunchKernelGGL((gemm_nn_narrow_kernel<E_, 0>), grid, block, 0, s, A, B, out, n, K, C, epi.Zl, epi.Tl, epi.nu, epi.Tio, epi.gate)
        if (epi.kind == 3) { CADMM_NARROW(3); }
        else if (epi.kind == 1) { CADMM_NARROW(1); }
        else if (epi.gate) { CADMM_NARROW(kGated); }
        else { CADMM_NARROW(0); }
#undef CADMM_NARROW
    }
}

void launch_gemm_nn_gradz(hipStream_t s, const float* Zl, const float* Tl, const float* SG, const float* Wt, float* out, int64_t n,
                          int K1, int C, float nu, double* row_sums, const int32_t* gate) {
    if (n <= 0) return;
    const dim3 grid((unsigned)((n + BM - 1) / BM));
    if (gate) hipLaunchKernelGGL((gemm_nn_gradz_kernel<true>), grid, dim3(256), 0, s, Zl, Tl, SG, Wt, out, n, K1, C, nu, row_sums, gate);
    else hipLaunchKernelGGL((gemm_nn_gradz_kernel<false>), grid, dim3(256), 0, s, Zl, Tl, SG, Wt, out, n, K1, C, nu, row_sums, gate);
}

int gemm_nn_tiles(int64_t n, int C, bool pair) {
    if (pair) return gemm_nn_pair_tiles(C);
    const int b = 64 * nn_tile(n, C, g_split);
    return (C + b - 1) / b;
}
int gemm_nn_most_tiles(int64_t n, int C) {
    const int b = 64 * nn_tile(n, C, 1);
    return (C + b - 1) / b;
}

bool gemm_nn_notes_bad(int C) { return C > 32; }

int64_t gemm_nn_blocks(int64_t n, int C, bool pair) {
    if (pair) return ((n + kPairRows - 1) / kPairRows) * gemm_nn_pair_tiles(C);
    const int b = 64 * nn_tile(n, C, g_split);
    return ((n + b - 1) / b) * ((C + b - 1) / b);
}

int launch_gemm_tn(hipStream_t s, const float* A, const float* G, float* out, int64_t n, int K, int C,
                   float* partial, const float* Zl, float nu, const float* W, double* norms, const int32_t* gate) {
    if (K <= 0 || C <= 0) return 0;
    TnPlan p = tn_plan(n, K, C, Zl != nullptr);
    const dim3 grid((unsigned)((int64_t)p.nchunks * p.tiles)), block(256);
#define CADMM_TN(KERNEL_, ...) hipLaunchKernelGGL(KERNEL_, grid, block, 0, s, A, G, Zl, nu, partial, n, K, C, p.rows_per_chunk, ##__VA_ARGS__)
    if (p.bn == 64) {
        if (Zl) CADMM_TN((gemm_tn_split_kernel<1, 1, 4>), gate);
        else CADMM_TN((gemm_tn_split_kernel<0, 1, 4>), gate);
    } else if (p.wide) {
        CADMM_TN(gemm_tn_wide_kernel, gate);
    } else if (g_split && p.bn == 128) {
        if (Zl) CADMM_TN((gemm_tn_split_kernel<1, 2, 1>), gate);
        else CADMM_TN((gemm_tn_split_kernel<0, 2, 1>), gate);
    } else if (p.bn == 128) {
        if (Zl) CADMM_TN((gemm_tn_kernel<128, 1, 0>));
        else CADMM_TN((gemm_tn_kernel<128, 0, 0>));
    } else {
        const bool full = K % 4 == 0 && C % 4 == 0;
        if (Zl) CADMM_TN((gemm_tn_kernel<32, 1, 0>));
        else if (full) CADMM_TN((gemm_tn_kernel<32, 0, 1>));
        else CADMM_TN((gemm_tn_kernel<32, 0, 0>));
    }
#undef CADMM_TN
    const int64_t count = (int64_t)K * C;
    const bool large = count >= 16384;               // a workgroup of 64 entries on every compute unit
    const int64_t tiles = (count + (large ? 63 : 15)) / (large ? 64 : 16);
    const int nb = (int)(tiles < kReduceBlocks ? tiles : kReduceBlocks);
#define CADMM_REDUCE(X_, G_) hipLaunchKernelGGL((gemm_tn_reduce_kernel<X_, G_>), dim3(nb), block, 0, s, partial, out, count, p.nchunks, W, norms, gate)
    if (large) { if (gate) CADMM_REDUCE(16, true); else CADMM_REDUCE(16, false); }
    else { if (gate) CADMM_REDUCE(4, true); else CADMM_REDUCE(4, false); }
#undef CADMM_REDUCE
    return nb;
}

double launch_mfma_chain(hipStream_t s, float* out, int blocks, int iters) {
    hipLaunchKernelGGL(mfma_chain_kernel, dim3((unsigned)blocks), dim3(256), 0, s, out, iters, 1.0f);
    return (double)blocks * 4.0 * iters * 4.0 * (32.0 * 32.0 * 2.0 * 2.0);      // flops
}

double launch_mfma_bf16_chain(hipStream_t s, float* out, int blocks, int iters, int valu) {
    if (valu <= 0) hipLaunchKernelGGL((mfma_bf16_chain_kernel<0>), dim3((unsigned)blocks), dim3(256), 0, s, out, iters, 1.0f);
    else if (valu <= 4) hipLaunchKernelGGL((mfma_bf16_chain_kernel<4>), dim3((unsigned)blocks), dim3(256), 0, s, out, iters, 1.0f);
    else if (valu <= 6) hipLaunchKernelGGL((mfma_bf16_chain_kernel<6>), dim3((unsigned)blocks), dim3(256), 0, s, out, iters, 1.0f);
    else hipLaunchKernelGGL((mfma_bf16_chain_kernel<8>), dim3((unsigned)blocks), dim3(256), 0, s, out, iters, 1.0f);
    return (double)blocks * 4.0 * iters * 4.0 * (32.0 * 32.0 * 16.0 * 2.0);      // flops
}

void launch_stream_copy(hipStream_t s, const float* src, float* dst, int64_t count) {
    const int64_t n4 = count / 4;
    hipLaunchKernelGGL(stream_copy_kernel, dim3(8192), dim3(256), 0, s, reinterpret_cast<const float4*>(src),
                       reinterpret_cast<float4*>(dst), n4);
}

void launch_stream_update(hipStream_t s, const float* src, float* dst, int64_t count) {
    hipLaunchKernelGGL(stream_update_kernel, dim3(8192), dim3(256), 0, s, reinterpret_cast<const float4*>(src),
                       reinterpret_cast<float4*>(dst), count / 4);
}

void launch_transpose(hipStream_t s, const float* in, float* out, int K, int C) {
    hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)((K * C + 255) / 256)), dim3(256), 0, s, in, out, K, C);
}

}  // namespace cadmm

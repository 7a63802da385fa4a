// Community-blocked sparse aggregation  Y = A~ X  on gfx950 (paper, Section 2, Problem 3: row block m
// is A~_{m,m} X_m + sum_{r in N_m} A~_{m,r} X_r; Appendix A: the same sum restricted to one
// neighbour community per output row, the "segments").
//
// Layout: a row list (the CSR rows, or the (row, community) segments with several entries) laid out by the host
// for these kernels: rows sorted by (community, length class); one 16-byte record per row (its chunk range and
// output row); the entries as (column, value) pairs in chunks of eight, padded with weight zero; and a table that
// names the rows of every workgroup.  Features are row-major fp32.
//
// Mapping: a group of LPR lanes (a power of two, up to the 64-lane wavefront) reads one gathered
// neighbour row with one fully coalesced VEC*4-byte load per lane and keeps VEC accumulators per lane.
// GPR such groups share one output row and take its chunks round-robin, one chunk = eight gathers in flight per
// group and trip; their partial sums are added by a wavefront-level xor-shuffle reduction.  GPR is chosen per run
// of one length class so that one trip covers the class's longest row: short rows pack many rows into a
// wavefront, long rows spread over it, and the rows of a wavefront need the same number of trips.
// What bounds the narrow shapes (rows of up to 64 bytes) is the rate at which the L2s take 64-byte requests from the
// L1s, one per gathered row (measured with gather_calibration_kernel below); everything around the gathers is kept
// out of their way: a lane group fetches its chunk with one load of 64 bytes spread over its lanes (one instruction
// per 128 entries at 16 columns) and hands the pairs round by lane exchanges, instead of one load of four bytes per
// entry and array.
// Rows beyond a length threshold (power-law hubs) are cut into parts that run first in the same launch, into a
// side buffer; a small kernel adds a row's parts in order.  Segments with a single entry are scaled copies of a
// gathered row and have a kernel of their own.  Everything is order-fixed: no atomics, results are reproducible.
// XCD k (blockIdx mod 8) walks the k-th slice of the workgroup table, whole communities one after the other with
// all their length classes, so that the rows of the gathered matrix a community reads are fetched into that XCD's
// L2 once.
#include "kernels.h"

namespace cadmm {

namespace {

// Rows of a width that is no multiple of four start at any dword; the chip takes 16-byte global accesses there.  VEC = 4
// therefore serves every width of four and more: the last quad of a row is moved back to end with the row, and the columns
// it shares with the quad before come out the same from both.  VEC = 1 is for widths of one to three.
typedef float float_x4 __attribute__((ext_vector_type(4), aligned(4)));
template <int VEC>
__device__ __forceinline__ void load_vec(float (&dst)[VEC], const float* p) {
    if constexpr (VEC == 4) {
        const float_x4 v = *reinterpret_cast<const float_x4*>(p);
        dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
    } else {
        dst[0] = *p;
    }
}


// results are written once and read by a later kernel: streamed past the L2's resident lines
template <int VEC>
__device__ __forceinline__ void store_vec(float* p, const float (&src)[VEC]) {
    if constexpr (VEC == 4) {
        float_x4 v = {src[0], src[1], src[2], src[3]};
        __builtin_nontemporal_store(v, reinterpret_cast<float_x4*>(p));
    } else {
        __builtin_nontemporal_store(src[0], p);
    }
}

// Row sums of a gradient g with its z and t, see RowSums: this lane's share of one quad whose first `skip` columns belong to
// the quad before it.
__device__ __forceinline__ void add_row_sums(double (&s)[3], const float* g, const float* z, const float* t, int skip) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double zd = v >= skip ? (double)z[v] : 0.0, gd = v >= skip ? (double)g[v] : 0.0;
        s[0] += (v >= skip ? zd - fmax((double)t[v], 0.0) : 0.0) * gd;
        s[1] += gd * gd;
        s[2] += zd * zd;
    }
}
// adds the shares of 2^lpr_log2 neighbouring lanes; every one of them gets the sums
__device__ __forceinline__ void reduce_row_sums(double (&s)[3], int lpr_log2) {
    for (int o = 1; o < (1 << lpr_log2); o <<= 1)
#pragma unroll
        for (int q = 0; q < 3; ++q) s[q] += __shfl_xor(s[q], o, 64);
}

// Largest magnitude of a result row: this lane's quad, over 2^lpr_log2 neighbouring lanes; every one of them gets it.
__device__ __forceinline__ float quad_max(const float (&v)[4]) {
    return fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3])));
}
template <class F>
__device__ __forceinline__ int reduce_row(int v, int lpr_log2, F f) {
    if (lpr_log2 < 3) {
        for (int o = 1; o < (1 << lpr_log2); o <<= 1) v = f(v, __shfl_xor(v, o, 64));
        return v;
    }
    v = over_lanes<8>(v, f);
    for (int o = 8; o < (1 << lpr_log2); o <<= 1) v = f(v, __shfl_xor(v, o, 64));
    return v;
}
// (the bits of numbers that are not negative are in the order of the numbers)
__device__ __forceinline__ float reduce_row_max(float m, int lpr_log2) {
    return __int_as_float(reduce_row(__float_as_int(m), lpr_log2, [](int a, int b) { return a > b ? a : b; }));
}
// RowRange (range_word_of): this lane's quad from entry `skip` on, against the row's largest magnitude m.
constexpr int kNearBinades = 4;
__device__ __forceinline__ int quad_counts(const float (&v)[4], float m, int skip) {
    const float t = range_near(m, kNearBinades);
    int n = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) n += e < skip ? 0 : (fabsf(v[e]) >= t ? 1 : 0) + (v[e] != 0.f ? 1 << 16 : 0);
    return n;
}
__device__ __forceinline__ int reduce_row_counts(int n, int lpr_log2) {
    return reduce_row(n, lpr_log2, [](int a, int b) { return a + b; });
}

// Slice k of the workgroup table (the workgroups of XCD k) is [start[k], start[k+1]).
struct XcdMap {
    long long start[9];
};

template <int S>
__device__ __forceinline__ int quad_bcast(int v) {       // lane j of every quad gets lane S's value
    return __builtin_amdgcn_mov_dpp(v, S * 0x55, 0xF, 0xF, true);
}

// The eight (column, value) pairs of chunk `chunk` for every lane of a lane group of 2^LPRL lanes (LPRL = 3 stands
// for 8 and more lanes, lpr_log2 then says how many).  The group's lanes share the chunk's 64 bytes among them in
// as few load instructions as possible and exchange the pairs afterwards.
template <int LPRL>
__device__ __forceinline__ void load_chunk(const int2* __restrict__ ent, int64_t chunk, int lpr_log2, int lane,
                                           int32_t (&c)[8], float (&a)[8]) {
    const int4* e4 = reinterpret_cast<const int4*>(ent) + chunk * 4;      // a chunk is four 16-byte pieces
    if constexpr (LPRL == 0) {
        const int4 q0 = e4[0], q1 = e4[1], q2 = e4[2], q3 = e4[3];
        c[0] = q0.x; c[1] = q0.z; c[2] = q1.x; c[3] = q1.z; c[4] = q2.x; c[5] = q2.z; c[6] = q3.x; c[7] = q3.z;
        a[0] = __int_as_float(q0.y); a[1] = __int_as_float(q0.w); a[2] = __int_as_float(q1.y); a[3] = __int_as_float(q1.w);
        a[4] = __int_as_float(q2.y); a[5] = __int_as_float(q2.w); a[6] = __int_as_float(q3.y); a[7] = __int_as_float(q3.w);
    } else if constexpr (LPRL == 1) {
        const int sub = lane & 1;
        const int4 q0 = e4[2 * sub], q1 = e4[2 * sub + 1];                // pairs 4 sub .. 4 sub + 3
        const int mine[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int src = (lane & ~1) | (u >> 2);
            c[u] = __shfl(mine[2 * (u & 3)], src, 64);
            a[u] = __int_as_float(__shfl(mine[2 * (u & 3) + 1], src, 64));
        }
    } else if constexpr (LPRL == 2) {
        const int4 q = e4[lane & 3];                                      // pairs 2 sub, 2 sub + 1
        c[0] = quad_bcast<0>(q.x); a[0] = __int_as_float(quad_bcast<0>(q.y));
        c[1] = quad_bcast<0>(q.z); a[1] = __int_as_float(quad_bcast<0>(q.w));
        c[2] = quad_bcast<1>(q.x); a[2] = __int_as_float(quad_bcast<1>(q.y));
        c[3] = quad_bcast<1>(q.z); a[3] = __int_as_float(quad_bcast<1>(q.w));
        c[4] = quad_bcast<2>(q.x); a[4] = __int_as_float(quad_bcast<2>(q.y));
        c[5] = quad_bcast<2>(q.z); a[5] = __int_as_float(quad_bcast<2>(q.w));
        c[6] = quad_bcast<3>(q.x); a[6] = __int_as_float(quad_bcast<3>(q.y));
        c[7] = quad_bcast<3>(q.z); a[7] = __int_as_float(quad_bcast<3>(q.w));
    } else {
        const int base = lane & ~((1 << lpr_log2) - 1);
        const int2 q = ent[chunk * 8 + (lane & 7)];                       // lane j of the group holds pair j mod 8
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            c[u] = __shfl(q.x, base + u, 64);
            a[u] = __int_as_float(__shfl(q.y, base + u, 64));
        }
    }
}

// LPRL: lanes per gathered row as a power of two (3 stands for 8 and more, lpr_log2_arg then says how many).
// blockIdx.y: tile of tile_cols columns.  The gathered matrix is walked one column tile after the other where a
// community's rows of it do not fit an XCD's L2 at full width (see launch_vec).
// OFF32: X has at most 2^24 rows and 4 GiB.  A gather is then a uniform base and a 32-bit offset of its lane, made by one
// 24-bit multiply-add and held in one register, not by a 64-bit multiply-add in two; eight wavefronts per SIMD fit instead
// of six (they are asked for where a row takes eight lanes and more: 63 registers, not 71).  Over the rows, us before and
// after: 200000 x 256 249 and 233, x 128 120 and 109, x 33 69 and 60; 500000 x 512 1398 and 1268; 2M power law x 128 2715 and
// 2465, x 16 456 and 446.
// EPI 2: epilogue 1 with a gate (an instance of its own, as the look at it keeps the other arguments from being loaded beside it).
// RANGE: leaves RowRange (a template parameter: its registers cost the other launches 3 %).
template <int VEC, int EPI, int LPRL, int OFF32, int RANGE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OFF32 && EPI == 0 && LPRL == 3 ? 8 : 1, 8))) void spmm_rows_kernel(
    const int4* __restrict__ rec, int64_t nrows, const int2* __restrict__ ent, const float* __restrict__ X,
    float* __restrict__ Y, float* __restrict__ side, int width, int lpr_log2_arg, const int4* __restrict__ blocks,
    XcdMap xm, int tile_cols, int xcd_remap, const float* __restrict__ Zl, const float* __restrict__ Tl, float nu,
    double* __restrict__ row_sums, uint32_t* __restrict__ row_range, int64_t n_out, const int32_t* __restrict__ gate) {
    if constexpr (EPI == 2) {
        if (*gate == 0) return;
    }
    if (EPI == 0 && gate && *gate == 0) return;
    // Workgroup b belongs to XCD b mod 8 and takes the (b / 8)-th entry of that XCD's slice of the table (or, without
    // the XCD-aware numbering, simply entry b).  Records from nrows on are the parts of split rows.
    const int lpr_log2 = LPRL < 3 ? LPRL : lpr_log2_arg;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    int64_t idx;
    if (xcd_remap) {
        const int k = (int)(blockIdx.x & 7);
        idx = xm.start[k] + (blockIdx.x >> 3);
        if (idx >= xm.start[k + 1]) return;
    } else {
        idx = blockIdx.x;
        if (idx >= xm.start[8]) return;
    }
    const int4 d = blocks[idx];                         // rows [d.x, d.y), 2^d.z lane groups per row
    const int gpr_log2 = d.z;
    const int span_log2 = lpr_log2 + gpr_log2;          // lanes that share one output row
    const int64_t vrow = (int64_t)d.x + ((wave << (6 - span_log2)) + (lane >> span_log2));
    if (vrow >= d.y) return;                            // uniform over the row's lane span
    const int4 r = rec[vrow];                           // chunks [r.x, r.y), output row r.z
    const bool is_part = vrow >= nrows;
    float* const dst = (is_part ? side : Y) + (int64_t)r.z * (int64_t)width;
    const int lpr = 1 << lpr_log2;
    const int gpr = 1 << gpr_log2;
    const int grp = (lane >> lpr_log2) & (gpr - 1);
    const int sub = lane & (lpr - 1);
    const int col0 = (int)blockIdx.y * tile_cols;
    const int col1 = width - col0 < tile_cols ? width : col0 + tile_cols;
    const bool on = col0 + sub * VEC < col1;
    // a lane past the last column reads the last columns again without storing them
    const int cc = on && col0 + sub * VEC + VEC <= width ? col0 + sub * VEC : (on ? width : col1) - VEC;

    const uint32_t pitch = 4u * (uint32_t)width, cc4 = 4u * (uint32_t)cc;
    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
    // the epilogue's operands (rows of Z_l and T_l at the output row) are asked for before the gathers, so that their
    // latency is not added at the end of every row
    float ez[VEC], et[VEC];
    if constexpr (EPI >= 1) {
        if (!is_part && grp == 0) {
            const int64_t o = (int64_t)r.z * (int64_t)width + cc;
            load_vec<VEC>(ez, Zl + o);
            load_vec<VEC>(et, Tl + o);
        }
    }
    // the groups of a row take its chunks grp, grp + gpr, ...: eight gathers in flight per group; the padding of a chunk
    // carries weight zero, so no entry is masked
    for (int ch = r.x + grp; ch < r.y; ch += gpr) {
        int32_t c[8];
        float a[8];
        load_chunk<LPRL>(ent, ch, lpr_log2, lane, c, a);
        float x[8][VEC];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if constexpr (OFF32)
                load_vec<VEC>(x[u], reinterpret_cast<const float*>(reinterpret_cast<const char*>(X) + (__umul24((uint32_t)c[u], pitch) + cc4)));
            else
                load_vec<VEC>(x[u], X + (int64_t)c[u] * width + cc);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = fmaf(a[u], x[u][v], acc[v]);
    }
    // wavefront-level reduction across the groups of the row
    for (int off = lpr; off < (lpr << gpr_log2); off <<= 1) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += __shfl_xor(acc[v], off, 64);
    }
    if (grp != 0) return;
    if constexpr (EPI >= 1) {
        if (!is_part) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = nu * (ez[v] - fmaxf(et[v], 0.f)) + acc[v];
            if constexpr (VEC == 4) {
                if (row_sums) {                          // (uniform; every lane of the row's first group is here)
                    double rs[3] = {0.0, 0.0, 0.0};
                    add_row_sums(rs, acc, ez, et, on ? col0 + sub * 4 - cc : 4);
                    reduce_row_sums(rs, lpr_log2);
                    double* const o = row_sums + ((int64_t)blockIdx.y * n_out + r.z) * 3;
                    if (sub < 3) o[sub] = sub == 0 ? rs[0] : sub == 1 ? rs[1] : rs[2];
                    if (lpr < 3 && sub == 0)
                        for (int q = lpr; q < 3; ++q) o[q] = q == 1 ? rs[1] : rs[2];
                }
            }
        }
    }
    if constexpr (RANGE) {
        if (!is_part) {                                   // (every lane of the row's first group; off lanes hold its last columns)
            const float m = reduce_row_max(quad_max(acc), lpr_log2);
            const int n = reduce_row_counts(quad_counts(acc, m, on ? col0 + sub * 4 - cc : 4), lpr_log2);
            if (sub == 0) row_range[(int64_t)blockIdx.y * n_out + r.z] = range_word_of(m, n);
        }
    }
    if (!on) return;
    store_vec<VEC>(dst + cc, acc);
}

// Output rows with a single entry (most (row, neighbour community) segments of a sparse graph): row pos[k] of Y is
// val[k] times row col[k] of X.  A lane group takes kSingleBatch consecutive k, so that their index loads, their
// gathers and their stores are in flight together; the lists are read front to back.
constexpr int kSingleBatch = 4;
template <int VEC>
__global__ __launch_bounds__(256) void spmm_single_kernel(const int32_t* __restrict__ pos,
                                                          const int32_t* __restrict__ col,
                                                          const float* __restrict__ val, const float* __restrict__ X,
                                                          float* __restrict__ Y, int64_t n, int width, int lpr_log2,
                                                          const int32_t* __restrict__ gate) {
    if (gate && *gate == 0) return;
    const int lpr = 1 << lpr_log2;
    const int sub = threadIdx.x & (lpr - 1);
    const int64_t group = (int64_t)blockIdx.x * (256 >> lpr_log2) + (threadIdx.x >> lpr_log2);
    const int64_t k0 = group * kSingleBatch;
    if (k0 >= n) return;
    int32_t o[kSingleBatch], c[kSingleBatch];
    float a[kSingleBatch];
#pragma unroll
    for (int j = 0; j < kSingleBatch; ++j) {
        const int64_t k = k0 + j < n ? k0 + j : n - 1;
        o[j] = pos[k];
        c[j] = col[k];
        a[j] = val[k];
    }
    for (int c0 = sub * VEC; c0 < width; c0 += lpr * VEC) {
        const int cc = c0 + VEC <= width ? c0 : width - VEC;
        float x[kSingleBatch][VEC];
#pragma unroll
        for (int j = 0; j < kSingleBatch; ++j) load_vec<VEC>(x[j], X + (int64_t)c[j] * width + cc);
#pragma unroll
        for (int j = 0; j < kSingleBatch; ++j) {
            if (k0 + j >= n) break;
#pragma unroll
            for (int v = 0; v < VEC; ++v) x[j][v] *= a[j];
            store_vec<VEC>(Y + (int64_t)o[j] * width + cc, x[j]);
        }
    }
}

// Machine calibration for the aggregation: the gathers of a row list and nothing else.  Every lane group takes one
// chunk of the entry array (the real column stream, in the order the aggregation reads it: XCD k, the workgroups with
// blockIdx mod 8 = k, walks the k-th eighth front to back), gathers the eight rows the chunk names and adds them up;
// there are no row records, no reduction across lanes and no result rows (a lane stores only if its sum is a value
// that does not occur, which keeps the loads alive).  What this reaches is the rate at which the memory system serves
// this column stream's gathers of 4 * VEC * 2^lpr_log2 bytes.
template <int LPRL>
__global__ __launch_bounds__(256) void gather_calibration_kernel(const int2* __restrict__ ent, int64_t n_chunks,
                                                                 const float* __restrict__ X, int width, int lpr_log2_arg,
                                                                 float* __restrict__ out) {
    const int lpr_log2 = LPRL < 3 ? LPRL : lpr_log2_arg;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int k = blockIdx.x & 7;
    const int64_t per_xcd = (n_chunks + 7) / 8;
    const int64_t lo = 1 + k * per_xcd, hi = lo + per_xcd < n_chunks ? lo + per_xcd : n_chunks;   // chunk 0 is padding
    const int groups = 64 >> lpr_log2;
    const int64_t ch = lo + ((int64_t)(blockIdx.x >> 3) * 4 + wave) * groups + (lane >> lpr_log2);
    if (ch >= hi) return;                               // uniform over a lane group
    const int cc = (lane & ((1 << lpr_log2) - 1)) * 4;
    int32_t c[8];
    float a[8];
    load_chunk<LPRL>(ent, ch, lpr_log2, lane, c, a);
    float x[8][4];
#pragma unroll
    for (int u = 0; u < 8; ++u) load_vec<4>(x[u], X + (int64_t)c[u] * width + cc);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = fmaf(a[u], x[u][v], acc[v]);
    const float sum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    if (sum == 1.2345678e33f) out[threadIdx.x] = sum;
}

int g_tile_cols = 0;
int g_xcd_remap = 1;

// Adds the parts of every split row and applies the epilogue.  One wavefront per row: 2^lpr_log2 lanes cover the
// columns of the tile; where that leaves lanes over, the 64 >> lpr_log2 lane groups take the parts round-robin and
// their sums are added by xor-shuffles, so that a hub with a hundred parts is not one chain of dependent loads.
// The order of the additions is fixed by the part count alone.
template <int VEC, int EPI>
__global__ __launch_bounds__(64) void spmm_combine_kernel(const float* __restrict__ side,
                                                          const int32_t* __restrict__ long_row,
                                                          const int32_t* __restrict__ long_part_ptr, int64_t n_long,
                                                          float* __restrict__ Y, int width,
                                                          const float* __restrict__ Zl, const float* __restrict__ Tl,
                                                          float nu, int lpr_log2, double* __restrict__ row_sums,
                                                          uint32_t* __restrict__ row_range, int n_tiles, int64_t n_out, const int32_t* __restrict__ gate) {
    const int64_t i = blockIdx.x;
    if (i >= n_long || (gate && *gate == 0)) return;
    const int64_t row = long_row[i];
    const int p0 = long_part_ptr[i], p1 = long_part_ptr[i + 1];
    const int lpr = 1 << lpr_log2, groups = 64 >> lpr_log2;
    const int sub = threadIdx.x & (lpr - 1), grp = threadIdx.x >> lpr_log2;
    double rs[3] = {0.0, 0.0, 0.0};
    float most = 0.f;
    for (int cb = 0; cb < width; cb += lpr * VEC) {             // same trip count in every lane
        const bool ok = cb + sub * VEC < width;
        const int c = cb + sub * VEC + VEC <= width ? cb + sub * VEC : width - VEC;
        float acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
        if (ok) {
            for (int p = p0 + grp; p < p1; p += groups) {
                float x[VEC];
                load_vec<VEC>(x, side + (int64_t)p * width + c);
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] += x[v];
            }
        }
        for (int off = lpr; off < 64; off <<= 1) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] += __shfl_xor(acc[v], off, 64);
        }
        if (!ok || grp != 0) continue;
        const int64_t o = row * (int64_t)width + c;
        if constexpr (EPI == 1) {
            float z[VEC], t[VEC];
            load_vec<VEC>(z, Zl + o);
            load_vec<VEC>(t, Tl + o);
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = nu * (z[v] - fmaxf(t[v], 0.f)) + acc[v];
            if constexpr (VEC == 4) add_row_sums(rs, acc, z, t, cb + sub * VEC - c);
        }
        if constexpr (VEC == 4) most = fmaxf(most, quad_max(acc));
        store_vec<VEC>(Y + o, acc);
    }
    if constexpr (VEC == 4) {
        if (row_range && grp == 0) {                            // the whole row's in the first tile's place
            most = reduce_row_max(most, lpr_log2);
            int n = 0;
            for (int cb = 0; cb + sub * VEC < width; cb += lpr * VEC) {              // (each lane reads what it has stored)
                const int c = cb + sub * VEC + VEC <= width ? cb + sub * VEC : width - VEC;
                float v[4];
                load_vec<VEC>(v, Y + row * (int64_t)width + c);
                n += quad_counts(v, most, cb + sub * VEC - c);
            }
            n = reduce_row_counts(n, lpr_log2);
            for (int tile = sub; tile < n_tiles; tile += lpr) row_range[(int64_t)tile * n_out + row] = tile == 0 ? range_word_of(most, n) : 0u;
        }
    }
    if constexpr (EPI == 1 && VEC == 4) {
        if (row_sums && grp == 0) {                             // the whole row's sums in the first tile's place
            reduce_row_sums(rs, lpr_log2);
            for (int tile = sub; tile < n_tiles; tile += lpr)
#pragma unroll
                for (int q = 0; q < 3; ++q) row_sums[((int64_t)tile * n_out + row) * 3 + q] = tile == 0 ? rs[q] : 0.0;
        }
    }
}

// Columns per tile.  The rows of a community gather mostly rows of that community: 4 * columns * rows-of-a-community bytes
// are what an XCD's 4 MB L2 would have to hold for those gathers to hit.  The tile that fits is 256 columns (a whole wavefront
// of 16-byte loads per gathered row, which is also the most the kernel takes), halved until that holds, down to 32: the
// requests of narrower rows cost the L2 as much as those of 128 bytes, and the entries are read once more per tile.
// Chosen against 256 columns: 200000 nodes in 32 communities, width 512: 535 against 575 us (128 columns); 500000 in 16, width
// 512: 1381 against 1787 (32); 13752 in 3, width 1000: 129 against 172 (128).  At 4.1e6 bytes for 256 columns, just below the
// line, 64000 nodes in 16, width 512, take 141 us so and 147 in tiles of 128, but 12000 in 3, width 1000, 138 and 109.
// Two things can make the fewest tiles the faster way all the same.  A pass costs what its lanes per row cost, whether the
// tile fills them or not (200000 in 32, width 160: 157 us whole, 209 as 128 + 32; 287602 in 4, width 36: 111 and 154 as 32 +
// 4).  And where rows do not start on 128-byte lines a tile of every row straddles one line more (287602 in 4, width 230:
// 549 us whole, 856 in tiles of 32).  The rule counts columns: a straddled line as ten of them, and a quarter more for columns
// that do not fit (a tenth in tiles of up to 128, where a wavefront has two rows and more to wait for).  Against the best of
// the tiles tried it is within 7 % in 122 of 124 measurements, widths 30 to 1000 on nine graphs.
// The tiles of a launch are about equally wide (13752 in 8, width 257: 47 us as 132 + 125, 51 as 256 + 1), in whole lines
// or half lines where the rows are.
int tile_of(const SpmmSchedule& sc, int width, int vec, int most) {
    constexpr int kMost = 256;
    int fit = kMost;
    while (fit > 32 && 4.0 * fit * sc.group_rows > 4.5e6) fit >>= 1;
    const int unit = width % 32 == 0 ? 32 : width % 16 == 0 ? 16 : vec;
    auto even = [&](int tiles) { return ((width + tiles - 1) / tiles + unit - 1) / unit * unit; };
    const int few = (width + kMost - 1) / kMost;
    int tiles = (width + fit - 1) / fit;
    if (few < tiles) {
        const int line = width % 32 == 0 ? 0 : 10;
        if (20 * tiles * (fit + line) > (even(few) <= 128 ? 22 : 25) * few * (even(few) + line)) tiles = few;
    }
    int tile = even(tiles);
    if (most > 0 && most < tile) tile = (most + vec - 1) / vec * vec;
    return tile < width ? tile : width;
}

template <int VEC>
void launch_vec(hipStream_t s, const SpmmSchedule& sc, const float* X, float* Y, int width, const SpmmEpilogue& epi) {
    const int tile = tile_of(sc, width, VEC, g_tile_cols);
    const int lanes_needed = (tile + VEC - 1) / VEC;
    int lpr_log2 = 0;
    while ((1 << lpr_log2) < lanes_needed) ++lpr_log2;
    XcdMap xm;
    int64_t longest = 0;
    for (int k = 0; k <= 8; ++k) xm.start[k] = sc.xcd_start[lpr_log2][k];
    for (int k = 0; k < 8; ++k) longest = xm.start[k + 1] - xm.start[k] > longest ? xm.start[k + 1] - xm.start[k] : longest;
    const int64_t nb = g_xcd_remap ? 8 * longest : (sc.n_blocks[lpr_log2] + 7) / 8 * 8;       // (a multiple of 8 either way)
    if (nb > 0) {
        const dim3 grid((unsigned)nb, (unsigned)((width + tile - 1) / tile)), block(256);
        const bool off32 = sc.n_cols <= (1 << 24) && 4 * sc.n_cols * (int64_t)width <= ((int64_t)1 << 32);
#define CADMM_ROWS(L_) do { if (off32) CADMM_ROWS_OFF(L_, 1); else CADMM_ROWS_OFF(L_, 0); } while (0)
#define CADMM_ROWS_OFF(L_, O_) do { if (VEC == 4 && epi.row_range) CADMM_ROWS_EPI(L_, O_, (VEC == 4)); else CADMM_ROWS_EPI(L_, O_, 0); } while (0)
#define CADMM_ROWS_EPI(L_, O_, R_) do { \
        if (epi.kind == 1 && epi.gate) CADMM_ROWS_KERNEL(2, L_, O_, R_); \
        else if (epi.kind == 1) CADMM_ROWS_KERNEL(1, L_, O_, R_); \
        else CADMM_ROWS_KERNEL(0, L_, O_, R_); } while (0)
#define CADMM_ROWS_KERNEL(E_, L_, O_, R_) \
        hipLaunchKernelGGL((spmm_rows_kernel<VEC, E_, L_, O_, R_>), grid, block, 0, s, sc.rec, sc.n_rows, sc.ent, X, Y, sc.side, width, lpr_log2, \
                           sc.blocks[lpr_log2], xm, tile, g_xcd_remap, epi.Zl, epi.Tl, epi.nu, epi.row_sums, epi.row_range, sc.n_out, epi.gate)
        if (lpr_log2 == 0) CADMM_ROWS(0);
        else if (lpr_log2 == 1) CADMM_ROWS(1);
        else if (lpr_log2 == 2) CADMM_ROWS(2);
        else CADMM_ROWS(3);
#undef CADMM_ROWS
#undef CADMM_ROWS_OFF
#undef CADMM_ROWS_EPI
#undef CADMM_ROWS_KERNEL
    }
    if (sc.n_long > 0) {
        const dim3 grid((unsigned)sc.n_long), block(64);
        int clog2 = 0;                                       // lanes that cover the columns of a combined row
        while (clog2 < 6 && (VEC << clog2) < width) ++clog2;
        if (epi.kind == 1)
            hipLaunchKernelGGL((spmm_combine_kernel<VEC, 1>), grid, block, 0, s, sc.side, sc.long_row,
                               sc.long_part_ptr, sc.n_long, Y, width, epi.Zl, epi.Tl, epi.nu, clog2, epi.row_sums,
                               epi.row_range, (width + tile - 1) / tile, sc.n_out, epi.gate);
        else
            hipLaunchKernelGGL((spmm_combine_kernel<VEC, 0>), grid, block, 0, s, sc.side, sc.long_row,
                               sc.long_part_ptr, sc.n_long, Y, width, nullptr, nullptr, 0.f, clog2, nullptr, epi.row_range, (width + tile - 1) / tile, sc.n_out, epi.gate);
    }
}

}  // namespace

int spmm_tiles(const SpmmSchedule& sched, int width) {
    const int tile = tile_of(sched, width, 4, g_tile_cols);
    return (width + tile - 1) / tile;
}
int spmm_default_tiles(const SpmmSchedule& sched, int width) {
    const int tile = tile_of(sched, width, 4, 0);
    return (width + tile - 1) / tile;
}

void set_spmm_tile_cols(int cols) { g_tile_cols = cols > 0 ? cols : 0; }
void set_spmm_xcd_remap(int on) { g_xcd_remap = on ? 1 : 0; }

double launch_gather_calibration(hipStream_t s, const SpmmSchedule& sc, int64_t n_chunks, const float* X, int width,
                                 float* out) {
    int lpr_log2 = 0;
    while ((4 << lpr_log2) < width) ++lpr_log2;
    const int64_t per_xcd = (n_chunks + 7) / 8, per_block = 4 * (64 >> lpr_log2);
    dim3 grid((unsigned)(8 * ((per_xcd + per_block - 1) / per_block))), block(256);
    if (lpr_log2 == 0) hipLaunchKernelGGL((gather_calibration_kernel<0>), grid, block, 0, s, sc.ent, n_chunks, X, width, lpr_log2, out);
    else if (lpr_log2 == 1) hipLaunchKernelGGL((gather_calibration_kernel<1>), grid, block, 0, s, sc.ent, n_chunks, X, width, lpr_log2, out);
    else if (lpr_log2 == 2) hipLaunchKernelGGL((gather_calibration_kernel<2>), grid, block, 0, s, sc.ent, n_chunks, X, width, lpr_log2, out);
    else hipLaunchKernelGGL((gather_calibration_kernel<3>), grid, block, 0, s, sc.ent, n_chunks, X, width, lpr_log2, out);
    return (double)(n_chunks - 1) * 8.0 * (8.0 + 4.0 * width);       // the pairs and the rows they name
}

void launch_spmm(hipStream_t s, const SpmmSchedule& sched, const float* X, float* Y, int width, const SpmmEpilogue& epi) {
    if ((sched.n_rows <= 0 && sched.n_parts <= 0) || width <= 0) return;
    if (width >= 4) launch_vec<4>(s, sched, X, Y, width, epi);
    else launch_vec<1>(s, sched, X, Y, width, epi);
}

void launch_spmm_single(hipStream_t s, const int32_t* pos, const int32_t* col, const float* val, const float* X,
                        float* Y, int64_t n, int width, const int32_t* gate) {
    if (n <= 0 || width <= 0) return;
    const int vec = width >= 4 ? 4 : 1;
    const int lanes_needed = (width + vec - 1) / vec;
    int lpr_log2 = 0;
    while ((1 << lpr_log2) < lanes_needed && lpr_log2 < 6) ++lpr_log2;
    const int64_t groups = (n + kSingleBatch - 1) / kSingleBatch;
    const int64_t per_block = 256 >> lpr_log2;
    const int64_t nb = (groups + per_block - 1) / per_block;
    if (vec == 4) hipLaunchKernelGGL((spmm_single_kernel<4>), dim3((unsigned)nb), dim3(256), 0, s, pos, col, val, X, Y, n, width, lpr_log2, gate);
    else hipLaunchKernelGGL((spmm_single_kernel<1>), dim3((unsigned)nb), dim3(256), 0, s, pos, col, val, X, Y, n, width, lpr_log2, gate);
}

}  // namespace cadmm

// SpMM Y = A.X for each storage format (the aggregation of a GNN layer,
// Sec. 2.1; formats of Sec. 2.2).  fp32 in and out, fused multiply-add.
//
// This file: the generic kernels (CSR, ELL and DIA of fewer than four columns;
// BSR of any block size and width) and the per-format entry points.
//
// Shared layout of the kernels here: a "row group" of G lanes (G in {8,16,32,64},
// always inside one 64-wide wavefront) owns one output row slice of G*VEC
// columns, lane l holding columns l*VEC .. l*VEC+VEC-1 as one vector; X rows
// are gathered with one VEC-wide load per lane.  grid.y walks F in slices of
// G*VEC columns when F is wider.  Index/value streams are read once and are
// loaded cooperatively by the group (one entry per lane) and broadcast with
// cross-lane shuffles.
//
// Every sequential fp32 chain is bounded (at most 128 terms), which keeps the
// rounding error far below 1e-5 |A||X|; partial sums of split rows are combined
// in a fixed order, so results are deterministic.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "gs_device.h"
#include "gs_gather.h"
#include "gs_internal.h"

namespace gs {
namespace {

constexpr int kBlock = 256;  // threads per workgroup for every SpMM kernel

template <int VEC>
struct Acc {
    float v[VEC];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) v[i] = 0.0f;
    }
    __device__ __forceinline__ void fma(float a, const Vec<VEC> &x)
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) v[i] = __builtin_fmaf(a, x.v[i], v[i]);
    }
    __device__ __forceinline__ void add(const Acc &o)
    {
#pragma unroll
        for (int i = 0; i < VEC; i++) v[i] += o.v[i];
    }
    __device__ __forceinline__ Vec<VEC> vec() const
    {
        Vec<VEC> r;
#pragma unroll
        for (int i = 0; i < VEC; i++) r.v[i] = v[i];
        return r;
    }
};

// Accumulates sum_{k in [k0,k1)} val[k] * X[col[k], c0 .. c0+VEC) for one
// group.  Entries are fetched G at a time (one per lane) and broadcast;
// four independent accumulators keep four X-row loads in flight per lane.
template <int VEC, int G>
__device__ __forceinline__ Acc<VEC> gather_range(const int32_t *__restrict__ col,
                                                 const float *__restrict__ val, int64_t k0,
                                                 int64_t k1, const float *__restrict__ X,
                                                 int64_t ldx, int64_t c0, bool active, int lane)
{
    Acc<VEC> a0, a1, a2, a3;
    a0.zero();
    a1.zero();
    a2.zero();
    a3.zero();
    for (int64_t kb = k0; kb < k1; kb += G) {
        const int64_t k = kb + lane;
        int cj = 0;
        float vj = 0.0f;
        if (k < k1) {
            cj = ld_stream(col + k);
            vj = ld_stream(val + k);
        }
        const int n = (int)((k1 - kb) < G ? (k1 - kb) : G);
        int j = 0;
        for (; j + 4 <= n; j += 4) {
            const int c_0 = __shfl(cj, j, G), c_1 = __shfl(cj, j + 1, G);
            const int c_2 = __shfl(cj, j + 2, G), c_3 = __shfl(cj, j + 3, G);
            const float v_0 = __shfl(vj, j, G), v_1 = __shfl(vj, j + 1, G);
            const float v_2 = __shfl(vj, j + 2, G), v_3 = __shfl(vj, j + 3, G);
            if (active) {
                const Vec<VEC> x0 = ld_vec<VEC>(X + (int64_t)c_0 * ldx + c0);
                const Vec<VEC> x1 = ld_vec<VEC>(X + (int64_t)c_1 * ldx + c0);
                const Vec<VEC> x2 = ld_vec<VEC>(X + (int64_t)c_2 * ldx + c0);
                const Vec<VEC> x3 = ld_vec<VEC>(X + (int64_t)c_3 * ldx + c0);
                a0.fma(v_0, x0);
                a1.fma(v_1, x1);
                a2.fma(v_2, x2);
                a3.fma(v_3, x3);
            }
        }
        for (; j < n; j++) {
            const int c_0 = __shfl(cj, j, G);
            const float v_0 = __shfl(vj, j, G);
            if (active) a0.fma(v_0, ld_vec<VEC>(X + (int64_t)c_0 * ldx + c0));
        }
    }
    a0.add(a1);
    a2.add(a3);
    a0.add(a2);
    return a0;
}

// ---------------------------------------------------------------- CSR
// Generic path (any F and alignment): one group per work item {row, start,
// len, slot} of the CSR plan; slot >= 0 items are chunks of long rows whose
// partial sums go to work[slot * F + c].

template <int VEC, int G>
__global__ __launch_bounds__(kBlock) void k_csr_items_generic(
    int64_t n_items, const int4 *__restrict__ items, const int32_t *__restrict__ col,
    const float *__restrict__ val, const float *__restrict__ X, int64_t ldx, float *__restrict__ Y,
    int64_t ldy, int64_t F, float *__restrict__ work)
{
    constexpr int GPB = kBlock / G;
    const int g = threadIdx.x / G, lane = threadIdx.x % G;
    const int64_t cl = (int64_t)blockIdx.y * (G * VEC) + (int64_t)lane * VEC;
    const int64_t c0 = cl < F - VEC ? cl : F - VEC;  // a ragged width ends in a lane that overlaps the one before
    const bool active = cl < F;
    const int64_t it = (int64_t)blockIdx.x * GPB + g;
    if (it >= n_items) return;
    const int4 d = items[it];
    // rows of the group tier are summed kChainFold entries at a time
    Acc<VEC> acc;
    acc.zero();
    for (int64_t cs = d.y, e = (int64_t)d.y + d.z; cs < e; cs += kChainFold)
        acc.add(gather_range<VEC, G>(col, val, cs, cs + kChainFold < e ? cs + kChainFold : e, X, ldx, c0, active,
                                     lane));
    if (!active) return;
    if (d.w < 0)
        st_vec_stream<VEC>(Y + (int64_t)d.x * ldy + c0, acc.vec());
    else
        st_vec<VEC>(work + (int64_t)d.w * F + c0, acc.vec());
}

// One group per long row: sums its chunks' partials in chunk order.
template <int VEC, int G>
__global__ __launch_bounds__(kBlock) void k_csr_combine(const int32_t *__restrict__ long_rows,
                                                        const int32_t *__restrict__ long_first,
                                                        int64_t n_long, const float *__restrict__ work,
                                                        float *__restrict__ Y, int64_t ldy, int64_t F)
{
    constexpr int GPB = kBlock / G;
    const int g = threadIdx.x / G, lane = threadIdx.x % G;
    const int64_t cl = (int64_t)blockIdx.y * (G * VEC) + (int64_t)lane * VEC;
    const int64_t c0 = cl < F - VEC ? cl : F - VEC;  // a ragged width ends in a lane that overlaps the one before
    const int64_t lr = (int64_t)blockIdx.x * GPB + g;
    if (lr >= n_long || cl >= F) return;
    Acc<VEC> acc;
    acc.zero();
    for (int64_t ch = long_first[lr]; ch < long_first[lr + 1]; ch++) {
        const Vec<VEC> p = ld_vec<VEC>(work + ch * F + c0);
#pragma unroll
        for (int i = 0; i < VEC; i++) acc.v[i] += p.v[i];
    }
    st_vec_stream<VEC>(Y + (int64_t)long_rows[lr] * ldy + c0, acc.vec());
}

// ---------------------------------------------------------------- ELL
// One group per row; slot (i,k) lives at k*R + i, so for a fixed k the
// groups of a block read consecutive addresses.  Padding (col = -1) ends
// the row (entries are packed to the front).

template <int VEC, int G>
__global__ __launch_bounds__(kBlock) void k_ell(int64_t R, int64_t K, const int32_t *__restrict__ ec,
                                                const float *__restrict__ ev,
                                                const float *__restrict__ X, int64_t ldx,
                                                float *__restrict__ Y, int64_t ldy, int64_t F,
                                                int64_t n_tiles)
{
    constexpr int GPB = kBlock / G;
    const int g = threadIdx.x / G, lane = threadIdx.x % G;
    const int64_t cl = (int64_t)blockIdx.y * (G * VEC) + (int64_t)lane * VEC;
    const int64_t c0 = cl < F - VEC ? cl : F - VEC;  // a ragged width ends in a lane that overlaps the one before
    const bool active = cl < F;
    const int64_t row = xcd_tile(blockIdx.x, n_tiles) * GPB + g;
    if (row >= R) return;
    const int gbase = (threadIdx.x % kWave) / G * G;
    Acc<VEC> a0, a1, tot;
    a0.zero();
    a1.zero();
    tot.zero();
    for (int64_t kb = 0; kb < K; kb += G) {
        if (kb > 0 && kb % kChainFold == 0) {  // fold the running chains every kChainFold slots
            tot.add(a0);
            tot.add(a1);
            a0.zero();
            a1.zero();
        }
        const int64_t k = kb + lane;
        int cj = -1;
        float vj = 0.0f;
        if (k < K) {
            cj = ld_stream(ec + k * R + row);
            vj = ld_stream(ev + k * R + row);
        }
        // entries are packed to the front: the stored ones form a prefix
        const unsigned long long live =
            (__ballot(cj >= 0) >> gbase) & (G == 64 ? ~0ull : ((1ull << G) - 1));
        const int n = __popcll(live);
        int j = 0;
        for (; j + 2 <= n; j += 2) {
            const int c_0 = __shfl(cj, j, G), c_1 = __shfl(cj, j + 1, G);
            const float v_0 = __shfl(vj, j, G), v_1 = __shfl(vj, j + 1, G);
            if (active) {
                const Vec<VEC> x0 = ld_vec<VEC>(X + (int64_t)c_0 * ldx + c0);
                const Vec<VEC> x1 = ld_vec<VEC>(X + (int64_t)c_1 * ldx + c0);
                a0.fma(v_0, x0);
                a1.fma(v_1, x1);
            }
        }
        if (j < n) {
            const int c_0 = __shfl(cj, j, G);
            const float v_0 = __shfl(vj, j, G);
            if (active) a0.fma(v_0, ld_vec<VEC>(X + (int64_t)c_0 * ldx + c0));
        }
        if (n < G) break;
    }
    tot.add(a0);
    tot.add(a1);
    if (active) st_vec_stream<VEC>(Y + row * ldy + c0, tot.vec());
}

// ---------------------------------------------------------------- DIA
// One group per row; diagonal d contributes data[d*R+i] * X[i + off_d].
// Padding slots hold +0 and are skipped, as are columns outside [0, C).

template <int VEC, int G>
__global__ __launch_bounds__(kBlock) void k_dia(int64_t R, int64_t C, int64_t ND,
                                                const int32_t *__restrict__ offsets,
                                                const float *__restrict__ data,
                                                const float *__restrict__ X, int64_t ldx,
                                                float *__restrict__ Y, int64_t ldy, int64_t F,
                                                int64_t n_tiles)
{
    constexpr int GPB = kBlock / G;
    const int g = threadIdx.x / G, lane = threadIdx.x % G;
    const int64_t cl = (int64_t)blockIdx.y * (G * VEC) + (int64_t)lane * VEC;
    const int64_t c0 = cl < F - VEC ? cl : F - VEC;  // a ragged width ends in a lane that overlaps the one before
    const bool active = cl < F;
    const int64_t row = xcd_tile(blockIdx.x, n_tiles) * GPB + g;
    if (row >= R) return;
    Acc<VEC> a0, a1, tot;
    a0.zero();
    a1.zero();
    tot.zero();
    int64_t d = 0;
    for (; d + 2 <= ND; d += 2) {
        if (d > 0 && d % kChainFold == 0) {  // fold the running chains every kChainFold diagonals
            tot.add(a0);
            tot.add(a1);
            a0.zero();
            a1.zero();
        }
        const int64_t j0 = row + offsets[d], j1 = row + offsets[d + 1];
        const float v0 = ld_stream(data + d * R + row);
        const float v1 = ld_stream(data + (d + 1) * R + row);
        if (active) {
            if (v0 != 0.0f && j0 >= 0 && j0 < C) a0.fma(v0, ld_vec<VEC>(X + j0 * ldx + c0));
            if (v1 != 0.0f && j1 >= 0 && j1 < C) a1.fma(v1, ld_vec<VEC>(X + j1 * ldx + c0));
        }
    }
    if (d < ND) {
        const int64_t j0 = row + offsets[d];
        const float v0 = ld_stream(data + d * R + row);
        if (active && v0 != 0.0f && j0 >= 0 && j0 < C) a0.fma(v0, ld_vec<VEC>(X + j0 * ldx + c0));
    }
    tot.add(a0);
    tot.add(a1);
    if (active) st_vec_stream<VEC>(Y + row * ldy + c0, tot.vec());
}

// ---------------------------------------------------------------- BSR
// One workgroup per block row.  Lanes split F as everywhere else; the
// kBlock/G row groups split the b rows of the block row (each thread owns
// up to RPT rows).  Each b x b block is staged in LDS; only the block
// columns with a nonzero (bit set in the block's column mask) gather their
// X row, so a sparse block costs its b*b values plus its touched X rows.

template <int VEC, int G, int RPT>
__global__ __launch_bounds__(kBlock) void k_bsr(int64_t R, int64_t C, int b, int64_t nbr,
                                                const int32_t *__restrict__ bptr,
                                                const int32_t *__restrict__ bcol,
                                                const float *__restrict__ bval,
                                                const uint64_t *__restrict__ bmask,
                                                const float *__restrict__ X, int64_t ldx,
                                                float *__restrict__ Y, int64_t ldy, int64_t F)
{
    constexpr int RG = kBlock / G;  // row groups
    __shared__ float blk_lds[64 * 64];
    const int g = threadIdx.x / G, lane = threadIdx.x % G;
    const int64_t cl = (int64_t)blockIdx.y * (G * VEC) + (int64_t)lane * VEC;
    const int64_t c0 = cl < F - VEC ? cl : F - VEC;  // a ragged width ends in a lane that overlaps the one before
    const bool active = cl < F;
    const int64_t br = xcd_tile(blockIdx.x, nbr);
    const int bb = b * b;
    Acc<VEC> acc[RPT], tot[RPT];
#pragma unroll
    for (int r = 0; r < RPT; r++) {
        acc[r].zero();
        tot[r].zero();
    }
    const int64_t fold = kChainFold / b > 0 ? kChainFold / b : 1;  // blocks per running chain
    for (int64_t blk = bptr[br]; blk < bptr[br + 1]; blk++) {
        if (blk > bptr[br] && (blk - bptr[br]) % fold == 0) {
#pragma unroll
            for (int r = 0; r < RPT; r++) {
                tot[r].add(acc[r]);
                acc[r].zero();
            }
        }
        __syncthreads();
        for (int t = threadIdx.x; t < bb; t += kBlock) blk_lds[t] = ld_stream(bval + blk * bb + t);
        __syncthreads();
        uint64_t mask = bmask[blk];
        const int64_t xc = (int64_t)bcol[blk] * b;
        while (mask) {
            const int j = __ffsll((unsigned long long)mask) - 1;
            mask &= mask - 1;
            if (!active) continue;
            const Vec<VEC> x = ld_vec<VEC>(X + (xc + j) * ldx + c0);
#pragma unroll
            for (int r = 0; r < RPT; r++) {
                const int rr = g + r * RG;
                if (rr < b) acc[r].fma(blk_lds[rr * b + j], x);
            }
        }
    }
    if (!active) return;
#pragma unroll
    for (int r = 0; r < RPT; r++) {
        tot[r].add(acc[r]);
        const int rr = g + r * RG;
        const int64_t row = br * b + rr;
        if (rr < b && row < R) st_vec_stream<VEC>(Y + row * ldy + c0, tot[r].vec());
    }
}

// ----------------------------------------------------------- dispatch

struct Shape {
    int vec;
    int g;
    int64_t fslices;  // grid.y
};

// Lanes of a group of the kernels for fewer than four columns (CSR, ELL, DIA),
// one column per lane.
constexpr int kNarrow = 8;

// BSR: four columns per lane from F = 4 on (any alignment, see Quads), one below.
Shape pick_shape(int64_t F)
{
    const int vec = F >= 4 ? 4 : 1;
    const int64_t lanes = ceil_div(F, vec);
    const int g = lanes <= 8 ? 8 : lanes <= 16 ? 16 : lanes <= 32 ? 32 : 64;
    return Shape{vec, g, ceil_div(F, (int64_t)g * vec)};
}

// Calls fn.template operator()<VEC, G>() for the runtime (vec, g).
template <class Fn>
void dispatch(const Shape &sh, Fn &&fn)
{
#define GS_CASE(V, GG) \
    if (sh.vec == V && sh.g == GG) return fn.template operator()<V, GG>();
    GS_CASE(4, 8) GS_CASE(4, 16) GS_CASE(4, 32) GS_CASE(4, 64)
    GS_CASE(1, 8)
#undef GS_CASE
    fail(GS_ERR_UNSUPPORTED, "no kernel for vec=%d g=%d", sh.vec, sh.g);
}

unsigned u32_grid(int64_t n)
{
    if (n > 0x7fffffffll) fail(GS_ERR_UNSUPPORTED, "grid of %lld workgroups is too large", (long long)n);
    return (unsigned)(n < 1 ? 1 : n);
}

}  // namespace

// --------------------------------------------------------------- launchers

void spmm_csr(gs_matrix_ &m, const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t F,
              hipStream_t s, const WorkArea *fixed)
{
    if (!m.csr_planned) {
        if (fixed) fail(GS_ERR_UNSUPPORTED, "CSR handle without a work plan (it is built with the handle)");
        plan_csr(m, s);
    }
    if (spmm_csr_vec4(m, X, ldx, Y, ldy, F, s, fixed)) return;
    // fewer than four columns
    constexpr int GPB = kBlock / kNarrow;
    float *work = m.n_long_chunks ? (float *)work_for(m, fixed, (size_t)m.n_long_chunks * F * 4, s) : nullptr;
    if (m.n_items) {
        k_csr_items_generic<1, kNarrow><<<u32_grid(ceil_div(m.n_items, GPB)), kBlock, 0, s>>>(
            m.n_items, m.csr_items.as<int4>(), m.col.as<int32_t>(), m.val.as<float>(), X, ldx, Y, ldy, F, work);
        GS_HIP(hipGetLastError());
    }
    if (m.n_long_rows) {
        k_csr_combine<1, kNarrow><<<u32_grid(ceil_div(m.n_long_rows, GPB)), kBlock, 0, s>>>(
            m.long_rows.as<int32_t>(), m.long_first.as<int32_t>(), m.n_long_rows, work, Y, ldy, F);
        GS_HIP(hipGetLastError());
    }
}

// COO: the entries are in row order, so their column and value arrays are
// those of the CSR form and the row kernel reads them as they are, by the row
// pointers and the row plan that the handle keeps beside them.  (Equal ranges
// of entries with a segmented sum, the schedule this replaces, took 43.7 us on
// the power-law graph at F = 64 against 33.7 us, 247 against 191 us on the
// block graph and 3.41 against 2.89 ms on the 2M-row graph: cut rows went
// through carry slots and a second launch.  The plan is made with the handle:
// building the power-law graph takes 248 us, without it 167.)
void spmm_coo(gs_matrix_ &m, const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t F,
              hipStream_t s, const WorkArea *fixed)
{
    if (fixed) fail(GS_ERR_UNSUPPORTED, "COO handles are not supported without allocation");
    spmm_csr(m, X, ldx, Y, ldy, F, s, fixed);
}

// CSC: rows gathered from the handle's row form, the products summed in fp64
// (they are exact there) and rounded once.  Scattering the columns into an
// R x F fp64 accumulator with atomics, which this replaces, took 781 us on the
// power-law graph at F = 64 (180 billion atomics a second) against 37 us.
// Without allocation 8 R F bytes stay the limit that the interface states (they
// were the accumulator's), though partial sums of long rows are all that is
// kept now.
void spmm_csc(gs_matrix_ &m, const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t F,
              hipStream_t s, const WorkArea *fixed)
{
    if (fixed) (void)work_for(m, fixed, (size_t)(m.R * F) * 8, s);
    spmm_rows_f64(*m.by_rows, X, ldx, Y, ldy, F, s, fixed);
}

void spmm_ell(gs_matrix_ &m, const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t F,
              hipStream_t s)
{
    if (spmm_ell_fast(m, X, ldx, Y, ldy, F, s)) return;
    const int64_t tiles = ceil_div(m.R, kBlock / kNarrow);  // fewer than four columns
    k_ell<1, kNarrow><<<u32_grid(tiles), kBlock, 0, s>>>(m.R, m.K, m.ell_col.as<int32_t>(), m.ell_val.as<float>(), X,
                                                         ldx, Y, ldy, F, tiles);
    GS_HIP(hipGetLastError());
}

void spmm_dia(gs_matrix_ &m, const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t F,
              hipStream_t s)
{
    if (spmm_dia_fast(m, X, ldx, Y, ldy, F, s)) return;
    const int64_t tiles = ceil_div(m.R, kBlock / kNarrow);  // fewer than four columns
    k_dia<1, kNarrow><<<u32_grid(tiles), kBlock, 0, s>>>(m.R, m.C, m.ND, m.offsets.as<int32_t>(), m.dia.as<float>(), X,
                                                         ldx, Y, ldy, F, tiles);
    GS_HIP(hipGetLastError());
}

void spmm_bsr(gs_matrix_ &m, const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t F,
              hipStream_t s)
{
    if (spmm_bsr16_mfma(m, X, ldx, Y, ldy, F, s)) return;
    const Shape sh = pick_shape(F);
    const int64_t nbr = ceil_div(m.R, m.b);
    if (!nbr) return;
    dispatch(sh, [&]<int VEC, int G>() {
        constexpr int RG = kBlock / G;
        const int rpt = (int)ceil_div(m.b, RG);
        dim3 grid(u32_grid(nbr), (unsigned)sh.fslices);
        auto go = [&](auto rpt_tag) {
            constexpr int RPT = decltype(rpt_tag)::value;
            k_bsr<VEC, G, RPT><<<grid, kBlock, 0, s>>>(m.R, m.C, m.b, nbr, m.bptr.as<int32_t>(),
                                                       m.bcol.as<int32_t>(), m.bval.as<float>(),
                                                       m.bmask.as<uint64_t>(), X, ldx, Y, ldy, F);
        };
        if (rpt <= 1) go(std::integral_constant<int, 1>{});
        else if (rpt <= 2) go(std::integral_constant<int, 2>{});
        else if (rpt <= 4) go(std::integral_constant<int, 4>{});
        else if (rpt <= 8) go(std::integral_constant<int, 8>{});
        else go(std::integral_constant<int, 16>{});
        GS_HIP(hipGetLastError());
    });
}

}  // namespace gs

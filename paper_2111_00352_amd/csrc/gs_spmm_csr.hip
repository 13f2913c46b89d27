// CSR SpMM, vectorised path (F of 4 and more).
//
// Work is cut at plan time into three tiers by row length:
//  * short rows (at most `long_thr` entries): one group of G lanes per row;
//    for skewed lengths (power-law graphs) ordered by decreasing length, so
//    a wavefront's groups have equal trip counts and the longest start first,
//    otherwise in natural order (neighbouring rows share X rows in L2);
//  * medium rows (up to `wg_thr` entries): one workgroup per row; its groups
//    take interleaved chunks of `chunk` entries, each summed in fresh
//    registers, and the groups' partial rows are added in LDS in group order;
//  * huge rows: chunks spread over many workgroups as independent items whose
//    partial sums a second, small launch adds in slot order.
// Every sequential fp32 chain stays within `chunk` terms and every combine
// runs in a fixed order, so results are deterministic.
//
// Lane layout: lane l of a group holds column quad q at c0 + 4*G*q, so one load
// instruction reads G*16 contiguous bytes of an X row; a width that is no
// multiple of 4 ends in a quad that overlaps the one before.  Entries are
// fetched 16 or 32 at a time (a whole wave: 64), one per lane, a batch ahead,
// and broadcast by DPP (a whole wave: from scalar registers); X rows are
// gathered several at a time before any is consumed, the last of them only up
// to the row's end.  The grid is persistent (a few workgroups per CU),
// long-row tiles first.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <numeric>
#include <string>
#include <vector>

#include "gs_device.h"
#include "gs_gather.h"
#include "gs_internal.h"

namespace gs {
namespace {

constexpr int kBlock = 256;

// Candidate row tiles of the LDS-staged kernel: 32 << k rows, k < kWinCands,
// each with halo 0 and 1.
constexpr int kWinCands = 4;

// The group's next batch of entries: [k, k + n) of the entry arrays, one per
// lane and register (every 16 lanes of a group of 32 load the same 16).  Lanes
// past the last entry hold a valid column and the value -0.
template <int G, int NB, int OFF, bool CLS> struct Batch {
    int c[NB];
    float v[NB];
    // (zlast: the matrix's last entry, read in the place of an empty row's)
    __device__ __forceinline__ void load(const int32_t *__restrict__ col, const float *__restrict__ val, int k, int n,
                                         int zlast, int lane)
    {
#pragma unroll
        for (int r = 0; r < NB; r++) {
            const int e = lane % kEntryReg<G> + r * kEntryReg<G>;
            int i = k + (e < n ? e : n > 0 ? n - 1 : 0);
            i = i < zlast ? i : zlast;
            c[r] = ld_stream(col + i);
            v[r] = ld_stream(val + i);
            if (e >= n) v[r] = -0.0f;
        }
    }
    __device__ __forceinline__ void refs(int64_t ldx, int hot_cls, RowRef<OFF> *ref, int *cold) const
    {
#pragma unroll
        for (int r = 0; r < NB; r++) {
            ref[r].set(CLS ? (c[r] & kColMask) : c[r], ldx);
            cold[r] = CLS ? (c[r] >> kColClassShift) < hot_cls : 0;
        }
    }
};

// Accumulates the n entries from k0 on into acc, the next batch's
// entries requested while the current one's X rows are gathered.
template <int NQ, int G, int NB, int U, int OFF, bool CLS, int NA, class Q, class A>
__device__ __forceinline__ void gather_span(const int32_t *__restrict__ col, const float *__restrict__ val, int k0,
                                            int n, int zlast, const float *__restrict__ X, int64_t ldx, const Q &cols,
                                            int lane, int hot_cls, A *acc)
{
    constexpr int EB = kEntryBatch<G, NB>;
    Batch<G, NB, OFF, CLS> b;
    b.load(col, val, k0, n < EB ? n : EB, zlast, lane);
    for (int kb = 0; kb < n; kb += EB) {
        const int left = n - kb;
        RowRef<OFF> ref[NB];
        int cold[NB];
        b.refs(ldx, hot_cls, ref, cold);
        float v[NB];
#pragma unroll
        for (int r = 0; r < NB; r++) v[r] = b.v[r];
        const int nl = left > EB ? left - EB : 0;
        b.load(col, val, k0 + kb + (left > EB ? EB : 0), nl < EB ? nl : EB, zlast, lane);
        gather_entries_of<0, U, NQ, G, NB, OFF, CLS, NA>(ref, v, cold, left < EB ? left : EB, X, cols, acc);
    }
}

// What a row kernel is compiled for, beside its lane shape:
//  A        the accumulator type (double: the products are summed exactly
//           enough that one rounding to fp32 is the only one that matters)
//  CLS      columns carry their reference class
//  GROUPED  the plan's group tier is active, so items may be rows of up to the
//           group limit, folded every kChainFold entries
//  DEPTH    X rows in flight per lane group where it is not 8 of CPL = 4 (8
//           float4 loads a lane; 4 where registers or L2 lines are short: fp64
//           sums, class gathers)
//  NA       2: chains of four entries that join two sums in turn, 1: one chain
//  NB       registers of entries per batch
template <class A_, bool CLS_, bool GROUPED_, int DEPTH_ = 0, int NA_ = 1, int NB_ = 1> struct RowVariant {
    typedef A_ A;
    static constexpr bool CLS = CLS_, GROUPED = GROUPED_;
    static constexpr int DEPTH = DEPTH_, NA = NA_, NB = NB_;
};

// Bound by the L2 fills of the gathered X rows (7.3 TB/s) where X exceeds the
// L2s, by the L2's gather rate (16 TB/s) where it does not, and on small
// matrices by the chain item -> entries -> X rows: a lane group runs its items
// in a software pipeline, holding the next item's descriptor and first batch
// of entries while it gathers the current one's X rows, and broadcasts entries
// by DPP (no LDS round trip).  Against shuffled batches of G entries without
// the pipeline: power-law graph (F = 128) 61.6 -> 60.2 us, block graph
// (F = 256) 199 -> 191, a 30,011 x 100,003 block of 450,000 entries at F = 47
// 23.1 -> 20.3.
//
template <int CPL, int G, bool FULL, int OFF, class V>
__global__ __launch_bounds__(kBlock) void k_csr_rows(
    int64_t n_long, const int32_t *__restrict__ long_rows, const int32_t *__restrict__ rp, int chunk, int64_t n_items,
    const int4 *__restrict__ items, const int32_t *__restrict__ col, const float *__restrict__ val, int zlast,
    const float *__restrict__ X, int64_t ldx, float *__restrict__ Y, int64_t ldy, int64_t F,
    typename V::A *__restrict__ work, int hot_cls, int by_xcd)
{
    typedef typename V::A A;
    constexpr bool CLS = V::CLS, GROUPED = V::GROUPED;
    constexpr int NA = V::NA, NB = V::NB;
    constexpr int GPB = kBlock / G;
    constexpr int NQ = CPL / 4;
    constexpr int EB = kEntryBatch<G, NB>;
    constexpr int U0 = V::DEPTH ? V::DEPTH : CLS || sizeof(A) == 8 ? 4 : 32 / CPL > 0 ? 32 / CPL : 1;
    constexpr int U = U0 < EB ? U0 : EB;
    typedef typename Quad<A>::type A4;
    __shared__ A4 part[GPB][G * NQ];
    const int g = threadIdx.x / G, lane = threadIdx.x % G;
    const Quads<NQ, G, FULL> cols((int64_t)blockIdx.y * (G * CPL), lane, F);

    // long rows first, a workgroup each.  Tiles in launch order: giving each
    // XCD neighbouring rows, so that they share X rows in its L2, made a mesh
    // of 512 x 512 slower (F = 128 77 against 59 us) and 140,001 rows of 20
    // entries (F = 128 168 against 131).  Only fp64 tiles of four rows, less
    // than a community, gain by it (by_xcd; block graph at F = 256 264 -> 248).
    int64_t t = blockIdx.x;
    if constexpr (G == 64 && sizeof(A) == 8)
        if (by_xcd) t = xcd_tile(blockIdx.x, gridDim.x);
    for (; t < n_long; t += gridDim.x) {
        const int64_t row = long_rows[t];
        const int64_t s = rp[row], e = rp[row + 1];
        // pieces of at most `chunk` entries, shorter where that gives every group one
        const int even = (int)((e - s + GPB - 1) / GPB + 15) / 16 * 16, piece = even < chunk ? even : chunk;
        A acc[CPL];
#pragma unroll
        for (int i = 0; i < CPL; i++) acc[i] = 0;
        for (int64_t cs = s + (int64_t)g * piece; cs < e; cs += (int64_t)GPB * piece) {
            A part_acc[NA * CPL];
#pragma unroll
            for (int i = 0; i < NA * CPL; i++) part_acc[i] = 0;
            gather_span<NQ, G, NB, U, OFF, CLS, NA>(col, val, (int)cs, e - cs < piece ? (int)(e - cs) : piece, zlast, X,
                                                    ldx, cols, lane, hot_cls, part_acc);
            add_sums<NA, CPL>(part_acc);
#pragma unroll
            for (int i = 0; i < CPL; i++) acc[i] += part_acc[i];
        }
#pragma unroll
        for (int q = 0; q < NQ; q++)
            part[g][q * G + lane] = A4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        __syncthreads();
        if (g == 0) {
#pragma unroll
            for (int q = 0; q < NQ; q++) {
                A4 a = part[0][q * G + lane];
#pragma unroll 4
                for (int gg = 1; gg < GPB; gg++) a += part[gg][q * G + lane];
#pragma unroll
                for (int i = 0; i < 4; i++) acc[4 * q + i] = a[i];
            }
            store_quads_stream<NQ>(Y + row * ldy, cols, acc);
        }
        __syncthreads();  // part[] is reused by the next long row
    }

    // items: the tiles after the long rows, GPB items each.  The next item and
    // its first entries are requested without a test, where there is none the
    // last ones again: tests in the inner loop cost more than they save (3,302
    // rows of 165 entries at F = 64 15.9 against 17.4 us).
    const int64_t stride = (int64_t)gridDim.x * GPB;
    int64_t it = (t - n_long) * GPB + g;
    if (it >= n_items) return;
    const int64_t last = n_items - 1;
    int4 d = items[it];
    int4 dn = items[it + stride < last ? it + stride : last];
    Batch<G, NB, OFF, CLS> b;
    b.load(col, val, d.y, d.z < EB ? d.z : EB, zlast, lane);
    while (true) {
        A acc[NA * CPL], tot[GROUPED ? CPL : 1];
#pragma unroll
        for (int i = 0; i < NA * CPL; i++) acc[i] = 0;
        if constexpr (GROUPED) {
#pragma unroll
            for (int i = 0; i < CPL; i++) tot[i] = 0;
        }
        for (int kb = 0;; kb += EB) {
            const int left = d.z - kb;
            const bool more = left > EB;
            RowRef<OFF> ref[NB];
            int cold[NB];
            b.refs(ldx, hot_cls, ref, cold);
            float v[NB];
#pragma unroll
            for (int r = 0; r < NB; r++) v[r] = b.v[r];
            // the next batch: of this row, or the next item's first
            const int nk = more ? d.y + kb + EB : dn.y, nn = more ? left - EB : dn.z;
            b.load(col, val, nk, nn < EB ? nn : EB, zlast, lane);
            gather_entries_of<0, U, NQ, G, NB, OFF, CLS, NA>(ref, v, cold, left < EB ? left : EB, X, cols, acc);
            if constexpr (GROUPED) {
                if ((kb + EB) % kChainFold == 0) {
                    add_sums<NA, CPL>(acc);
#pragma unroll
                    for (int i = 0; i < CPL; i++) tot[i] += acc[i];
#pragma unroll
                    for (int i = 0; i < NA * CPL; i++) acc[i] = 0;
                }
            }
            if (!more) break;
        }
        add_sums<NA, CPL>(acc);
        if constexpr (GROUPED) {
#pragma unroll
            for (int i = 0; i < CPL; i++) acc[i] = tot[i] + acc[i];
        }
        // (the empty asm statements keep the compiler from merging the branches'
        // stores into ones that have lost the non-temporal hint: a 512 x 512
        // mesh at F = 128 took 65 us against 59)
        if (d.w < 0) {
            asm volatile("");
            store_quads_stream<NQ>(Y + (int64_t)d.x * ldy, cols, acc);
            asm volatile("");
        } else {  // a chunk of a huge row: its partial sum, added later in slot order
            store_quads<NQ>(work + (int64_t)d.w * F, cols, acc);
        }
        it += stride;
        if (it >= n_items) break;
        d = dn;
        dn = items[it + stride < last ? it + stride : last];
    }
}

// One group per huge row: adds the row's chunk partials (consecutive slots)
// in slot order, sixteen float4 per lane in flight, and writes the row of Y.
template <int CPL, int G, class A>
__global__ __launch_bounds__(kBlock) void k_csr_combine(const int32_t *__restrict__ rows,
                                                        const int32_t *__restrict__ first,
                                                        int64_t n, const A *__restrict__ work,
                                                        float *__restrict__ Y, int64_t ldy, int64_t F)
{
    constexpr int GPB = kBlock / G;
    constexpr int NQ = CPL / 4;
    typedef typename Quad<A>::type A4;
    const int g = threadIdx.x / G, lane = threadIdx.x % G;
    const int64_t r = (int64_t)blockIdx.x * GPB + g;
    if (r >= n) return;
    const Quads<NQ, G, false> cols((int64_t)blockIdx.y * (G * CPL), lane, F);
    A acc[CPL];
#pragma unroll
    for (int i = 0; i < CPL; i++) acc[i] = 0;
    const int64_t s0 = first[r], s1 = first[r + 1];
    // B partials in flight, summed as a tree (zeros past the last) before
    // they join the running sum: a row of n chunks adds log2(B) + n / B terms
    // in sequence
    constexpr int B = (NQ >= 4 ? 4 : NQ == 2 ? 8 : 16) / (sizeof(A) / 4);  // 16 float4 of partials per lane
    for (int64_t sl = s0; sl < s1; sl += B) {
        A4 p[B][NQ];
#pragma unroll
        for (int u = 0; u < B; u++)
#pragma unroll
            for (int q = 0; q < NQ; q++) {
                p[u][q] = A4{0, 0, 0, 0};
                if (sl + u < s1)
                    p[u][q] = *reinterpret_cast<const A4 *>(work + (sl + u) * F + cols.base(q) + cols.step(q));
            }
#pragma unroll
        for (int w = 1; w < B; w <<= 1)
#pragma unroll
            for (int u = 0; u < B; u += 2 * w)
#pragma unroll
                for (int q = 0; q < NQ; q++) p[u][q] += p[u + w][q];
#pragma unroll
        for (int q = 0; q < NQ; q++)
#pragma unroll
            for (int i = 0; i < 4; i++) acc[4 * q + i] += p[0][q][i];
    }
    store_quads_stream<NQ>(Y + (int64_t)rows[r] * ldy, cols, acc);
}

// Widths below 4, in fp64: a wave per item of the plan (or, without items, per
// row), its lanes over the entries, one sum per column.  Chunks of long rows
// go to work[slot * F + c].
__global__ __launch_bounds__(kBlock) void k_rows_f64_narrow(int64_t n, const int4 *__restrict__ items,
                                                            const int32_t *__restrict__ rp,
                                                            const int32_t *__restrict__ col,
                                                            const float *__restrict__ val, const float *__restrict__ X,
                                                            int64_t ldx, float *__restrict__ Y, int64_t ldy, int F,
                                                            double *__restrict__ work)
{
    const int lane = threadIdx.x % kWave;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave; i < n; i += waves) {
        int4 d;
        if (items)
            d = items[i];
        else
            d = make_int4((int)i, rp[i], rp[i + 1] - rp[i], -1);
        double a[3] = {0.0, 0.0, 0.0};
        for (int k = lane; k < d.z; k += kWave) {
            const double v = val[d.y + k];
            const float *x = X + (int64_t)col[d.y + k] * ldx;
            for (int c = 0; c < F; c++) a[c] = __builtin_fma(v, (double)x[c], a[c]);
        }
        for (int c = 0; c < F; c++) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) a[c] += __shfl_xor(a[c], o, kWave);
            if (lane != 0) continue;
            if (d.w < 0)
                Y[(int64_t)d.x * ldy + c] = (float)a[c];
            else
                work[(int64_t)d.w * F + c] = a[c];
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_combine_f64_narrow(int64_t n, const int32_t *__restrict__ rows,
                                                               const int32_t *__restrict__ first,
                                                               const double *__restrict__ work,
                                                               float *__restrict__ Y, int64_t ldy, int F)
{
    const int64_t r = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
    const int lane = threadIdx.x % kWave;
    if (r >= n) return;
    for (int c = 0; c < F; c++) {
        double a = 0.0;
        for (int64_t sl = first[r] + lane; sl < first[r + 1]; sl += kWave) a += work[sl * F + c];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, kWave);
        if (lane == 0) Y[(int64_t)rows[r] * ldy + c] = (float)a;
    }
}

// Row tiles with their X window staged in LDS (natural row order, rows of at
// most the short-row limit).  A workgroup takes T consecutive rows [r0, r1)
// and first copies the X rows [r0 - halo, r1 + halo) of its column slice
// into LDS with coalesced loads; its groups then run the rows as the plain
// kernel does, reading every entry whose column lies in the window from LDS
// and the others from global memory.  Graphs whose edges stay mostly inside
// such tiles (communities of consecutive nodes, stencils) then gather most
// X rows once per tile instead of once per entry through L2.
template <int CPL, int G, bool FULL>
__global__ __launch_bounds__(kBlock) void k_csr_window(
    int64_t R, int64_t C, const int32_t *__restrict__ rp, const int32_t *__restrict__ col,
    const float *__restrict__ val, const float *__restrict__ X, int64_t ldx, float *__restrict__ Y,
    int64_t ldy, int64_t F, int T, int halo, int64_t ntiles)
{
    constexpr int GPB = kBlock / G;
    constexpr int NQ = CPL / 4;
    constexpr int RW = G * NQ;  // float4 per staged row
    constexpr int B0 = 32 / CPL > 0 ? 32 / CPL : 1;
    constexpr int B = B0 < G ? B0 : G;  // X rows in flight per batch
    extern __shared__ float4 xs[];
    const int g = threadIdx.x / G, lane = threadIdx.x % G;
    const int64_t cbase = (int64_t)blockIdx.y * (G * CPL);
    const Quads<NQ, G, FULL> cols(cbase, lane, F);

    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t r0 = t * T, r1 = r0 + T < R ? r0 + T : R;
        const int64_t w0 = r0 - halo > 0 ? r0 - halo : 0;
        const int64_t w1 = r1 + halo < C ? r1 + halo : C;
        const int W = w1 > w0 ? (int)(w1 - w0) : 0;
        __syncthreads();  // the previous tile's rows are done with xs
        stage_window<RW, kBlock>(xs, W, w0, X, ldx, cbase, F);
        __syncthreads();
        for (int64_t r = r0 + g; r < r1; r += GPB) {
            float acc[CPL];  // rows hold at most the short-row limit of entries: one chain
#pragma unroll
            for (int i = 0; i < CPL; i++) acc[i] = 0.0f;
            const int64_t s = rp[r], e = rp[r + 1];
            for (int64_t kb = s; kb < e; kb += G) {
                const int m = (e - kb) < G ? (int)(e - kb) : G;
                int cj = 0;
                float vj = 0.0f;
                if (lane < m) {
                    cj = ld_stream(col + kb + lane);
                    vj = ld_stream(val + kb + lane);
                }
                for (int j = 0; j < m; j += B)
                    window_batch<B, NQ, G>(cj, vj, j, m, xs, w0, w1, lane, X, ldx, cols, acc);
            }
            store_quads_stream<NQ>(Y + r * ldy, cols, acc);
        }
    }
}

int env_int(const char *name, int dflt)
{
    const char *v = std::getenv(name);
    if (!v || !*v) return dflt;
    int x = std::atoi(v);
    return x > 0 ? x : dflt;
}

}  // namespace

// ------------------------------------------------------------------ plan
//
// csr_items = [chunk items of medium long rows | chunk items of huge rows |
// short items (slot -1)]; long_rows = [medium rows | huge rows], each part in
// decreasing length, long_first[] giving each long row's first partial slot.
// The generic path runs every chunk item and combines every long row; the
// vectorised path runs medium rows a workgroup each and only the huge rows'
// chunks (combined by a second small launch).
//
// The plan is built on the device: every row gets the 64-bit key
// (group << 32 | rank) with group 0 = medium, 1 = huge, 2 = short and rank =
// maxlen - len for long rows, thr - len for short rows of a skewed matrix
// (0 otherwise); a stable radix sort on those keys gives the row order
// (natural order within equal keys), a scan of the rows' item counts gives
// each row's first item, and one kernel writes the items.  A long row's
// chunk slots are its item positions.

namespace {

struct PlanStats {
    unsigned long long sum, sum2;
    int maxlen, n_long, n_huge, n_group;
};

// Row-length statistics: one partial record per workgroup (a one-workgroup
// grid writes the result itself); k_plan_stats_final combines the partials.
__device__ __forceinline__ PlanStats block_plan_stats(unsigned long long sum, unsigned long long sum2, int mx,
                                                      int nl, int nh, int ng)
{
    __shared__ unsigned long long t64[kBlock / kWave];
    __shared__ int t32[kBlock / kWave];
    PlanStats p;
    p.sum = block_sum_u64<kBlock>(sum, t64);
    p.sum2 = block_sum_u64<kBlock>(sum2, t64);
    p.maxlen = block_max_i32<kBlock>(mx, t32);
    p.n_long = (int)block_sum_u64<kBlock>((unsigned long long)nl, t64);
    p.n_huge = (int)block_sum_u64<kBlock>((unsigned long long)nh, t64);
    p.n_group = (int)block_sum_u64<kBlock>((unsigned long long)ng, t64);
    return p;
}

__global__ __launch_bounds__(kBlock) void k_plan_stats(const int32_t *__restrict__ rp, int64_t R,
                                                       int thr, int wg_thr, int group_max,
                                                       PlanStats *__restrict__ part,
                                                       PlanStats *__restrict__ st)
{
    unsigned long long sum = 0, sum2 = 0;
    int mx = 0, nl = 0, nh = 0, ng = 0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < R;
         i += (int64_t)gridDim.x * kBlock) {
        const int len = rp[i + 1] - rp[i];
        sum += (unsigned long long)len;
        sum2 += (unsigned long long)len * (unsigned long long)len;
        mx = len > mx ? len : mx;
        nl += len > thr;
        nh += len > wg_thr;
        ng += len > group_max;
    }
    const PlanStats p = block_plan_stats(sum, sum2, mx, nl, nh, ng);
    if (threadIdx.x == 0) (gridDim.x == 1 ? *st : part[blockIdx.x]) = p;
}

__global__ __launch_bounds__(kBlock) void k_plan_stats_final(const PlanStats *__restrict__ part, int64_t G,
                                                             PlanStats *__restrict__ st)
{
    unsigned long long sum = 0, sum2 = 0;
    int mx = 0, nl = 0, nh = 0, ng = 0;
    for (int64_t g = threadIdx.x; g < G; g += kBlock) {
        const PlanStats q = part[g];
        sum += q.sum;
        sum2 += q.sum2;
        mx = q.maxlen > mx ? q.maxlen : mx;
        nl += q.n_long;
        nh += q.n_huge;
        ng += q.n_group;
    }
    const PlanStats p = block_plan_stats(sum, sum2, mx, nl, nh, ng);
    if (threadIdx.x == 0) *st = p;
}

// Key of row i: its group (0 medium, 1 huge, 2 short) in the bits above the
// rank, the rank (distance below the longest length, so longer rows first)
// in the low `L` bits, so that the sort needs only L + 2 bits.
__global__ __launch_bounds__(kBlock) void k_plan_keys(const int32_t *__restrict__ rp, int64_t R,
                                                      int thr, int wg_thr, int sorted, int maxlen, int L,
                                                      uint64_t *__restrict__ keys)
{
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < R;
         i += (int64_t)gridDim.x * kBlock) {
        const int len = rp[i + 1] - rp[i];
        const uint64_t group = len > thr ? (len > wg_thr ? 1u : 0u) : 2u;
        const uint32_t rank = group < 2 ? (uint32_t)(maxlen - len) : sorted ? (uint32_t)(thr - len) : 0u;
        keys[i] = (group << L) | rank;
    }
}

__global__ __launch_bounds__(kBlock) void k_plan_count(const int32_t *__restrict__ rp,
                                                       const uint64_t *__restrict__ keys,
                                                       const uint32_t *__restrict__ perm, int64_t R,
                                                       int chunk, int L, int32_t *__restrict__ cnt)
{
    for (int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x; p < R;
         p += (int64_t)gridDim.x * kBlock) {
        const int64_t r = perm ? perm[p] : p;
        const int len = rp[r + 1] - rp[r];
        cnt[p] = keys && (keys[p] >> L) < 2 ? (len + chunk - 1) / chunk : 1;  // no keys: every row short
    }
}

__global__ __launch_bounds__(kBlock) void k_plan_items(const int32_t *__restrict__ rp,
                                                       const uint32_t *__restrict__ perm,
                                                       const int32_t *__restrict__ off, int64_t R,
                                                       int chunk, int64_t n_long,
                                                       int4 *__restrict__ items,
                                                       int32_t *__restrict__ long_rows,
                                                       int32_t *__restrict__ long_first)
{
    for (int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x; p < R;
         p += (int64_t)gridDim.x * kBlock) {
        const int r = perm ? (int)perm[p] : (int)p;
        const int start = rp[r], len = rp[r + 1] - start, o = off[p];
        if (p < n_long) {
            long_rows[p] = r;
            long_first[p] = o;
            for (int j = 0, c = 0; c < len; j++, c += chunk)
                items[o + j] = make_int4(r, start + c, len - c < chunk ? len - c : chunk, o + j);
        } else {
            items[o] = make_int4(r, start, len, -1);
        }
        if (p == 0) long_first[n_long] = off[n_long];
    }
}

inline unsigned plan_grid(int64_t n)
{
    int64_t g = ceil_div(n, (int64_t)kBlock);
    return (unsigned)(g < 1 ? 1 : g > 4096 ? 4096 : g);
}

inline unsigned stats_grid(int64_t n)
{
    int64_t g = ceil_div(n, (int64_t)kBlock * 4);
    return (unsigned)(g < 1 ? 1 : g > 2048 ? 2048 : g);
}

// The item counts at the three tier boundaries, gathered for one read-back.
__global__ void k_pick3(const int32_t *__restrict__ cnt, int64_t a, int64_t b, int64_t c,
                        int32_t *__restrict__ out)
{
    if (threadIdx.x == 0) {
        out[0] = cnt[a];
        out[1] = cnt[b];
        out[2] = cnt[c];
    }
}

// Reference class of a column with n entries: the bit length of n, at most 15.
__device__ __forceinline__ int col_class(int n)
{
    const int b = 32 - __clz(n);
    return b < 15 ? b : 15;
}

// Reference class of every column, one byte each (so that the tagging pass
// gathers from an array a quarter the size of the counts), and the number of
// columns per class.  The 16 bins are counted per wave by ballots (a power
// law puts most columns in two classes: LDS atomics on one bin serialised),
// and each workgroup writes its own 16 counts to part (atomics of thousands
// of workgroups on the same 16 words queued: 50 us at 2M columns);
// k_class_total adds them.
__global__ __launch_bounds__(kBlock) void k_col_classes(const int32_t *__restrict__ cc, int64_t C,
                                                        uint8_t *__restrict__ cls, int32_t *__restrict__ part)
{
    constexpr int U = 4;  // columns per lane in flight
    __shared__ int h[16];
    if (threadIdx.x < 16) h[threadIdx.x] = 0;
    __syncthreads();
    const int lane = threadIdx.x % kWave;
    const int64_t stride = (int64_t)gridDim.x * kBlock * U;
    // every lane of a wave runs the same number of rounds, so the ballots see whole waves
    for (int64_t j0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x - lane) * U; j0 < C; j0 += stride) {
        int k[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t j = j0 + u * kWave + lane;
            k[u] = j < C ? cc[j] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t j = j0 + u * kWave + lane;
            if (k[u] >= 0) {
                k[u] = col_class(k[u]);
                cls[j] = (uint8_t)k[u];
            }
        }
        for (int c = 0; c < 16; c++) {
            int n = 0;
#pragma unroll
            for (int u = 0; u < U; u++) n += __popcll(__ballot(k[u] == c));
            if (lane == 0 && n) atomicAdd(&h[c], n);
        }
    }
    __syncthreads();
    if (threadIdx.x < 16) part[(int64_t)blockIdx.x * 16 + threadIdx.x] = h[threadIdx.x];
}

// hist[c] = the sum of the G workgroups' counts of class c (one workgroup;
// sixteen readers per class, each adding every sixteenth workgroup's count).
__global__ __launch_bounds__(kBlock) void k_class_total(const int32_t *__restrict__ part, int G,
                                                        int32_t *__restrict__ hist)
{
    __shared__ int h[16];
    if (threadIdx.x < 16) h[threadIdx.x] = 0;
    __syncthreads();
    const int c = threadIdx.x % 16;
    int sum = 0;
    for (int i = threadIdx.x / 16; i < G; i += kBlock / 16) sum += part[(int64_t)i * 16 + c];
    atomicAdd(&h[c], sum);
    __syncthreads();
    if (threadIdx.x < 16) hist[threadIdx.x] = h[threadIdx.x];
}

// Class-tagged copy of the column indices: col | class(col) << 27.  Sixteen
// entries per thread (four 16-byte loads and stores), so that sixteen class
// bytes are gathered at once; a scalar tail.
__global__ __launch_bounds__(kBlock) void k_tag_cols(const int32_t *__restrict__ col, int64_t Z,
                                                     const uint8_t *__restrict__ cls, int32_t *__restrict__ tagged)
{
    const int64_t nv = Z / 16;  // whole groups of sixteen
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < nv; v += stride) {
        const int4 *src = reinterpret_cast<const int4 *>(col) + v * 4;
        int4 c[4];
#pragma unroll
        for (int u = 0; u < 4; u++) c[u] = src[u];
        int t[16];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            t[4 * u + 0] = cls[c[u].x];
            t[4 * u + 1] = cls[c[u].y];
            t[4 * u + 2] = cls[c[u].z];
            t[4 * u + 3] = cls[c[u].w];
        }
        int4 *dst = reinterpret_cast<int4 *>(tagged) + v * 4;
#pragma unroll
        for (int u = 0; u < 4; u++)
            dst[u] = make_int4(c[u].x | (t[4 * u + 0] << kColClassShift), c[u].y | (t[4 * u + 1] << kColClassShift),
                               c[u].z | (t[4 * u + 2] << kColClassShift), c[u].w | (t[4 * u + 3] << kColClassShift));
    }
    for (int64_t e = nv * 16 + (int64_t)blockIdx.x * kBlock + threadIdx.x; e < Z; e += stride)
        tagged[e] = col[e] | ((int)cls[col[e]] << kColClassShift);
}

// Entries whose column lies in their row's tile window, for the row tiles
// of 32 << k rows with halo 0 (counts[2k]) and halo 1 (counts[2k+1]):
// one partial set per workgroup, added into counts.
__global__ __launch_bounds__(kBlock) void k_win_counts(const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ col, int64_t R, int64_t C,
                                                       unsigned long long *__restrict__ counts)
{
    __shared__ unsigned long long t64[kBlock / kWave];
    unsigned long long n[2 * kWinCands] = {};
    for (int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x; r < R; r += (int64_t)gridDim.x * kBlock) {
        for (int64_t k = rp[r]; k < rp[r + 1]; k++) {
            const int64_t c = col[k];
#pragma unroll
            for (int w = 0; w < kWinCands; w++) {
                const int64_t T = 32 << w;
                const int64_t b = r / T * T, top = b + T < R ? b + T : R;
                n[2 * w] += (c >= b && c < top) ? 1u : 0u;
                n[2 * w + 1] += (c >= b - 1 && c < top + 1) ? 1u : 0u;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 2 * kWinCands; i++) {
        const unsigned long long tot = block_sum_u64<kBlock>(n[i], t64);
        if (threadIdx.x == 0 && tot) atomicAdd(&counts[i], tot);
    }
}

}  // namespace

// Locality of the row tiles: how many entries fall in their tile's window
// for each candidate tile and halo, for the LDS-staged kernel, into
// counts[2 * kWinCands] [dev].
static void enqueue_window_counts(const gs_matrix_ &m, const int32_t *rp, const int32_t *col,
                                  unsigned long long *counts, hipStream_t s)
{
    GS_HIP(hipMemsetAsync(counts, 0, sizeof(unsigned long long) * 2 * kWinCands, s));
    k_win_counts<<<stats_grid(m.R), kBlock, 0, s>>>(rp, col, m.R, m.C, counts);
    GS_HIP(hipGetLastError());
}

void count_windows(gs_matrix_ &m, const int32_t *rp, const int32_t *col, hipStream_t s)
{
    DevBuf cnt;
    unsigned long long h[2 * kWinCands];
    cnt.alloc(sizeof h, s);
    enqueue_window_counts(m, rp, col, cnt.as<unsigned long long>(), s);
    GS_HIP(hipMemcpyAsync(h, cnt.p, sizeof h, hipMemcpyDeviceToHost, s));
    GS_HIP(hipStreamSynchronize(s));
    for (int i = 0; i < 2 * kWinCands; i++) m.win_entries[i] = (int64_t)h[i];
    m.win_counted = true;
}

// Measured (F = 64..256): a tile pays for its staging only when most of its
// entries are inside the window and there are several tiles per resident
// workgroup.  On the mesh (about 60% inside) the staged ELL kernel took 38
// against 34 us; on the block graph (76% inside, 6,400 tiles) 217 against
// 236 us; on matrices of 10-15k rows (a few hundred tiles) the staged CSR and
// ELL kernels were about twice as slow as the plain ones (stage, barrier and
// rows in sequence on a short critical path).
bool pick_window(const gs_matrix_ &m, int64_t row_bytes, int &T, int &h)
{
    T = h = 0;
    if (!m.win_counted) return false;
    const int64_t lds_cap = std::min<int64_t>(max_lds_bytes(), (int64_t)env_int("GS_CSR_WIN_KB", 32) * 1024);
    const int64_t min_in = m.Z * env_int("GS_CSR_WIN_PCT", 65) / 100;
    const int64_t min_tiles = env_int("GS_WIN_MIN_TILES", 2 * resident_workgroups());
    int64_t best = -1;
    for (int w = 0; w < kWinCands; w++)
        for (int hh = 0; hh < 2; hh++) {
            const int64_t bytes = (int64_t)((32 << w) + 2 * hh) * row_bytes;
            const int64_t in = m.win_entries[2 * w + hh];
            if (bytes <= lds_cap && in >= min_in && in > best && ceil_div(m.R, (int64_t)(32 << w)) >= min_tiles) {
                best = in;
                T = 32 << w;
                h = hh;
            }
        }
    if (const char *e = std::getenv("GS_CSR_WIN_T"); e && *e) {  // tests and sweeps: force a tile
        const char *he = std::getenv("GS_CSR_WIN_H");
        const int t = std::atoi(e), hh = he && std::atoi(he) > 0 ? 1 : 0;
        if (t > 0 && (int64_t)(t + 2 * hh) * row_bytes <= max_lds_bytes()) {
            T = t;
            h = hh;
        }
    }
    return T > 0;
}

// Reference classes of the columns, for gathers that keep often referenced X
// rows in the caches: counts per column, each column's class (one byte) and
// the number of columns in each class into hist[16] [dev].  The class-tagged
// copy of the column indices is made by the first SpMM that uses the classes.
// Built for skewed matrices (rows ordered by length; GS_CSR_HOTCOLD = on / off
// forces it) whose column count fits the 27-bit column field; false: no
// classes.
static bool enqueue_col_classes(gs_matrix_ &m, int32_t *hist, hipStream_t s)
{
    const char *e = std::getenv("GS_CSR_HOTCOLD");
    const bool on = e && *e ? std::string(e) == "on" : m.csr_sorted;
    if (!on || m.Z == 0 || m.C > kColMask + 1) {
        m.col_counts.reset();
        return false;
    }
    DevBuf cc = std::move(m.col_counts);  // counted by feature extraction, if it ran
    if (!cc.p) {
        cc.alloc((size_t)m.C * 4, s);
        column_counts(m.col.as<int32_t>(), m.C, m.Z, cc.as<int32_t>(), s);
    }
    const unsigned G = std::min(plan_grid(ceil_div(m.C, 4)), 512u);
    DevBuf part;
    part.alloc((size_t)G * 16 * 4, s);
    m.col_cls.alloc((size_t)m.C, s);
    k_col_classes<<<G, kBlock, 0, s>>>(cc.as<int32_t>(), m.C, m.col_cls.as<uint8_t>(), part.as<int32_t>());
    GS_HIP(hipGetLastError());
    k_class_total<<<1, kBlock, 0, s>>>(part.as<int32_t>(), (int)G, hist);
    GS_HIP(hipGetLastError());
    return true;
}

namespace {

// What the host needs of a plan, read back in one copy: the item counts at the
// tier boundaries, the columns of each class, the window counts.
struct PlanBack {
    int32_t off[4];
    int32_t cls[16];
    unsigned long long win[2 * kWinCands];
};

struct Gathers {
    bool classes = false, windows = false;
};

Gathers enqueue_gathers(gs_matrix_ &m, PlanBack *back, hipStream_t s)
{
    const char *no_win = std::getenv("GS_CSR_WINDOW");
    Gathers have;
    have.classes = enqueue_col_classes(m, back->cls, s);
    have.windows = !(no_win && std::string(no_win) == "off") && !m.csr_sorted && !m.csr_grouped &&
                   m.n_long_rows == 0 && m.Z > 0;
    if (have.windows) enqueue_window_counts(m, m.row_ptr.as<int32_t>(), m.col.as<int32_t>(), back->win, s);
    return have;
}

void take_gathers(gs_matrix_ &m, Gathers have, const PlanBack &back)
{
    if (have.classes) std::copy(back.cls, back.cls + 16, m.col_class_cols);
    if (have.windows) {
        std::copy(back.win, back.win + 2 * kWinCands, m.win_entries);
        m.win_counted = true;
    }
    m.gathers_planned = true;
}

}  // namespace

void plan_gathers(gs_matrix_ &m, hipStream_t s)
{
    PlanBack back = {};
    DevBuf d_back;
    d_back.alloc(sizeof back, s);
    const Gathers have = enqueue_gathers(m, d_back.as<PlanBack>(), s);
    if (have.classes || have.windows) {
        GS_HIP(hipMemcpyAsync(&back, d_back.p, sizeof back, hipMemcpyDeviceToHost, s));
        GS_HIP(hipStreamSynchronize(s));
    }
    take_gathers(m, have, back);
}

void plan_csr(gs_matrix_ &m, hipStream_t s, bool gathers)
{
    const int thr = env_int("GS_CSR_LONG_ROW", kCsrLongRow);
    const int chunk = std::min(env_int("GS_CSR_CHUNK", kCsrChunk), thr);
    const int wg_thr = env_int("GS_CSR_WG_ROW", kCsrWgRow);
    m.csr_long_thr = thr;
    m.csr_chunk = chunk;
    const int64_t R = m.R;
    const int32_t *rp = m.row_ptr.as<int32_t>();

    const int group_max = std::max(env_int("GS_CSR_GROUP_ROW", kCsrGroupRow), thr);
    PlanStats st = {0, 0, 0, 0, 0, 0};
    if (R > 0) {
        const unsigned G = stats_grid(R);
        DevBuf d_st, part;
        d_st.alloc(sizeof st, s);
        if (G > 1) part.alloc(sizeof(PlanStats) * G, s);
        k_plan_stats<<<G, kBlock, 0, s>>>(rp, R, thr, wg_thr, group_max, part.as<PlanStats>(),
                                          d_st.as<PlanStats>());
        GS_HIP(hipGetLastError());
        if (G > 1) {
            k_plan_stats_final<<<1, kBlock, 0, s>>>(part.as<PlanStats>(), G, d_st.as<PlanStats>());
            GS_HIP(hipGetLastError());
        }
        GS_HIP(hipMemcpyAsync(&st, d_st.p, sizeof st, hipMemcpyDeviceToHost, s));
        GS_HIP(hipStreamSynchronize(s));
    }
    // Skewed row lengths (coefficient of variation above 1/2): order by length.
    const double mean = R ? (double)st.sum / (double)R : 0.0;
    const double var = R ? std::max(0.0, (double)st.sum2 / (double)R - mean * mean) : 0.0;
    const int force = env_int("GS_CSR_SORT", 0);  // 1: never, 2: always
    bool sorted = mean > 0 && std::sqrt(var) > 0.5 * mean;
    if (force == 1) sorted = false;
    if (force == 2) sorted = true;
    m.csr_sorted = sorted;
    // A workgroup per medium row pays off for a few hub rows running beside
    // the short ones; with more medium rows than resident workgroups they
    // would queue behind each other with most of each workgroup idle, so
    // then every long row is cut into chunk items whose partial sums a second
    // launch adds.  With many more (at least 8 per resident workgroup), every
    // row of up to group_max entries instead takes one lane group, which sums
    // it chunk by chunk in registers: the rows alone fill the groups, and no
    // partial sum goes through memory.  Measured on uniform random matrices
    // of 18-50k rows of 300-1500 entries at F = 128: 1.3-1.6x faster than
    // chunk items; with 9-13k such rows chunk items stay ahead at F = 64.
    int thr_eff = thr, wg_thr_eff = wg_thr;
    int64_t n_long = st.n_long, n_huge = st.n_huge;
    const int64_t n_medium = st.n_long - st.n_huge;
    const int64_t group_min = env_int("GS_CSR_GROUP_MIN", resident_workgroups() * 8);
    m.csr_grouped = false;
    if (n_medium > group_min && group_max > thr) {
        thr_eff = wg_thr_eff = group_max;
        n_long = n_huge = st.n_group;
        m.csr_grouped = true;
    } else if (n_medium > resident_workgroups()) {
        wg_thr_eff = thr;
        n_huge = st.n_long;
    }
    m.csr_wg_thr = wg_thr_eff;
    m.n_long_rows = n_long;
    m.n_medium_rows = n_long - n_huge;
    m.n_short = R - n_long;

    PlanBack back = {};
    DevBuf d_back;
    d_back.alloc(sizeof back, s);
    PlanBack *db = d_back.as<PlanBack>();
    DevBuf ka, kb, pa, pb, cnt;
    uint32_t *perm = nullptr;
    if (R > 0) {
        // ranks are at most max(longest row, thr): L bits, the group above them
        const int L = bits_for(std::max(st.maxlen, thr_eff));
        uint64_t *keys = nullptr;
        if (sorted || n_long > 0) {  // otherwise every key is equal: natural order, no sort
            ka.alloc((size_t)R * 8, s);
            kb.alloc((size_t)R * 8, s);
            pa.alloc((size_t)R * 4, s);
            pb.alloc((size_t)R * 4, s);
            k_plan_keys<<<plan_grid(R), kBlock, 0, s>>>(rp, R, thr_eff, wg_thr_eff, sorted ? 1 : 0, st.maxlen,
                                                        L, ka.as<uint64_t>());
            GS_HIP(hipGetLastError());
            std::vector<int> shifts;
            for (int sft = 0; sft < L + 2; sft += 8) shifts.push_back(sft);
            radix_sort_pairs(ka.as<uint64_t>(), kb.as<uint64_t>(), pa.as<uint32_t>(), pb.as<uint32_t>(), R,
                             shifts, s, &keys, &perm);
        }
        cnt.alloc((size_t)(R + 1) * 4, s);
        k_plan_count<<<plan_grid(R), kBlock, 0, s>>>(rp, keys, perm, R, chunk, L, cnt.as<int32_t>());
        GS_HIP(hipGetLastError());
        exclusive_scan_i32(cnt.as<int32_t>(), cnt.as<int32_t>(), R, true, s);
        k_pick3<<<1, kWave, 0, s>>>(cnt.as<int32_t>(), m.n_medium_rows, n_long, R, db->off);
        GS_HIP(hipGetLastError());
    }
    const Gathers have = gathers ? enqueue_gathers(m, db, s) : Gathers{};
    if (R > 0) {
        GS_HIP(hipMemcpyAsync(&back, d_back.p, sizeof back, hipMemcpyDeviceToHost, s));
        GS_HIP(hipStreamSynchronize(s));
    }
    m.n_medium_chunks = back.off[0];
    m.n_long_chunks = back.off[1];
    m.n_items = back.off[2];
    if (gathers) take_gathers(m, have, back);
    m.csr_items.alloc((size_t)m.n_items * sizeof(int4), s);
    m.long_rows.alloc((size_t)n_long * 4, s);
    m.long_first.alloc((size_t)(n_long + 1) * 4, s);
    if (R > 0) {
        k_plan_items<<<plan_grid(R), kBlock, 0, s>>>(rp, perm, cnt.as<int32_t>(), R, chunk, n_long,
                                                     m.csr_items.as<int4>(), m.long_rows.as<int32_t>(),
                                                     m.long_first.as<int32_t>());
        GS_HIP(hipGetLastError());
    } else {
        GS_HIP(hipMemsetAsync(m.long_first.p, 0, 4, s));
    }
    m.csr_planned = true;
}

// ------------------------------------------------------------- launcher

namespace {

// Kernel modes: full column slices with 32-bit X offsets, any width with
// them, and any width with 64-bit offsets (X of 4 GiB and more).
enum { kModeFull = 0, kModeAny = 1, kModeWide = 2 };

// Dynamic LDS of row kernels that shall leave 4 workgroups on a CU (and keep 4
// X rows in flight per lane group instead of 8).  Their X exceeds the caches
// and they run at the rate of the L2 fills (7.3 TB/s), so what counts is the L2
// hit rate, and every row in flight takes its lines of a 4 MiB L2.  Class
// gathers of the group tier (2M-row graph, F = 128): 8 rows 2966 us, 4 rows
// 2970, 4 rows and 4 workgroups 2910.  Class gathers otherwise run 4 rows
// without it (10^6 rows of 7 entries, F = 128: 479 us, with it 506, 8 rows 489;
// 150,000 rows of 17 139, 150, 142; of 5 at F = 200 100, 136, 110).
constexpr size_t kFewLds = 32000;

// Entries a row on average from which groups of 32 lanes take 32 at a time, in
// two registers (30,000 uniform rows at F = 128, 16 against 32 at a time: of 12
// entries 24.5 and 24.8 us, of 15 36.3 and 34.9, of 24 43.1 and 42.0, of 48
// 80.4 and 78.3; 9,000 of 720 185 and 164).
constexpr int64_t kFillRow = 14;

// Every byte offset into X stays below 4 GiB.
bool fits_off32(int64_t C, int64_t ldx, int64_t F)
{
    constexpr int64_t lim = 1ll << 30;  // elements
    return C <= 1 || (ldx < lim && (C - 1) <= (lim - F) / ldx);
}

// Workgroups of a row kernel: `rounds` times those resident on the chip, whose
// lane groups loop over their items.  A single round left the end of the
// launch unbalanced (items are dealt out statically): 1 / 2 / 4 / 8 rounds
// measured 68.1 / 61.7 / 60.2 / 61.1 us on the power-law graph, 137 / 163 /
// 108 / 107 on a 9,000-row uniform matrix (8% dense, F = 64), 190 (2) / 187 /
// 185 on the block graph; gathering by class 4 / 8 / 16 took 485 / 480 / 479 on
// 10^6 rows of 7 entries and 140 / 139 / 141 on 150,000 of 17, and on the
// 2M-row graph (4 resident) 14 / 28 / 56 took 3051 / 2910 / 2913.
unsigned rows_grid(const void *fn, size_t lds, int64_t tiles, int64_t slices, int rounds)
{
    const int64_t cap = (int64_t)resident_blocks(fn, kBlock, lds) * compute_units() * env_int("GS_WG_MULT", rounds);
    return (unsigned)std::max<int64_t>(1, std::min(tiles, cap / slices));
}

}  // namespace

bool spmm_csr_vec4(gs_matrix_ &m, const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t F,
                   hipStream_t s, const WorkArea *fixed)
{
    if (F < 4) return false;
    // Lane shape, measured over 160 profiled matrices at F = 64..256: four
    // columns per lane (wide groups, 8 X rows in flight per lane) is best or
    // near it, except in natural row order for very short rows (fewer than 8
    // entries on average) and for wide X (F >= 256) with rows under 64
    // entries, where more columns per lane -- more rows per wave -- win: 16, or
    // 8 for short rows at F <= 64 (mesh 33.8 us, with 16 37.8 and with 4 38.0;
    // 30,000 rows of 6 10.6, 11.7, 10.8; mesh at F = 128 62.7, 60.2, 70.3).
    const bool short_rows = !m.csr_sorted && m.Z < 8 * m.R;
    const bool many_rows_per_wave = short_rows || (!m.csr_sorted && F >= 256 && m.Z < 64 * m.R);
    // Chains of four entries, joining two sums in turn, where the operands are no
    // 16-byte quads (F, strides or addresses) and on COO handles: the kernels
    // that served those before this one summed in four chains, or in pieces of
    // a few dozen entries, and one chain of up to 128 has up to 70% more error.
    // Rows of under 4 entries have least error in one chain, which rounds each
    // product with its addition.  At most 8 columns per lane hold them.
    // Error (2-norm, against 64 bits) and time of the earlier kernels, of one
    // chain, of fours: 30,011 rows of 15 at F = 47 5.6e-8 23.8 us, 7.4e-8 21.1,
    // 5.6e-8 21.0; 140,001 of 20 at F = 33 5.9e-8 86.9, 8.4e-8 52.1, 5.9e-8 52.6;
    // power-law graph of 10^6 entries, COO, F = 64 3.3e-8 43.8, 3.5e-8 33.6,
    // 3.1e-8 33.9; four sums, entry j going to sum j % 4, 3.3e-8 35.0.
    auto quads = [](const void *p, int64_t ld) { return (uintptr_t)p % 16 == 0 && ld % 4 == 0; };
    const bool odd = F % 4 || !quads(X, ldx) || !quads(Y, ldy);
    const bool fours = (odd || (m.fmt == GS_COO && !many_rows_per_wave)) && (m.csr_sorted || m.Z >= 4 * m.R);
    int cpl = m.csr_grouped ? 4 : env_int("GS_CSR_CPL", !many_rows_per_wave ? 4 : F <= 64 || fours ? 8 : 16);
    if (fours) cpl = std::min(cpl, 8);
    if (cpl != 4 && cpl != 8 && cpl != 16) cpl = 16;
    while (cpl > 4 && F < 4 * (int64_t)cpl) cpl /= 2;  // at least 4 lanes per group
    const int64_t lanes = ceil_div(F, cpl);
    const int g = lanes <= 4 ? 4 : lanes <= 8 ? 8 : lanes <= 16 ? 16 : lanes <= 32 ? 32 : 64;
    const int64_t slices = ceil_div(F, (int64_t)g * cpl);
    const bool full = (F % ((int64_t)g * cpl)) == 0;
    const int mode = !fits_off32(m.C, ldx, F) ? kModeWide : full && !(fours && (odd || cpl > 4)) ? kModeFull : kModeAny;
    // Reference classes: the rows of the most referenced columns, whole
    // classes of them up to GS_CSR_HOT_KB (64 MiB) at this width, are
    // gathered with plain loads, every other row non-temporally, so that
    // rows read a few times do not displace them from the memory-side cache.
    // Measured on the 2M-row power-law graph at F = 128 (52M entries, rows
    // of columns with at least 64 entries hot): 3426 -> 3126 us; budgets of
    // 4 / 32 / 128 / 256 MiB gave 4185 / 3286 / 3231 / 3306 us.  Not used
    // when the rows of every referenced column fit the budget, nor (its gathers
    // keep 4 rows in flight) for rows of under 6 entries on an X of up to 4
    // budgets: 150,000 rows of 3 at F = 128 51.9 us, without 48.2, of 5 61.3,
    // 59.5; of 17 138.4, 144.7; 10^6 rows of 7 478, 497.
    int hot_cls = 0;
    const int64_t hot_kb = env_int("GS_CSR_HOT_KB", 65536);
    if (m.col_cls.p && cpl == 4 && (m.Z >= 6 * m.R || m.C * F * 4 > hot_kb * 4096)) {
        const int64_t budget = hot_kb * 1024 / (F * 4);
        int64_t cum = 0;
        for (int c = 15; c >= 1 && !hot_cls; c--) {
            cum += m.col_class_cols[c];
            if (cum > budget) hot_cls = c < 15 ? c + 1 : 15;
        }
        if (hot_cls && !m.csr_colf.p) {
            if (fixed || is_capturing(s)) {
                hot_cls = 0;  // no allocation allowed, or the copy would be made by the first replay: plain gathers
            } else {          // first use: the class-tagged column copy
                m.csr_colf.alloc((size_t)m.Z * 4, s);
                k_tag_cols<<<plan_grid(ceil_div(m.Z, 16)), kBlock, 0, s>>>(
                    m.col.as<int32_t>(), m.Z, m.col_cls.as<uint8_t>(), m.csr_colf.as<int32_t>());
                GS_HIP(hipGetLastError());
            }
        }
    }
    // LDS-staged row tiles (pick_window): the candidate (tile, halo) that
    // keeps the most entries in the window within GS_CSR_WIN_KB (32 KiB) of
    // LDS per workgroup.  More LDS per workgroup costs resident waves: on the
    // block-community graph (F = 256) tiles of 32 / 64 / 128 rows (32 / 64 /
    // 128 KiB) measured 193 / 280 / 480 us against 209 us without staging
    // (with today's plain kernel both take 203 us there).
    int win_T = 0, win_h = 0;
    if (m.n_long_rows == 0 && !m.csr_grouped && !fours) pick_window(m, (int64_t)g * cpl * 4, win_T, win_h);
    auto launch = [&](auto cpl_t, auto g_t, auto mode_t) {
        constexpr int CPL = decltype(cpl_t)::value, G = decltype(g_t)::value, M = decltype(mode_t)::value;
        constexpr bool FU = M == kModeFull;
        constexpr int OFF = M == kModeWide ? kOff64 : kOff32;
        constexpr int GPB = kBlock / G;
        if (win_T > 0) {
            const int64_t ntiles = ceil_div(m.R, win_T);
            const size_t lds = (size_t)(win_T + 2 * win_h) * G * CPL * 4;
            const int64_t cap = (int64_t)resident_workgroups() * env_int("GS_WG_MULT", 8);
            dim3 grid((unsigned)std::max<int64_t>(1, std::min(ntiles, cap / slices)), (unsigned)slices);
            k_csr_window<CPL, G, FU><<<grid, kBlock, lds, s>>>(m.R, m.C, m.row_ptr.as<int32_t>(),
                                                               m.col.as<int32_t>(), m.val.as<float>(), X, ldx, Y,
                                                               ldy, F, win_T, win_h, ntiles);
            GS_HIP(hipGetLastError());
            return;
        }
        const int64_t n_group_items = m.n_items - m.n_medium_chunks;  // huge chunks + short rows
        const int64_t n_huge = m.n_long_rows - m.n_medium_rows;
        const int64_t tiles = m.n_medium_rows + ceil_div(n_group_items, GPB);
        if (!tiles) return;
        float *work = n_huge ? (float *)work_for(m, fixed, (size_t)m.n_long_chunks * F * 4, s) : nullptr;
        auto rows = [&](auto v_t, const int32_t *cols, int rounds, size_t lds = 0) {
            auto fn = k_csr_rows<CPL, G, FU, OFF, decltype(v_t)>;
            dim3 grid(rows_grid((const void *)fn, lds, tiles, slices, rounds), (unsigned)slices);
            fn<<<grid, kBlock, lds, s>>>(m.n_medium_rows, m.long_rows.as<int32_t>(), m.row_ptr.as<int32_t>(),
                                         m.csr_chunk, n_group_items, m.csr_items.as<int4>() + m.n_medium_chunks,
                                         cols ? cols : m.row_ptr.as<int32_t>(),
                                         m.Z ? m.val.as<float>() : m.row_ptr.as<float>(),
                                         (int)std::max<int64_t>(m.Z - 1, 0), X, ldx, Y, ldy, F, work, hot_cls, 0);
            GS_HIP(hipGetLastError());
        };
        auto pick = [&](auto na_t) {
            constexpr int NA = decltype(na_t)::value;
            constexpr int NB = G == 32 ? 2 : 1;  // (of long rows)
            const int32_t *col = m.col.as<int32_t>();
            const int rounds = m.csr_sorted ? 4 : 8;
            if constexpr (CPL == 4) {
                if (hot_cls) {  // reference classes: only the length-sorted lane shape
                    const int32_t *tagged = m.csr_colf.as<int32_t>();
                    if (m.csr_grouped) return rows(RowVariant<float, true, true, 0, NA, NB>{}, tagged, 32, kFewLds);
                    return rows(RowVariant<float, true, false, 0, NA, NB>{}, tagged, 8);
                }
            }
            if constexpr (CPL == 4) {
                if (m.csr_grouped) return rows(RowVariant<float, false, true, 0, NA, NB>{}, col, rounds);
            }
            if constexpr (CPL == 4 && G >= 16 && OFF == kOff32) {
                // Small skewed matrices, whose time is the longest rows' chain of
                // round trips: 16 rows in flight.  Power-law graphs of 11 entries
                // a row, 16 against 8: 275,000 entries 15.5 and 16.8 us (F = 64),
                // 19.5 and 20.7 (128); 385,000 19.8 and 21.5, 26.4 and 26.5;
                // 495,000 21.0 and 21.8, 30.1 and 28.8; 660,000 24.2 and 24.9,
                // 38.2 and 36.7; without long rows slower (2,048 nodes 5.9, 5.1).
                if (m.csr_sorted && m.n_long_rows > 0 && m.Z <= (F <= 64 ? 1 << 19 : 3 << 17))
                    return rows(RowVariant<float, false, false, 16, NA>{}, col, rounds);
                // Long rows in numbers: 4 rows in flight and 4 workgroups per CU.
                // Against 8: 9,000 rows of 720 entries, X of 30,000 rows (7 to 18
                // MiB) 131 -> 114 us at F = 64, 334 -> 274 at 128, 498 -> 398 at
                // 156, X of 1,500 105.1 -> 103.7, 168 -> 155, 244 -> 235 (200);
                // 15,000 rows of 300 162 -> 136 at 128, 348 -> 253 at 200; up to 3%
                // slower near an X of 3.5 MiB (15,000 of 300 at F = 64, 13,283 of 375
                // at 156) and below this line (3,302 rows of 165 at F = 176 30 -> 34,
                // F = 32 143 -> 145).
                if (m.Z >= 128 * m.R && F >= 64 && m.Z >= (1ll << 28) / F)
                    return rows(RowVariant<float, false, false, 4, NA, NB>{}, col, 2 * rounds, kFewLds);
            }
            if constexpr (G == 32) {
                if (m.Z >= kFillRow * m.R) return rows(RowVariant<float, false, false, 0, NA, NB>{}, col, rounds);
            }
            rows(RowVariant<float, false, false, 0, NA>{}, col, rounds);
        };
        if constexpr (CPL == 4 || (CPL == 8 && M != kModeFull)) {
            if (fours)
                pick(std::integral_constant<int, 2>{});
            else
                pick(std::integral_constant<int, 1>{});
        } else {
            pick(std::integral_constant<int, 1>{});
        }
        if (n_huge) {
            dim3 g2((unsigned)ceil_div(n_huge, GPB), (unsigned)slices);
            k_csr_combine<CPL, G, float><<<g2, kBlock, 0, s>>>(m.long_rows.as<int32_t>() + m.n_medium_rows,
                                                               m.long_first.as<int32_t>() + m.n_medium_rows,
                                                               n_huge, work, Y, ldy, F);
            GS_HIP(hipGetLastError());
        }
    };
    auto by_mode = [&](auto cpl_t, auto g_t) {
        if (mode == kModeFull)
            launch(cpl_t, g_t, std::integral_constant<int, kModeFull>{});
        else if (mode == kModeAny)
            launch(cpl_t, g_t, std::integral_constant<int, kModeAny>{});
        else
            launch(cpl_t, g_t, std::integral_constant<int, kModeWide>{});
        return true;
    };
#define GS_L(C, GG) \
    if (cpl == C && g == GG) return by_mode(std::integral_constant<int, C>{}, std::integral_constant<int, GG>{});
    GS_L(16, 4) GS_L(16, 8) GS_L(16, 16) GS_L(16, 32) GS_L(16, 64)
    GS_L(8, 4) GS_L(8, 8) GS_L(8, 16) GS_L(8, 32) GS_L(8, 64)
    GS_L(4, 4) GS_L(4, 8) GS_L(4, 16) GS_L(4, 32) GS_L(4, 64)
#undef GS_L
    return false;
}

void spmm_rows_f64(gs_matrix_ &m, const float *X, int64_t ldx, float *Y, int64_t ldy, int64_t F, hipStream_t s,
                   const WorkArea *fixed)
{
    // Partial sums of the long rows cut into chunks.  A fixed workspace too
    // small for them: no chunks, every long row takes a workgroup (a wave).
    const size_t need = (size_t)m.n_long_chunks * F * 8;
    const bool chunks = !fixed || need <= fixed->cap;
    const int32_t *rp = m.row_ptr.as<int32_t>();
    const int32_t *col = m.Z ? m.col.as<int32_t>() : rp;
    const float *val = m.Z ? m.val.as<float>() : m.row_ptr.as<float>();
    const int4 *items = m.csr_items.as<int4>();
    if (F < 4) {
        double *work = chunks && need ? (double *)work_for(m, fixed, need, s) : nullptr;
        const int64_t n = chunks ? m.n_items : m.R;
        const int64_t g = std::min<int64_t>(ceil_div(n, kBlock / kWave), 1 << 16);
        k_rows_f64_narrow<<<(unsigned)std::max<int64_t>(g, 1), kBlock, 0, s>>>(n, chunks ? items : nullptr, rp, col, val,
                                                                              X, ldx, Y, ldy, (int)F, work);
        GS_HIP(hipGetLastError());
        if (chunks && m.n_long_rows) {
            k_combine_f64_narrow<<<(unsigned)ceil_div(m.n_long_rows, kBlock / kWave), kBlock, 0, s>>>(
                m.n_long_rows, m.long_rows.as<int32_t>(), m.long_first.as<int32_t>(), work, Y, ldy, (int)F);
            GS_HIP(hipGetLastError());
        }
        return;
    }
    const int64_t lanes = ceil_div(F, 4);
    const int g = lanes <= 4 ? 4 : lanes <= 8 ? 8 : lanes <= 16 ? 16 : lanes <= 32 ? 32 : 64;
    const int64_t slices = ceil_div(F, (int64_t)g * 4);
    const int64_t n_wg = chunks ? m.n_medium_rows : m.n_long_rows;       // long rows that take a workgroup
    const int64_t skip = chunks ? m.n_medium_chunks : m.n_long_chunks;   // their chunk items
    const int64_t n_huge = m.n_long_rows - n_wg;
    double *work = n_huge ? (double *)work_for(m, fixed, need, s) : nullptr;
    auto launch = [&](auto g_t, auto mode_t) {
        constexpr int G = decltype(g_t)::value, M = decltype(mode_t)::value, GPB = kBlock / G;
        const auto fn =
            k_csr_rows<4, G, M == kModeFull, M == kModeWide ? kOff64 : kOff32, RowVariant<double, false, false>>;
        const int64_t tiles = n_wg + ceil_div(m.n_items - skip, GPB);
        if (!tiles) return;
        dim3 grid(rows_grid((const void *)fn, 0, tiles, slices, m.csr_sorted ? 4 : 8), (unsigned)slices);
        fn<<<grid, kBlock, 0, s>>>(n_wg, m.long_rows.as<int32_t>(), rp, m.csr_chunk, m.n_items - skip, items + skip, col,
                                   val, (int)std::max<int64_t>(m.Z - 1, 0), X, ldx, Y, ldy, F, work, 0,
                                   !m.csr_sorted && m.n_long_rows == 0);
        GS_HIP(hipGetLastError());
        if (n_huge) {
            dim3 g2((unsigned)ceil_div(n_huge, GPB), (unsigned)slices);
            k_csr_combine<4, G, double><<<g2, kBlock, 0, s>>>(m.long_rows.as<int32_t>() + n_wg,
                                                              m.long_first.as<int32_t>() + n_wg, n_huge, work, Y, ldy,
                                                              F);
            GS_HIP(hipGetLastError());
        }
    };
    const bool full = F % ((int64_t)g * 4) == 0, wide = !fits_off32(m.C, ldx, F);
    auto by_g = [&](auto mode_t) {
        switch (g) {
        case 4: launch(std::integral_constant<int, 4>{}, mode_t); break;
        case 8: launch(std::integral_constant<int, 8>{}, mode_t); break;
        case 16: launch(std::integral_constant<int, 16>{}, mode_t); break;
        case 32: launch(std::integral_constant<int, 32>{}, mode_t); break;
        default: launch(std::integral_constant<int, 64>{}, mode_t); break;
        }
    };
    if (wide)
        by_g(std::integral_constant<int, kModeWide>{});
    else if (full)
        by_g(std::integral_constant<int, kModeFull>{});
    else
        by_g(std::integral_constant<int, kModeAny>{});
}

}  // namespace gs

// Dense products of a GNN layer whose one long dimension is the node count
// (Sec. 2.1: the layer's weights act on the aggregated features): the weight
// gradient H^T G, a contraction over the n rows of two tall matrices.
//
// fp32 on the matrix cores (V_MFMA_F32_32X32X2_F32: fp32 products and sums).
// Bound by them at 128 x 128 (3.3 GFLOP at n = 100,000: 21 us at their rate,
// 20 us of memory time): what matters is that n is split over the whole chip
// and that neither operand is transposed on the way, so both are staged as
// they lie in memory (rows of H and G are the k index of the product).
// Measured at n = 100,000: 128 x 128 50 us (the sum of the partials included),
// 128 x 64 30 us; a transposed copy of H, PyTorch's batched product over chunks
// and its sum took 141 and 110 us.
#include <algorithm>
#include <type_traits>

#include "gs_device.h"
#include "gs_gather.h"
#include "gs_internal.h"

namespace gs {
namespace {

constexpr int kBlock = 256;
constexpr int kRows = 32;  // rows of H and G per stage
// Workgroups of more than kChainRows rows add their running sums into totals
// every kFoldRows rows, so that no chain grows with n (512 x 512 leaves a
// workgroup n / 32 rows).  The totals are a second set of registers, which costs
// the shorter ones more than it gives: n = 2,000,000, 128 x 128 (3,936 rows) in
// one chain 631 us with an error of 5.0e-8 (2-norm, operands in [0, 1)), folded
// 760 and 3.5e-8; 512 x 512 (62,528 rows) 8.5 ms and 1.0e-6, folded 11.4 ms and
// 3.5e-8.  PyTorch's batched product over 2,048-row chunks: 1,830 us and 6.5e-8,
// 11.7 ms and 6.6e-8.  Adding into the partial in memory instead took 15.0 ms.
constexpr int kFoldRows = 1024, kChainRows = 4096;
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Rows [r0, r0 + kRows) x columns [c0, c0 + W) of M (n x c, leading dimension
// ld) into registers, zeros outside.
template <int W>
__device__ __forceinline__ void load_stage(f4u *v, const float *__restrict__ M, int64_t ld, int64_t r0, int64_t n,
                                           int c0, int c)
{
    constexpr int Q = W / 4, PER = kRows * Q / kBlock;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int e = i * kBlock + threadIdx.x, r = e / Q, col = c0 + 4 * (e % Q);
        const float *p = M + (r0 + r) * ld + col;
        v[i] = f4u{0.f, 0.f, 0.f, 0.f};
        if (r0 + r < n) {
            if (col + 4 <= c) {
                v[i] = *reinterpret_cast<const f4u *>(p);
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++)
                    if (col + j < c) v[i][j] = p[j];
            }
        }
    }
}

template <int W> __device__ __forceinline__ void store_stage(float *lds, const f4u *v)
{
    constexpr int Q = W / 4, PER = kRows * Q / kBlock;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int e = i * kBlock + threadIdx.x;
        *reinterpret_cast<float4 *>(lds + (e / Q) * W + 4 * (e % Q)) = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
    }
}

// Workgroup (x, y): rows [x * per, (x + 1) * per) of H and G, output tile y of
// MT x NT (of the a x b product), four waves WM x WN x KS: a wave owns
// MT / WM x NT / WN of the tile and every KS-th pair of rows, and writes its
// sums as partial (x * KS + ks).  The next stage's rows are loaded while the
// current one's are multiplied.  FOLD: per exceeds kChainRows.
template <int MT, int NT, int WM, int WN, bool FOLD>
__global__ __launch_bounds__(kBlock) void k_tn_partial(const float *__restrict__ H, int64_t ldh,
                                                       const float *__restrict__ G, int64_t ldg, int64_t n, int a, int b,
                                                       int64_t per, float *__restrict__ part)
{
    constexpr int KS = 4 / (WM * WN);
    constexpr int TM = MT / WM / 32, TN = NT / WN / 32;
    __shared__ __align__(16) float hs[kRows * MT], gsm[kRows * NT];
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int ks = wave / (WM * WN), wm = wave % (WM * WN) / WN, wn = wave % WN;
    const int nbt = (b + NT - 1) / NT;
    const int m0 = (blockIdx.y / nbt) * MT, n0 = (blockIdx.y % nbt) * NT;
    const int64_t r0 = (int64_t)blockIdx.x * per, r1 = r0 + per < n ? r0 + per : n;
    f32x16 acc[TM][TN], tot[FOLD ? TM : 1][FOLD ? TN : 1];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) {
            acc[i][j] = f32x16{};
            if constexpr (FOLD) tot[i][j] = f32x16{};
        }
    auto fold = [&] {
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++) {
                tot[FOLD ? i : 0][FOLD ? j : 0] += acc[i][j];
                acc[i][j] = FOLD ? f32x16{} : acc[i][j];
            }
    };
    f4u hv[kRows * MT / 4 / kBlock], gv[kRows * NT / 4 / kBlock];
    load_stage<MT>(hv, H, ldh, r0, r1, m0, a);
    load_stage<NT>(gv, G, ldg, r0, r1, n0, b);
    const float *hp = hs + (lane / 32) * MT + wm * (TM * 32) + lane % 32;
    const float *gp = gsm + (lane / 32) * NT + wn * (TN * 32) + lane % 32;
    for (int64_t r = r0; r < r1; r += kRows) {
        __syncthreads();  // the previous stage has been read
        store_stage<MT>(hs, hv);
        store_stage<NT>(gsm, gv);
        __syncthreads();
        load_stage<MT>(hv, H, ldh, r + kRows, r1, m0, a);  // zeros past the last row
        load_stage<NT>(gv, G, ldg, r + kRows, r1, n0, b);
#pragma unroll
        for (int k = 0; k < kRows; k += 2 * KS) {
            const int kk = k + 2 * ks;
            float av[TM], bv[TN];
#pragma unroll
            for (int i = 0; i < TM; i++) av[i] = hp[kk * MT + 32 * i];
#pragma unroll
            for (int j = 0; j < TN; j++) bv[j] = gp[kk * NT + 32 * j];
#pragma unroll
            for (int i = 0; i < TM; i++)
#pragma unroll
                for (int j = 0; j < TN; j++)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[j], acc[i][j], 0, 0, 0);
        }
        if constexpr (FOLD)
            if ((r - r0) % kFoldRows == kFoldRows - kRows) fold();
    }
    if constexpr (FOLD) fold();
    // accumulator layout: lane l, register e hold row 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32
    float *out = part + ((int64_t)blockIdx.x * KS + ks) * a * b;
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const int row = m0 + wm * (TM * 32) + 32 * i + 8 * (e / 4) + 4 * (lane / 32) + e % 4;
                const int col = n0 + wn * (TN * 32) + 32 * j + lane % 32;
                if (row < a && col < b) out[(int64_t)row * b + col] = FOLD ? tot[FOLD ? i : 0][FOLD ? j : 0][e] : acc[i][j][e];
            }
}

// out[e] = the sum of the P partials' element e, in a fixed order: sixteen
// slices of the partials per 64 elements, added in LDS.
__global__ __launch_bounds__(1024) void k_tn_reduce(const float *__restrict__ part, int P, int64_t ab,
                                                    float *__restrict__ out)
{
    __shared__ float red[16][64];
    const int lane = threadIdx.x % 64, sl = threadIdx.x / 64;
    const int64_t e = (int64_t)blockIdx.x * 64 + lane;
    float s = 0.0f;
    if (e < ab) {
        constexpr int U = 8;  // partials in flight
        for (int p = sl; p < P; p += 16 * U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; u++) v[u] = p + 16 * u < P ? part[(int64_t)(p + 16 * u) * ab + e] : 0.0f;
#pragma unroll
            for (int u = 0; u < U; u++) s += v[u];
        }
    }
    red[sl][lane] = s;
    __syncthreads();
#pragma unroll
    for (int w = 8; w > 0; w >>= 1) {
        if (sl < w) red[sl][lane] += red[sl + w][lane];
        __syncthreads();
    }
    if (sl == 0 && e < ab) out[e] = red[0][lane];
}

int tile_of(int64_t x) { return x <= 32 ? 32 : x <= 64 ? 64 : 128; }

struct TnPlan {
    int mt, nt, ks;
    int64_t tiles, chunks, per;
};

// One round of workgroups, two to a CU, at least two stages of rows each.
TnPlan tn_plan(int64_t n, int64_t a, int64_t b)
{
    TnPlan p;
    p.mt = tile_of(a);
    p.nt = tile_of(b);
    const int t = (p.mt / 32) * (p.nt / 32);
    p.ks = t >= 4 ? 1 : 4 / t;
    p.tiles = ceil_div(a, p.mt) * ceil_div(b, p.nt);
    const int64_t want = std::max<int64_t>(1, 512 / p.tiles);
    p.chunks = std::max<int64_t>(1, std::min(want, ceil_div(n, 2 * kRows)));
    p.per = std::max<int64_t>(kRows, ceil_div(ceil_div(n, p.chunks), kRows) * kRows);
    p.chunks = std::max<int64_t>(1, ceil_div(n, p.per));
    return p;
}

}  // namespace
}  // namespace gs

using namespace gs;

extern "C" {

int gs_weight_grad_workspace(int64_t n, int64_t a, int64_t b, uint64_t *bytes)
{
    return guarded([&] {
        if (!bytes) fail(GS_ERR_INVALID_ARG, "null output");
        if (n < 0 || a <= 0 || b <= 0) fail(GS_ERR_INVALID_ARG, "bad product size");
        if (a > 4096 || b > 4096 || n > INT32_MAX) fail(GS_ERR_UNSUPPORTED, "a and b are at most 4096");
        const TnPlan p = tn_plan(n, a, b);
        *bytes = (uint64_t)(p.chunks * p.ks * a * b) * 4;
    });
}

int gs_weight_grad(const float *H, int64_t ldh, const float *G, int64_t ldg, int64_t n, int64_t a, int64_t b,
                   float *out, void *work, uint64_t work_bytes, gs_stream stream)
{
    return guarded([&] {
        uint64_t need = 0;
        if (const int rc = gs_weight_grad_workspace(n, a, b, &need); rc != GS_OK) throw Error{rc};
        if (!out || !work || (n > 0 && (!H || !G))) fail(GS_ERR_INVALID_ARG, "null operand");
        if (ldh < a || ldg < b) fail(GS_ERR_INVALID_ARG, "leading dimensions must be >= the widths");
        if (work_bytes < need) fail(GS_ERR_INVALID_ARG, "workspace of %llu bytes is below the %llu needed",
                                    (unsigned long long)work_bytes, (unsigned long long)need);
        const hipStream_t s = (hipStream_t)stream;
        const TnPlan p = tn_plan(n, a, b);
        const dim3 grid((unsigned)p.chunks, (unsigned)p.tiles);
        float *part = (float *)work;
        auto go = [&](auto mt, auto nt, auto wm, auto wn, auto fold) {
            k_tn_partial<decltype(mt)::value, decltype(nt)::value, decltype(wm)::value, decltype(wn)::value,
                         decltype(fold)::value>
                <<<grid, kBlock, 0, s>>>(H, ldh, G, ldg, n, (int)a, (int)b, p.per, part);
        };
        auto tiled = [&](auto mt, auto nt, auto wm, auto wn) {
            if (p.mt != decltype(mt)::value || p.nt != decltype(nt)::value) return;
            if (p.per > kChainRows)
                go(mt, nt, wm, wn, std::true_type{});
            else
                go(mt, nt, wm, wn, std::false_type{});
        };
#define GS_TN(M, N, WM, WN)                                                                                       \
    tiled(std::integral_constant<int, M>{}, std::integral_constant<int, N>{}, std::integral_constant<int, WM>{}, \
          std::integral_constant<int, WN>{});
        GS_TN(128, 128, 2, 2) GS_TN(128, 64, 2, 2) GS_TN(64, 128, 2, 2) GS_TN(64, 64, 2, 2)
        GS_TN(128, 32, 4, 1) GS_TN(32, 128, 1, 4) GS_TN(64, 32, 2, 1) GS_TN(32, 64, 1, 2) GS_TN(32, 32, 1, 1)
#undef GS_TN
        GS_HIP(hipGetLastError());
        k_tn_reduce<<<(unsigned)ceil_div(a * b, 64), 1024, 0, s>>>(part, (int)(p.chunks * p.ks), a * b, out);
        GS_HIP(hipGetLastError());
    });
}

}  // extern "C"

// pbs_attn_fwd in fp32 arithmetic: float32 storage (any d, any block), bf16 storage with blocks of 16 or 32.
//
// Everything is kept transposed, as in the bf16 kernels (S^T = K' Q'^T, O^T += V'^T P^T), on the fp32 matrix
// instruction v_mfma_f32_16x16x4_f32: inputs, products and sums are those of a chain of fp32 fused multiply-adds, at
// the same 157 TFLOP/s peak as the vector unit, but one instruction reads two registers for 2048 operations instead
// of one LDS word per lane for every multiply-add.
//
// A workgroup owns 16 queries of one head and its waves share the key list among them (wave w takes sub-tiles w,
// w + WAVES, ... of KT = min(block, 32) keys), every wave with a softmax of its own; the partial (m, l, O) meet in
// LDS at the end.  That is what fills the chip at the small sizes fp32 layers have (2 heads x 2048 tokens are 256
// workgroups of 8 waves; with a workgroup per query block they would be 64), and it means that no K' or V' element is
// wanted by two waves of a workgroup, so nothing goes through LDS: with
//     A operand of S^T:   lane (key = lane % 16, g = lane / 16) holds K'[key][16 u + 4 g + c],  step (u, c)
//     A operand of O^T:   lane (e = lane % 16, g)               holds V'^T[16 t + e][4 g + r],  step r
// both are 16-byte loads straight from K' rows and Vt rows, and the S^T accumulator (query = lane % 16, keys 4 g + r)
// is already the B operand of the second product.  The contraction order over features is permuted the same way in K'
// and Q', which changes nothing but the order of an fp32 sum.
//
// Bound: the fp32 matrix rate (64 operations per clock and SIMD): 64 instructions of 32 clocks per 32 keys and 16
// queries at d = 64, against 16 loads that the next sub-tile's arithmetic covers.  Measured (float32, d = 64, block 64):
// 2 heads x 2048 tokens 35 us; the vector kernel before it (two threads per query, K' and V' through LDS, one LDS word
// read per multiply-add) took 1549 us.
#include <limits.h>

#include "pbs_host.h"

namespace pbs {
namespace fp32 {

constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f;
constexpr int kXcds = 8;
constexpr int kQ = 16;                                     // queries per workgroup
// A reference that has been set moves again only when a score passes it by this many powers of two: sums relative to
// it then stay below 2^6 per key, and the rescale of O and l is rare.
constexpr float kLead = 6.0f;

typedef int int4u __attribute__((ext_vector_type(4), aligned(4)));

// grid: linear ids (x fastest; y only where x alone would pass 2^32 threads), cohorts of `cohort` workgroups of one kv
// head per XCD, longest lists first (see the decoding below)
template <typename E, int D, int KT, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_fp32_kernel(
    const E *__restrict__ Qp, const E *__restrict__ Kp, const E *__restrict__ Vt, const int32_t *__restrict__ qidx,
    const int32_t *__restrict__ kidx, const int32_t *__restrict__ row_cnt, const int32_t *__restrict__ col_idx,
    E *__restrict__ Op, float *__restrict__ lse, Geo g, int cohort)
{
    constexpr int NK = KT / 16;                            // 16-key tiles per sub-tile
    constexpr int NU = D / 16;                             // 16-feature steps of S^T = feature tiles of O^T
    constexpr int kPad = kQ + 1;
    __shared__ float sm[WAVES][kQ], sl[WAVES][kQ];
    __shared__ float so[WAVES][D * kPad];

    const int tiles = ceil_div(g.n, kQ);                   // query tiles per head
    const int rows_per_unit = g.r * tiles;
    const int coh_per_unit = ceil_div(rows_per_unit, cohort);
    const uint32_t wg = blockIdx.y * gridDim.x + blockIdx.x;
    const int xcd = wg % kXcds, slot = wg / kXcds;
    const int coh = (slot / cohort) * kXcds + xcd;
    const int nbk = g.batch * g.h_kv;
    if (coh >= nbk * coh_per_unit) return;
    const int unit = coh % nbk;
    const int mrow = (coh / nbk) * cohort + slot % cohort;
    if (mrow >= rows_per_unit) return;
    const int q0 = (tiles - 1 - mrow / g.r) * kQ;
    const int i = q0 / g.block;                            // kQ divides every block size
    const int b = unit / g.h_kv, hq = (unit % g.h_kv) * g.r + mrow % g.r;
    const size_t bhq = (size_t)b * g.h_q + hq, bhk = unit;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ln = lane & 15, lg = lane >> 4;

    const int qs = q0 + ln;
    const bool live = qs < g.n;
    const int qpos = live ? (qidx ? qidx[bhq * g.n + qs] : qs) : -1;
    const float c2 = g.scale * kLog2eF;
    floatx4 q[NU];
    {
        const E *src = Qp + (bhq * g.n + (live ? qs : g.n - 1)) * D + 4 * lg;
#pragma unroll
        for (int u = 0; u < NU; ++u) q[u] = load4(src + 16 * u);
    }
    floatx4 acc[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) acc[u] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    float mref = 0.0f, l = 0.0f;                           // this lane's keys only for l
    bool seen = !live;                                     // mref is set; padding rows never hold the wave back

    const int ni = allowed_cols(i, g);
    const int subs = g.block / KT;                         // 1, 2 or 4
    const int total = min(row_cnt[bhq * g.T + i], g.T) * subs;
    const int32_t *cols = col_idx + (bhq * g.T + i) * g.T;
    const E *Kh = Kp + bhk * (size_t)g.n * D;
    const E *Vh = Vt + bhk * (size_t)g.T * D * g.block;
    const int32_t *kih = kidx + bhk * (size_t)g.n;

    // first slot of this wave's next admitted sub-tile at or after u, -1 past the end
    int u_next = wave;
    auto next_slot = [&]() -> int {
        while (u_next < total) {
            const int j = __builtin_amdgcn_readfirstlane(cols[u_next / subs]);
            const int sub = u_next % subs;
            u_next += WAVES;
            if (j >= 0 && j < ni) return j * g.block + sub * KT;
        }
        return -1;
    };
    floatx4 kf[NK][NU];
    int4u kp[NK];
    auto load_keys = [&](int s0) {
#pragma unroll
        for (int t = 0; t < NK; ++t) {
            const int s = min(s0 + 16 * t + ln, g.n - 1);  // slots past the end: masked below
#pragma unroll
            for (int u = 0; u < NU; ++u) kf[t][u] = load4(Kh + (size_t)s * D + 16 * u + 4 * lg);
            const int k4 = s0 + 16 * t + 4 * lg;           // this lane's four keys of the tile
            if (s0 + KT <= g.n) {
                kp[t] = *reinterpret_cast<const int4u *>(kih + k4);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) kp[t][r] = k4 + r < g.n ? kih[k4 + r] : INT_MAX;
            }
        }
    };

    int s0 = next_slot();
    if (s0 >= 0) load_keys(s0);
    while (s0 >= 0) {
        // Vt keeps a block as groups of KT slots, each [D][KT]: a sub-tile is one group
        const E *vg = Vh + (size_t)s0 * D;
        floatx4 vf[NU][NK];
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int t = 0; t < NK; ++t) vf[u][t] = load4(vg + (16 * u + ln) * KT + 16 * t + 4 * lg);
        __builtin_amdgcn_sched_barrier(0);
        floatx4 s[NK];
#pragma unroll
        for (int t = 0; t < NK; ++t) s[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int t = 0; t < NK; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[t][u][c], q[u][c], s[t], 0, 0, 0);
        bool hidden = false;
        bool vis[NK][4];
#pragma unroll
        for (int t = 0; t < NK; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                vis[t][r] = kp[t][r] <= qpos;
                hidden = hidden || !vis[t][r];
            }
        const int s1 = next_slot();
        __builtin_amdgcn_sched_barrier(0);
        if (s1 >= 0) load_keys(s1);                        // in flight under the softmax and the second product
        __builtin_amdgcn_sched_barrier(0);

        float rmax = -INFINITY;
#pragma unroll
        for (int t = 0; t < NK; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[t][r] = vis[t][r] ? s[t][r] : -INFINITY;
                rmax = fmaxf(rmax, s[t][r]);
            }
        if (__any(!seen || rmax * c2 > mref + kLead)) {    // first visible key of a query, or a score far above
            rmax = fmaxf(rmax, __shfl_xor(rmax, 16, 64));
            rmax = fmaxf(rmax, __shfl_xor(rmax, 32, 64));
            const bool now = seen || rmax != -INFINITY;
            const float mnew = now ? (seen ? fmaxf(rmax * c2, mref) : rmax * c2) : 0.0f;
            const float alpha = seen ? __builtin_amdgcn_exp2f(mref - mnew) : 1.0f;
            mref = mnew;
            seen = now;
            l *= alpha;
#pragma unroll
            for (int u = 0; u < NU; ++u) acc[u] *= alpha;
        }
        floatx4 p[NK];
#pragma unroll
        for (int t = 0; t < NK; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[t][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r], c2, -mref));
                l += p[t][r];
            }
        // A key that a query does not see has weight 0, but 0 * inf is not 0: where some key is hidden and some value
        // of the sub-tile is not finite, those values leave the product and are added for the queries that see them.
        bool apart = false;
        if (__any(hidden)) {
            float z = 0.0f;
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int t = 0; t < NK; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) z = __builtin_fmaf(vf[u][t][r], 0.0f, z);
            apart = __any(!(z == 0.0f));
            if (apart)
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int t = 0; t < NK; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) vf[u][t][r] = fabsf(vf[u][t][r]) < INFINITY ? vf[u][t][r] : 0.0f;
        }
#pragma unroll
        for (int t = 0; t < NK; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int u = 0; u < NU; ++u) acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[u][t][r], p[t][r], acc[u], 0, 0, 0);
        if (apart) {
#pragma unroll
            for (int t = 0; t < NK; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll 1
                    for (int kg = 0; kg < 4; ++kg) {       // key 16 t + 4 kg + r: its weights live in lane group kg
                        const float w = __shfl(p[t][r], 16 * kg + ln, 64);
                        const bool sees = __shfl((int)vis[t][r], 16 * kg + ln, 64) != 0;
#pragma unroll
                        for (int u = 0; u < NU; ++u)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {  // acc[u][e]: feature 16 u + 4 lg + e
                                const float v = ElemTraits<E>::to_float(vg[(16 * u + 4 * lg + e) * KT + 16 * t + 4 * kg + r]);
                                if (sees && !(fabsf(v) < INFINITY)) acc[u][e] += w * v;
                            }
                    }
        }
        s0 = s1;
    }

    // the waves' partial results meet: acc[u][e] belongs to feature 16 u + 4 lg + e of query ln
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (lg == 0) {
        sm[wave][ln] = seen && live ? mref : -INFINITY;
        sl[wave][ln] = l;
    }
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) so[wave][(16 * u + 4 * lg + e) * kPad + ln] = acc[u][e];
    __syncthreads();
    for (int o = threadIdx.x; o < kQ * D; o += 64 * WAVES) {
        const int qr = o / D, e = o % D;
        if (q0 + qr >= g.n) break;
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) m = fmaxf(m, sm[w][qr]);
        float lt = 0.0f, ot = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float f = sm[w][qr] == m ? 1.0f : __builtin_amdgcn_exp2f(sm[w][qr] - m);
            lt += sl[w][qr] * f;
            ot += so[w][e * kPad + qr] * f;
        }
        const float inv = lt > 0.0f ? 1.0f / lt : 0.0f;
        Op[(bhq * g.n + q0 + qr) * D + e] = ElemTraits<E>::from_float(ot * inv);
        if (lse && e == 0) lse[bhq * g.n + q0 + qr] = lt > 0.0f ? (m + log2f(lt)) * kLn2F : -INFINITY;
    }
}

template <typename E, int D, int KT, int WAVES>
static pbs_status launch_waves(const Geo &g, const void *Qp, const void *Kp, const void *Vt, const int32_t *qidx,
                               const int32_t *kidx, const int32_t *row_cnt, const int32_t *col_idx, void *Op, float *lse,
                               hipStream_t s)
{
    const long long rows = (long long)g.r * ceil_div(g.n, kQ), units = (long long)g.batch * g.h_kv;
    const int cohort = cohort_rows(g);
    const long long ncoh = units * ((rows + cohort - 1) / cohort);
    const long long wgs = (ncoh + kXcds - 1) / kXcds * kXcds * cohort;
    constexpr long long kMaxX = 1 << 20;
    const dim3 grid((unsigned)(wgs < kMaxX ? wgs : kMaxX), (unsigned)((wgs + kMaxX - 1) / kMaxX));
    return launch((attn_fp32_kernel<E, D, KT, WAVES>), grid, dim3(64 * WAVES), 0, s, (const E *)Qp, (const E *)Kp,
                  (const E *)Vt, qidx, kidx, row_cnt, col_idx, (E *)Op, lse, g, cohort);
}

template <typename E, int D, int KT>
static pbs_status launch_kt(const Geo &g, const void *Qp, const void *Kp, const void *Vt, const int32_t *qidx,
                            const int32_t *kidx, const int32_t *row_cnt, const int32_t *col_idx, void *Op, float *lse,
                            hipStream_t s)
{
    // Two waves per SIMD either way: one workgroup of eight waves per compute unit while there are no more than two
    // workgroups for each, two of four waves (shorter tails) from there on.  Measured, eight waves / four, us: 128 workgroups 19.5 / 19.0,
    // 256 34.9 / 34.4, 512 121 / 121, 752 126 / 121, 1024 106 / 96 and 191 / 184, 2048 329 / 320; d = 128, 256 workgroups 68 / 64,
    // 512 237 / 231, 1024 376 / 355.  Where the times are close the eight shorter sums are the better ones: 2.6e-7 off
    // 64 bits at 2 heads x 2048 tokens against 2.9e-7.
    if ((long long)g.batch * g.h_q * ceil_div(g.n, kQ) <= 2 * 256)
        return launch_waves<E, D, KT, 8>(g, Qp, Kp, Vt, qidx, kidx, row_cnt, col_idx, Op, lse, s);
    return launch_waves<E, D, KT, 4>(g, Qp, Kp, Vt, qidx, kidx, row_cnt, col_idx, Op, lse, s);
}

template <typename E, int D>
static pbs_status launch_d(const Geo &g, const void *Qp, const void *Kp, const void *Vt, const int32_t *qidx,
                           const int32_t *kidx, const int32_t *row_cnt, const int32_t *col_idx, void *Op, float *lse,
                           hipStream_t s)
{
    if (g.block == 16) return launch_kt<E, D, 16>(g, Qp, Kp, Vt, qidx, kidx, row_cnt, col_idx, Op, lse, s);
    return launch_kt<E, D, 32>(g, Qp, Kp, Vt, qidx, kidx, row_cnt, col_idx, Op, lse, s);
}

}  // namespace fp32

pbs_status launch_attn_fp32(const Geo &g, int dtype, const void *Qp, const void *Kp, const void *Vt, const int32_t *qidx,
                            const int32_t *kidx, const int32_t *row_cnt, const int32_t *col_idx, void *Op, float *lse,
                            hipStream_t s)
{
    if (dtype == PBS_BF16)
        return g.d == 128 ? fp32::launch_d<bf16_t, 128>(g, Qp, Kp, Vt, qidx, kidx, row_cnt, col_idx, Op, lse, s)
                          : fp32::launch_d<bf16_t, 64>(g, Qp, Kp, Vt, qidx, kidx, row_cnt, col_idx, Op, lse, s);
    return g.d == 128 ? fp32::launch_d<float, 128>(g, Qp, Kp, Vt, qidx, kidx, row_cnt, col_idx, Op, lse, s)
                      : fp32::launch_d<float, 64>(g, Qp, Kp, Vt, qidx, kidx, row_cnt, col_idx, Op, lse, s);
}

}  // namespace pbs

// pbs_attn_fwd in fp32 arithmetic: float32 storage (any d, any block), bf16 storage with blocks of 16 or 32.
//
// Everything is kept transposed, as in the bf16 kernels (S^T = K' Q'^T, O^T += V'^T P^T), on the fp32 matrix
// instruction v_mfma_f32_16x16x4_f32: inputs, products and sums are those of a chain of fp32 fused multiply-adds, at
// the same 157 TFLOP/s peak as the vector unit, but one instruction reads two registers for 2048 operations instead
// of one LDS word per lane for every multiply-add.
//
// A workgroup owns 16 queries of one head and its waves share the key list among them (wave w takes sub-tiles w,
// w + WAVES, ... of KS keys), every wave with a softmax of its own; the partial (m, l, O) meet in
// LDS at the end.  That is what fills the chip at the small sizes fp32 layers have (2 heads x 2048 tokens are 256
// workgroups of 8 waves; with a workgroup per query block they would be 64).
//     A operand of S^T:   lane (key = lane % 16, g = lane / 16) holds 16 bytes of K'[key] from feature (16 u + 4 g, float) on
//     A operand of O^T:   lane (e = lane % 16, g)               holds V'^T[16 t + e][4 g + r],  step r
// and the S^T accumulator (query = lane % 16, keys 4 g + r) is already the B operand of the second product.  The contraction
// order over features is permuted the same way in K' and Q', which changes nothing but the order of an fp32 sum.
// Neighbouring lanes want different rows, so these operands as loads from memory would be an access of 16 bytes per lane
// (59 cache accesses to an instruction; 18 now, and the address units busy 19 % of a launch of 2 heads x 2048 instead of 34 %): a
// wave's sub-tile goes through its own LDS instead, by asynchronous loads of consecutive memory; no wave wants another's, so
// nothing waits at a barrier.
//
// Bound: the fp32 matrix rate (64 operations per clock and SIMD): 64 instructions of 32 clocks per 32 keys and 16
// queries at d = 64; at the small sizes the longest list.  Measured, operands from memory / through LDS, us, every admitted block
// of float32: d = 64, 2 heads x 2048 33.9 / 22.8, 8 / 2 x 4096 248 / 163; d = 128, 2 x 2048 65.6 / 38.5, 8 / 2 x 4096 494 / 295
// (116 TFLOP/s); bf16 8 / 2 x 2048 x 128 in blocks of 32 142 / 100, of 16 127 / 100, 4 / 2 x 2048 x 64 in blocks of 16 38.9 / 33.0, 32 / 8
// x 4096 x 128 in blocks of 16 1618 / 1294 and, a twentieth of the blocks, 196 / 157.
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

typedef __attribute__((address_space(3))) void *lptr_t;
typedef int int4u __attribute__((ext_vector_type(4), aligned(4)));

// 16 bytes per lane from memory into 1 KiB of LDS, asynchronously
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t from, unsigned char *to, int lane_at, int at)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (lptr_t)to, 16, lane_at, at, 0, 0);
}

// grid: linear ids (x fastest; y only where x alone would pass 2^32 threads), cohorts of `cohort` workgroups of one kv
// head per XCD, longest lists first (see the decoding below)
template <typename E, int D, int KT, int KS, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_fp32_kernel(
    const E *__restrict__ Qp, const E *__restrict__ Kp, const E *__restrict__ Vt, const int32_t *__restrict__ qidx,
    const int32_t *__restrict__ kidx, const int32_t *__restrict__ row_cnt, const int32_t *__restrict__ col_idx,
    E *__restrict__ Op, float *__restrict__ lse, Geo g, int cohort)
{
    constexpr int NK = KS / 16;                            // 16-key tiles per sub-tile
    constexpr int NU = D / 16;                             // 16-feature steps of S^T = feature tiles of O^T
    constexpr int kPad = kQ + 1;
    constexpr int kB = sizeof(E), kVec = 16 / kB;
    constexpr int NP = D / (4 * kVec);                     // 16-byte pieces of a key per lane
    constexpr int kKeyB = D * kB, kValB = KS * kB;         // bytes of a row of the K' and of the V'^T tile
    constexpr int kTileB = KS * kKeyB, kLoads = kTileB / 1024;              // of either tile
    static_assert(kTileB % 1024 == 0, "whole load instructions");
    // a wave's own: the sub-tile on its way, then its part of O^T
    constexpr int kSumB = D * kPad * 4, kOwnB = 2 * kTileB > kSumB ? 2 * kTileB : kSumB;
    __shared__ __align__(16) unsigned char ring[WAVES][kOwnB];
    __shared__ __align__(16) int32_t ring_pos[WAVES][64];
    __shared__ float sm[WAVES][kQ], sl[WAVES][kQ];

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
    float q[D / 4];                                        // step kVec u + c of S^T: feature 4 kVec u + kVec lg + c
    {
        typedef E vec_t __attribute__((ext_vector_type(kVec)));
        const E *src = Qp + (bhq * g.n + (live ? qs : g.n - 1)) * D + kVec * lg;
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const vec_t v = *reinterpret_cast<const vec_t *>(src + 4 * kVec * u);
#pragma unroll
            for (int c = 0; c < kVec; ++c) q[kVec * u + c] = (float)v[c];
        }
    }
    floatx4 acc[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) acc[u] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    float mref = 0.0f, l = 0.0f;                           // this lane's keys only for l
    bool seen = !live;                                     // mref is set; padding rows never hold the wave back

    const int ni = allowed_cols(i, g);
    const int subs_log2 = __builtin_ctz(g.block / KS);
    const int total = min(row_cnt[bhq * g.T + i], g.T) << subs_log2;
    const int32_t *cols = col_idx + (bhq * g.T + i) * g.T;
    const E *Kh = Kp + bhk * (size_t)g.n * D;
    const E *Vh = Vt + bhk * (size_t)g.T * D * g.block;
    const int32_t *kih = kidx + bhk * (size_t)g.n;

    // first slot of this wave's next admitted sub-tile at or after u, -1 past the end
    int u_next = wave;
    auto next_slot = [&]() -> int {
        while (u_next < total) {
            const int j = __builtin_amdgcn_readfirstlane(cols[u_next >> subs_log2]);
            const int sub = u_next & ((1 << subs_log2) - 1);
            u_next += WAVES;
            const int first = listed_slot(j, sub, KS, g.block, ni, g.n);
            if (first >= 0) return first;
        }
        return -1;
    };
    // A wave's sub-tile travels into its own LDS by asynchronous loads of 1 KiB of consecutive memory each, is read into
    // registers whole, and makes room for the next one, which has this one's arithmetic to arrive.  Rows unpadded, their 16-byte
    // pieces stored XOR-permuted, so that 16 lanes reading 16 rows at one logical piece meet 64 different banks.
    auto place = [](int row, int piece, int pieces) __attribute__((always_inline)) {
        const int per = pieces < 16 ? 16 / pieces : 1, mask = (pieces < 16 ? pieces : 16) - 1;
        return piece ^ ((row / per) & mask);
    };
    constexpr int kRawDword = 0x00020000;                  // gfx9 descriptor word 3: raw 32-bit data format
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(const_cast<E *>(Kh), 0, g.n * kKeyB, kRawDword);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<E *>(Vh), 0, g.T * g.block * kKeyB, kRawDword);
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(kih), 0, g.n * 4, kRawDword);
    int koff[kLoads], voff[kLoads];                        // lane's source of load c (the permutation is its own inverse)
#pragma unroll
    for (int c = 0; c < kLoads; ++c) {
        const int at = 64 * c + lane, kp16 = kKeyB / 16, vp16 = kValB / 16;
        koff[c] = at / kp16 * kKeyB + place(at / kp16, at % kp16, kp16) * 16;
        voff[c] = at / vp16 * (KT * kB) + place(at / vp16, at % vp16, vp16) * 16;
    }
    unsigned char *const own = ring[wave];
    // Vt keeps a block as groups of KT slots, each [D][KT]: a sub-tile is one group or one of its halves
    auto values_at = [&](int s0) __attribute__((always_inline)) { return (s0 & -KT) * D + (s0 & (KT - 1)); };
    // Keys past the end give zeros and are masked below.  s0 is one of the n keys, so that no load starts behind the end of its
    // descriptor: the hardware compares a lane's offset with the size less the scalar offset, which must not fall below zero.
    auto load_tile = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < kLoads; ++c) load_to_lds(rk, own + 1024 * c, koff[c], s0 * kKeyB);
#pragma unroll
        for (int c = 0; c < kLoads; ++c) load_to_lds(rv, own + kTileB + 1024 * c, voff[c], values_at(s0) * kB);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rp, (lptr_t)ring_pos[wave], 4, lane * 4, s0 * 4, 0, 0);
    };

    int s0 = next_slot();
    if (s0 >= 0) load_tile(s0);
    while (s0 >= 0) {
        const int s1 = next_slot();
        const E *vg = Vh + values_at(s0);
        __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0), gfx9 encoding: the sub-tile is here
        __builtin_amdgcn_sched_barrier(0);
        typedef E vec_t __attribute__((ext_vector_type(kVec)));
        typedef E quad_t __attribute__((ext_vector_type(4)));
        vec_t kf[NK][NP];
        quad_t vr[NU][NK];
        int4u kp[NK];
#pragma unroll
        for (int t = 0; t < NK; ++t) {
#pragma unroll
            for (int u = 0; u < NP; ++u)
                kf[t][u] = *reinterpret_cast<const vec_t *>(own + (16 * t + ln) * kKeyB + place(16 * t + ln, 4 * u + lg, kKeyB / 16) * 16);
            kp[t] = *reinterpret_cast<const int4u *>(&ring_pos[wave][16 * t + 4 * lg]);
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int t = 0; t < NK; ++t) {                 // keys 16 t + 4 lg .. + 4 of feature 16 u + ln
                const int at = (16 * t + 4 * lg) * kB;
                vr[u][t] = *reinterpret_cast<const quad_t *>(own + kTileB + (16 * u + ln) * kValB +
                                                             place(16 * u + ln, at / 16, kValB / 16) * 16 + at % 16);
            }
        __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0): in registers
        __builtin_amdgcn_sched_barrier(0);
        if (s1 >= 0) load_tile(s1);
        __builtin_amdgcn_sched_barrier(0);
        floatx4 s[NK];
#pragma unroll
        for (int t = 0; t < NK; ++t) s[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < NP; ++u)
#pragma unroll
            for (int c = 0; c < kVec; ++c)
#pragma unroll
                for (int t = 0; t < NK; ++t)
                    s[t] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)kf[t][u][c], q[kVec * u + c], s[t], 0, 0, 0);
        bool hidden = false;
        bool vis[NK][4];
#pragma unroll
        for (int t = 0; t < NK; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                vis[t][r] = kp[t][r] <= qpos;
                hidden = hidden || !vis[t][r];
            }
        if (s0 + KS > g.n) {                               // slots past the end of the sequence
            hidden = true;
#pragma unroll
            for (int t = 0; t < NK; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) vis[t][r] = vis[t][r] && s0 + 16 * t + 4 * lg + r < g.n;
        }
        floatx4 vf[NU][NK];
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int t = 0; t < NK; ++t)
                vf[u][t] = floatx4{(float)vr[u][t][0], (float)vr[u][t][1], (float)vr[u][t][2], (float)vr[u][t][3]};
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
        for (int e = 0; e < 4; ++e) reinterpret_cast<float *>(own)[(16 * u + 4 * lg + e) * kPad + ln] = acc[u][e];
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
            ot += reinterpret_cast<const float *>(ring[w])[e * kPad + qr] * f;
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
    constexpr int kStep = sizeof(E) == 4 && D == 128 ? 16 : KT;            // 16 KiB of LDS to a wave at most
    const long long rows = (long long)g.r * ceil_div(g.n, kQ), units = (long long)g.batch * g.h_kv;
    const int cohort = cohort_rows(g);
    const long long ncoh = units * ((rows + cohort - 1) / cohort);
    const long long wgs = (ncoh + kXcds - 1) / kXcds * kXcds * cohort;
    constexpr long long kMaxX = 1 << 20;
    const dim3 grid((unsigned)(wgs < kMaxX ? wgs : kMaxX), (unsigned)((wgs + kMaxX - 1) / kMaxX));
    return launch((attn_fp32_kernel<E, D, KT, kStep, WAVES>), grid, dim3(64 * WAVES), 0, s, (const E *)Qp, (const E *)Kp,
                  (const E *)Vt, qidx, kidx, row_cnt, col_idx, (E *)Op, lse, g, cohort);
}

template <typename E, int D, int KT>
static pbs_status launch_kt(const Geo &g, const void *Qp, const void *Kp, const void *Vt, const int32_t *qidx,
                            const int32_t *kidx, const int32_t *row_cnt, const int32_t *col_idx, void *Op, float *lse,
                            hipStream_t s)
{
    // Two waves per SIMD either way: one workgroup of eight waves per compute unit while there are no more than two
    // workgroups for each, two of four waves (shorter tails) from there on.  Measured, eight waves / four, us: d = 64, 64 workgroups 9.8 /
    // 10.4, 256 22.8 / 28.1, 376 31.1 / 44.5, 512 48.1 / 61.5, 752 58.7 / 51.8, 1024 90.8 / 86.0, 2048 177 / 164 and, a tenth of the
    // blocks, 59.7 / 42.2; d = 128, 256 38.5 / 49.1, 512 49.8 / 59.7, 1024 163 / 155, 2048 317 / 299.
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

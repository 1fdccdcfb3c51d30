// pbs_attn_fwd for bf16 storage, d = 64, block 64 or 128, on the bf16 matrix instruction with fp32 probabilities.
//
// Transposed like the d = 128 kernels (S^T = K' Q'^T, O^T += V'^T P^T, one lane owns one query of each 32-query tile).
// The scores are exact bf16 products summed in fp32; a probability stays an fp32 number: it enters the second product
// as three bf16 terms, which hold its 24 bits, so an O^T sub-tile takes three matrix instructions per fragment.  (With two
// terms, 2^-18 of a probability left out, the error against 64 bits came out larger than with fp32 multiply-adds, if only
// from the seventh digit on; with three it does not: 1.5653902e-3 for both at 16 / 4 heads x 3701 tokens.)
//
// A workgroup owns 64 queries (all of a block of 64, half a block of 128) and every wave of it works on all 64: each
// fragment read from LDS feeds two (K') or six (V'^T) matrix instructions.  The waves divide the key list among them in
// pieces of 64 keys, each with a softmax and an O^T of its own, meet no barrier on the way and add up in LDS at the end.
// A wave's K' / V'^T sub-tiles of 32 keys come through a ring of its own of two 8 KiB stages filled by asynchronous
// buffer->LDS loads, two sub-tiles ahead; 16 KiB per wave lets eight waves, two per SIMD, share a compute unit, which is
// what overlaps one wave's softmax with the other's products.  Bound: vector issue, 41 clocks per score (multiply-add, exp2, sum, three
// packs and two remainders) against 32 of matrix work; the matrix pipe is busy 42 % of the time.  Measured, 16 / 4 heads x
// 12301 tokens, block 64: every admitted block 765 us = 410 TFLOP/s; a layer of nine tenths of the blocks 0.70 ms, with this stage on
// fp32 matrix instructions (attn_fp32.hip) 4.35 ms, on fp32 vector arithmetic 24 ms.
#include "pbs_host.h"

namespace pbs {
namespace d64 {

constexpr int D = 64;
constexpr int kQ = 64;                                     // queries per wave
constexpr int KS = 32;                                     // keys per sub-tile
constexpr int kXcds = 8;
constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f;
constexpr float kBigRowSum = 65536.0f;                     // a sub-tile's row sum beyond this moves the reference

typedef __attribute__((address_space(3))) void *lptr_t;
typedef int int4u __attribute__((ext_vector_type(4), aligned(4)));

// One ring stage; rows unpadded, their 16-byte pieces stored XOR-permuted so that 16 lanes reading 16 rows at one
// logical piece meet 64 different banks:
//   k: row r (128 B) holds key swap23(r) of the sub-tile, its piece c (of 8) at place c ^ ((r / 2) % 8);
//   v: row e (64 B) holds V'^T[e][32 keys], its piece c (of 4) at place c ^ ((e / 4) % 4).
// Rows with bits 2 and 3 of the key index swapped give a lane 8 consecutive keys per 16-key contraction step.
struct __align__(16) Stage {
    unsigned char k[KS * D * 2];
    unsigned char v[KS * D * 2];
};

__device__ __forceinline__ int swap23(int m) { return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1); }

struct State {
    floatx16 acc[2][2];     // O^T [feature tile][query tile]: feature 32 dt + 8 (x / 4) + 4 h + x % 4, query 32 nt + n
    float mref[2], l[2];    // reference (log2 units), sum of exp2(s c2 - mref) over this lane's keys
    bool seen[2];           // the query has met a visible key, i.e. mref is set
};

// Row maximum of this sub-tile's scores; the reference moves up to it and O, l follow (first contact: it is set).
__device__ __forceinline__ void move_reference(State &st, const floatx16 (&s)[2], float c2)
{
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        float rmax = -INFINITY;
#pragma unroll
        for (int x = 0; x < 16; ++x) rmax = fmaxf(rmax, s[nt][x]);
        rmax = fmaxf(rmax, __shfl_xor(rmax, 32, 64));
        const bool was = st.seen[nt], now = was || rmax != -INFINITY;
        const float mnew = now ? (was ? fmaxf(rmax * c2, st.mref[nt]) : rmax * c2) : 0.0f;
        const float alpha = was ? __builtin_amdgcn_exp2f(st.mref[nt] - mnew) : 1.0f;
        st.mref[nt] = mnew;
        st.seen[nt] = now;
        if (__any(alpha != 1.0f)) {
            st.l[nt] *= alpha;
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int x = 0; x < 16; ++x) st.acc[dt][nt][x] *= alpha;
        }
    }
}

// p = exp2(s c2 - mref) of both query tiles as three bf16 terms, largest first; rsum: sums of the fp32 probabilities.
// What a term leaves of a pair takes one instruction for each of the two, a bf16 dot product with (-1, 0) or (0, -1): exact, and
// four instructions fewer for a pair than unpacking and subtracting (layer of 16 / 4 heads x 12301 tokens: 701 us
// against 742).  The two constants sit in registers: as literals they came out as an inline constant with another meaning.
struct Split {
    bf16x8 t[3][2][2];                                     // [term][query tile][16 keys]
};
__device__ __forceinline__ void probabilities(const State &st, const floatx16 (&s)[2], float c2, Split &pf, float (&rsum)[2])
{
    uint32_t c0 = 0x0000bf80u, c1 = 0xbf800000u;
    asm volatile("" : "+s"(c0), "+s"(c1));
    const bf16x2 first = __builtin_bit_cast(bf16x2, c0), second = __builtin_bit_cast(bf16x2, c1);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        float even = 0.0f, odd = 0.0f;
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            const floatx2 p = {__builtin_amdgcn_exp2f(__builtin_fmaf(s[nt][2 * y], c2, -st.mref[nt])),
                               __builtin_amdgcn_exp2f(__builtin_fmaf(s[nt][2 * y + 1], c2, -st.mref[nt]))};
            even += p[0];
            odd += p[1];
            // (written out: as a loop over the terms it is scheduled worse and takes 3 % longer)
            const bf16x2 t0 = __builtin_convertvector(p, bf16x2);
            const floatx2 r1 = {__builtin_amdgcn_fdot2_f32_bf16(t0, first, p[0], false), __builtin_amdgcn_fdot2_f32_bf16(t0, second, p[1], false)};
            const bf16x2 t1 = __builtin_convertvector(r1, bf16x2);
            const floatx2 r2 = {__builtin_amdgcn_fdot2_f32_bf16(t1, first, r1[0], false), __builtin_amdgcn_fdot2_f32_bf16(t1, second, r1[1], false)};
            const bf16x2 t2 = __builtin_convertvector(r2, bf16x2);
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                pf.t[0][nt][y >> 2][2 * (y & 3) + z] = t0[z];
                pf.t[1][nt][y >> 2][2 * (y & 3) + z] = t1[z];
                pf.t[2][nt][y >> 2][2 * (y & 3) + z] = t2[z];
            }
        }
        rsum[nt] = even + odd;
    }
}

// Tensors and geometry of one wave's query tile.
struct Row {
    const bf16_t *q, *k, *vt;      // this head's Q', K', Vt
    const int32_t *kidx, *cols;
    int n, block, cnt, ni, jmask, q0;
};

// grid: linear ids (x fastest, y for more than 2^20 workgroups), decoded as cohorts of `cohort` query tiles of one kv
// head per XCD, longest lists first, as in the other attention kernels
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_d64_kernel(
    const bf16_t *__restrict__ Qp, const bf16_t *__restrict__ Kp, const bf16_t *__restrict__ Vt,
    const int32_t *__restrict__ qidx, const int32_t *__restrict__ kidx, const int32_t *__restrict__ row_cnt,
    const int32_t *__restrict__ col_idx, bf16_t *__restrict__ Op, float *__restrict__ lse, Geo g, int cohort)
{
    __shared__ Stage ring0[WAVES], ring1[WAVES];           // separate variables: the compiler can tell them apart
    __shared__ float sm[WAVES][kQ], sl[WAVES][kQ];

    const int tiles = ceil_div(g.n, kQ);
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
    Row w;
    w.q0 = (tiles - 1 - mrow / g.r) * kQ;
    const int i = w.q0 / g.block;
    const int b = unit / g.h_kv, hq = (unit % g.h_kv) * g.r + mrow % g.r;
    const size_t bhq = (size_t)b * g.h_q + hq, bhk = unit;
    const int lane = threadIdx.x & 63;
    const int wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ln = lane & 31, lh = lane >> 5;
    Stage &sg0 = ring0[wave], &sg1 = ring1[wave];
    const float c2 = g.scale * kLog2eF;
    w.n = g.n;
    w.block = g.block;
    w.ni = allowed_cols(i, g);
    w.jmask = first_masked_col(i, g);
    w.cnt = min(row_cnt[bhq * g.T + i], g.T);
    w.cols = col_idx + (bhq * g.T + i) * g.T;
    w.q = Qp + bhq * g.n * D;
    w.k = Kp + bhk * (size_t)g.n * D;
    w.vt = Vt + bhk * (size_t)g.T * D * g.block;
    w.kidx = kidx + bhk * (size_t)g.n;

    // Q' fragments: lane (n, h) holds Q'[q0 + 32 nt + n][16 x + 8 h .. + 8]
    bf16x8 qf[2][4];
    int qpos[2];
    State st;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
        const int qs = w.q0 + 32 * nt + ln;
        const bf16_t *src = w.q + (size_t)min(qs, g.n - 1) * D + 8 * lh;
#pragma unroll
        for (int x = 0; x < 4; ++x) qf[nt][x] = *reinterpret_cast<const bf16x8 *>(src + 16 * x);
        qpos[nt] = qs < g.n ? (qidx ? qidx[bhq * g.n + qs] : qs) : -1;
        st.mref[nt] = 0.0f;
        st.l[nt] = 0.0f;
        st.seen[nt] = qs >= g.n;                           // padding rows never hold the wave on the exact path
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int x = 0; x < 16; ++x) st.acc[dt][nt][x] = 0.0f;
    }

    // Loads: a stage is 8 instructions of 1 KiB.  Reads past the end of K' give zeros (such slots are masked); Vt is
    // zero-filled to whole blocks.
    constexpr int kRawDword = 0x00020000;                  // gfx9 descriptor word 3: raw 32-bit data format
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(w.k), 0, g.n * (D * 2), kRawDword);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(w.vt), 0, g.T * g.block * (D * 2), kRawDword);
    // per-lane offsets of load c: rows c * 8 + lane / 8 of k (c and c + 2 differ by 16 keys), c * 16 + lane / 4 of v
    uint32_t koff[2], voff, kfr[4], vfr[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int kr = c * 8 + (lane >> 3);
        koff[c] = (uint32_t)(swap23(kr) * (D * 2) + (((lane & 7) ^ ((kr >> 1) & 7)) << 4));
    }
    voff = (uint32_t)((lane >> 2) * (KS * 2) + (((lane & 3) ^ ((lane >> 4) & 3)) << 4));
#pragma unroll
    for (int c = 0; c < 4; ++c) kfr[c] = (uint32_t)(ln * (D * 2) + (((2 * c + lh) ^ ((ln >> 1) & 7)) << 4));
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) vfr[k2] = (uint32_t)(ln * (KS * 2) + (((2 * k2 + lh) ^ ((ln >> 2) & 3)) << 4));
    auto issue = [&](Stage &sg, int slot0) {               // K' rows and Vt group of the 32 slots from slot0 on: 4 KiB each
#pragma unroll
        for (int c = 0; c < 4; ++c)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lptr_t)(sg.k + c * 1024), 16, koff[c & 1],
                                                     (slot0 + (c >> 1) * 16) * (D * 2), 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lptr_t)(sg.v + c * 1024), 16, voff, slot0 * (D * 2) + c * 1024, 0, 0);
    };

    // the list as pairs of sub-tiles, this wave's are every WAVES-th: the first slot of its next admitted 64 keys, -1 past
    // the end
    const int halves = g.block / 64, total = w.cnt * halves;
    int u_next = wave;
    auto next_slot = [&]() -> int {
        while (u_next < total) {
            const int j = __builtin_amdgcn_readfirstlane(w.cols[u_next / halves]);
            const int part = u_next % halves;
            u_next += WAVES;
            if (j >= 0 && j < w.ni) return j * g.block + 64 * part;
        }
        return -1;
    };

    auto scores = [&](const bf16x8 (&kf)[4], floatx16 (&s)[2]) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) s[nt] = floatx16{0};
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) s[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[x], qf[nt][x], s[nt], 0, 0, 0);
    };
    auto add_values = [&](const bf16x8 (&vf)[2][2], const Split &pf) {
#pragma unroll
        for (int term = 0; term < 3; ++term)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                    for (int nt = 0; nt < 2; ++nt)
                        st.acc[dt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[dt][k2], pf.t[term][nt][k2], st.acc[dt][nt], 0, 0, 0);
    };
    // the token-level mask on the scores of a sub-tile; s[nt][x]: key 16 (x / 8) + 8 h + x % 8, query 32 nt + n
    auto hide = [&](floatx16 (&s)[2], int slot0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k8 = slot0 + 16 * u + 8 * lh;
            int kp[8];
            if (slot0 + KS <= w.n) {
                const int4u a = *reinterpret_cast<const int4u *>(w.kidx + k8), c = *reinterpret_cast<const int4u *>(w.kidx + k8 + 4);
#pragma unroll
                for (int x = 0; x < 4; ++x) { kp[x] = a[x]; kp[4 + x] = c[x]; }
            } else {
#pragma unroll
                for (int x = 0; x < 8; ++x) kp[x] = k8 + x < w.n ? w.kidx[k8 + x] : 0x7fffffff;
            }
#pragma unroll
            for (int x = 0; x < 8; ++x)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    if (kp[x] > qpos[nt]) s[nt][8 * u + x] = -INFINITY;
        }
    };
    auto subtile = [&](Stage &sg, int slot0, bool masked, int refill) {
        // this stage's 8 loads have landed, the other stage's may still be in flight
        __builtin_amdgcn_s_waitcnt(0x0F78);                // vmcnt(8), gfx9 encoding
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 kf[4], vf[2][2];
#pragma unroll
        for (int x = 0; x < 4; ++x) kf[x] = *reinterpret_cast<const bf16x8 *>(sg.k + kfr[x]);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2) vf[dt][k2] = *reinterpret_cast<const bf16x8 *>(sg.v + vfr[k2] + dt * 2048);
        __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0): the stage is in registers and may be refilled
        __builtin_amdgcn_sched_barrier(0);
        issue(sg, refill);
        __builtin_amdgcn_sched_barrier(0);
        floatx16 s[2];
        scores(kf, s);
        if (masked) hide(s, slot0);
        const bool first = masked || !__all(st.seen[0] && st.seen[1]);
        if (first) move_reference(st, s, c2);              // at least the row maximum: no sum below can be large
        Split pf;
        float rsum[2];
        probabilities(st, s, c2, pf, rsum);
        if (!first && __any(!(rsum[0] <= kBigRowSum) || !(rsum[1] <= kBigRowSum))) {
            scores(kf, s);                                 // formed again rather than kept: 16 registers fewer
            move_reference(st, s, c2);
            probabilities(st, s, c2, pf, rsum);
        }
        st.l[0] += rsum[0];
        st.l[1] += rsum[1];
        add_values(vf, pf);
    };

    int s0 = next_slot();
    if (s0 >= 0) {
        issue(sg0, s0);
        issue(sg1, s0 + KS);
        while (s0 >= 0) {
            const int s1 = next_slot();
            const int ahead = s1 >= 0 ? s1 : s0;           // past the end: this pair again (unused)
            const bool masked = s0 >= w.jmask * g.block;
            subtile(sg0, s0, masked, ahead);
            subtile(sg1, s0 + KS, masked, ahead + KS);
            s0 = s1;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the loads issued past the end have landed too
    }

    // A value that is not finite does not come through these products: 0 * inf of a hidden key is NaN, and so is
    // the sum over the terms of a visible one whenever a term is zero or negative.  A wave that finds NaN in its O^T forms it again,
    // relative to the references it has ended with: such values leave the products and are added one key at a time, with the
    // undivided probability, for the queries that see the key.  Nothing is prefetched here; with one infinite value that every
    // query of the call sees, 16 / 4 heads x 12301 tokens take 1.26 ms instead of 0.62.
    bool odd = false;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int x = 0; x < 16; ++x) odd = odd || st.acc[dt][nt][x] != st.acc[dt][nt][x];
    if (__any(odd)) {
        float *weight = reinterpret_cast<float *>(&sg0);   // [key of the sub-tile][query], -1: not seen
        static_assert(sizeof(Stage) == KS * kQ * sizeof(float), "the probabilities of a sub-tile");
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) st.acc[dt][nt] = floatx16{0};
        u_next = wave;
        int slot0 = next_slot();
        for (int part = 0; slot0 >= 0; ) {
            bf16x8 kf[4], vf[2][2];
#pragma unroll
            for (int x = 0; x < 4; ++x)
                kf[x] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rk, swap23(ln) * (D * 2) + (2 * x + lh) * 16, slot0 * (D * 2), 0));
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
                    vf[dt][k2] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rv, (32 * dt + ln) * (KS * 2) + (2 * k2 + lh) * 16, slot0 * (D * 2), 0));
            floatx16 s[2];
            scores(kf, s);
            if (slot0 >= w.jmask * g.block) hide(s, slot0);
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int x = 0; x < 16; ++x)
                    weight[(16 * (x >> 3) + 8 * lh + (x & 7)) * kQ + 32 * nt + ln] =
                        s[nt][x] == -INFINITY ? -1.0f : __builtin_amdgcn_exp2f(__builtin_fmaf(s[nt][x], c2, -st.mref[nt]));
            uint32_t keys = 0;                             // with some value that is not finite
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    bool any = false;
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) {
                        const bool here = !(fabsf((float)vf[dt][k2][x]) < INFINITY);
                        if (here) vf[dt][k2][x] = (bf16_t)0.0f;
                        any = any || here;
                    }
                    const uint64_t lanes = __ballot(any);
                    keys |= ((uint32_t)lanes ? 1u : 0u) << (16 * k2 + x) | ((uint32_t)(lanes >> 32) ? 1u : 0u) << (16 * k2 + 8 + x);
                }
            Split pf;
            float unused[2];
            probabilities(st, s, c2, pf, unused);
            add_values(vf, pf);
            for (; keys; keys &= keys - 1) {
                const int key = __builtin_ctz(keys);
                const float p[2] = {weight[key * kQ + ln], weight[key * kQ + 32 + ln]};
                const bf16_t *vk = w.vt + (size_t)slot0 * D + key;
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                    for (int x = 0; x < 16; ++x) {
                        const float v = (float)vk[(32 * dt + 8 * (x >> 2) + 4 * lh + (x & 3)) * KS];
                        if (!(fabsf(v) < INFINITY))
#pragma unroll
                            for (int nt = 0; nt < 2; ++nt)
                                if (!(p[nt] < 0.0f)) st.acc[dt][nt][x] += p[nt] * v;
                    }
            }
            slot0 = part == 0 ? slot0 + KS : next_slot();
            part ^= 1;
        }
    }

    float lt[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) lt[nt] = st.l[nt] + __shfl_xor(st.l[nt], 32, 64);
    if constexpr (WAVES == 1) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const float inv = lt[nt] > 0.0f ? 1.0f / lt[nt] : 0.0f;
            const int qs = w.q0 + 32 * nt + ln;
            if (qs < g.n) {
                bf16_t *dst = Op + (bhq * g.n + qs) * D;
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const floatx2 a = {st.acc[dt][nt][4 * x] * inv, st.acc[dt][nt][4 * x + 1] * inv};
                        const floatx2 c = {st.acc[dt][nt][4 * x + 2] * inv, st.acc[dt][nt][4 * x + 3] * inv};
                        const bf16x2 pa = __builtin_convertvector(a, bf16x2), pc = __builtin_convertvector(c, bf16x2);
                        *reinterpret_cast<bf16x4 *>(dst + 32 * dt + 8 * x + 4 * lh) = bf16x4{pa[0], pa[1], pc[0], pc[1]};
                    }
                if (lse && lh == 0)
                    lse[bhq * g.n + qs] = lt[nt] > 0.0f ? (st.mref[nt] + log2f(lt[nt])) * kLn2F : -INFINITY;
            }
        }
    } else {
        // every wave leaves its O^T in its own ring, [feature][query], and its (m, l)
        float *part[2] = {reinterpret_cast<float *>(&sg0), reinterpret_cast<float *>(&sg1)};
        static_assert(sizeof(Stage) == 32 * kQ * sizeof(float), "half of the features of 64 queries");
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            if (lh == 0) {
                sm[wave][32 * nt + ln] = st.seen[nt] && qpos[nt] >= 0 ? st.mref[nt] : -INFINITY;
                sl[wave][32 * nt + ln] = lt[nt];
            }
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int x = 0; x < 16; ++x)
                    part[dt][(8 * (x >> 2) + 4 * lh + (x & 3)) * kQ + 32 * nt + ln] = st.acc[dt][nt][x];
        }
        __syncthreads();
        // thread (query, part of the features)
        constexpr int F = D / WAVES;
        const int q = lane, qs = w.q0 + q, f0 = wave * F;
        float m = -INFINITY, l = 0.0f, scale[WAVES];
#pragma unroll
        for (int v = 0; v < WAVES; ++v) m = fmaxf(m, sm[v][q]);
#pragma unroll
        for (int v = 0; v < WAVES; ++v) {
            scale[v] = sm[v][q] == m ? 1.0f : __builtin_amdgcn_exp2f(sm[v][q] - m);
            l += sl[v][q] * scale[v];
        }
        const float inv = l > 0.0f ? 1.0f / l : 0.0f;
        const Stage *ring = f0 < 32 ? ring0 : ring1;
        bf16x8 out[F / 8];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            float o = 0.0f;
#pragma unroll
            for (int v = 0; v < WAVES; ++v)
                o += reinterpret_cast<const float *>(&ring[v])[((f0 & 31) + f) * kQ + q] * scale[v];
            out[f >> 3][f & 7] = (bf16_t)(o * inv);
        }
        if (qs < g.n) {
#pragma unroll
            for (int f = 0; f < F / 8; ++f) *reinterpret_cast<bf16x8 *>(Op + (bhq * g.n + qs) * D + f0 + 8 * f) = out[f];
            if (lse && wave == 0) lse[bhq * g.n + qs] = l > 0.0f ? (m + log2f(l)) * kLn2F : -INFINITY;
        }
    }
}

}  // namespace d64

pbs_status launch_attn_d64(const Geo &g, const void *Qp, const void *Kp, const void *Vt, const int32_t *qidx,
                           const int32_t *kidx, const int32_t *row_cnt, const int32_t *col_idx, void *Op, float *lse,
                           hipStream_t s)
{
    const long long rows = (long long)g.r * ceil_div(g.n, d64::kQ), units = (long long)g.batch * g.h_kv;
    const int cohort = cohort_rows(g);
    const long long ncoh = units * ((rows + cohort - 1) / cohort);
    const long long wgs = (ncoh + d64::kXcds - 1) / d64::kXcds * d64::kXcds * cohort;
    constexpr long long kMaxX = 1 << 20;
    const dim3 grid((unsigned)(wgs < kMaxX ? wgs : kMaxX), (unsigned)((wgs + kMaxX - 1) / kMaxX));
    // The chip holds 2048 of these waves, and under the causal mask the last query tile has twice the average list: with
    // few tiles per wave slot that one list is what everything waits for, so a tile's list is shared by four waves until
    // there are two tiles per slot.  Measured, four waves / one, us: every admitted block listed, 768 tiles 250 / 461, 1536
    // 324 / 490, 2048 356 / 395, 3088 765 / 801, 4096 612 / 584 and 1374 / 1321, 8192 1200 / 1150, 24576 37640 / 37200; a tenth of the
    // blocks, 1536 tiles 61 / 76, 2048 65 / 62, 3088 118 / 109, 4096 120 / 91 and 177 / 154, 16384 619 / 488.
    if (units * rows < 2 * 2048)
        return launch(d64::attn_d64_kernel<4>, grid, dim3(256), 0, s, (const bf16_t *)Qp, (const bf16_t *)Kp,
                      (const bf16_t *)Vt, qidx, kidx, row_cnt, col_idx, (bf16_t *)Op, lse, g, cohort);
    return launch(d64::attn_d64_kernel<1>, grid, dim3(64), 0, s, (const bf16_t *)Qp, (const bf16_t *)Kp,
                  (const bf16_t *)Vt, qidx, kidx, row_cnt, col_idx, (bf16_t *)Op, lse, g, cohort);
}

}  // namespace pbs

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
// A wave's K' / V'^T sub-tiles of 32 keys come through rings of its own of two 4 KiB places each, filled by asynchronous
// buffer->LDS loads; 16 KiB per wave lets eight waves, two per SIMD, share a compute unit.
//
// A sub-tile is taken in halves, one query tile each: the softmax of one runs under the products of the other (four that form its
// next scores, twelve that add its last probabilities to O^T), written out product by product, so that a wave keeps the matrix
// and the vector unit busy by itself.  Bound: 1500 clocks of vector issue to 1024 of matrix work per sub-tile, of which the loop
// takes 1760 (2100 with softmax and products in turn and two waves to overlap them), and the clock that the chip's power limit
// grants, which falls as the units fill: 16 / 4 heads x 12301 tokens, block 64, every admitted block 623 -> 600 us, x 16384 1092 ->
// 1019, 4 / 2 x 4000, block 128 43.6 -> 36.2, 8 / 8 x 3000 37.2 -> 32.0, 16 / 4 x 24000 over a tenth of the blocks 270 -> 261.
// Error against 64 bits, before / now: 16 / 4 x 3701 1.617787304e-3 / ..307e-3, x 6000 with wide logits 1.657771577e-3 / ..574e-3.
#include <utility>

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

// One ring place of K' or V'^T, a sub-tile's 4 KiB; rows unpadded, their 16-byte pieces stored XOR-permuted so that 16
// lanes reading 16 rows at one logical piece meet 64 different banks:
//   K': row r (128 B) holds key swap23(r) of the sub-tile, its piece c (of 8) at place c ^ ((r / 2) % 8);
//   V'^T: row e (64 B) holds V'^T[e][32 keys], its piece c (of 4) at place c ^ ((e / 4) % 4).
// Rows with bits 2 and 3 of the key index swapped give a lane 8 consecutive keys per 16-key contraction step.
struct __align__(16) Tile {
    unsigned char b[KS * D * 2];
};

__device__ __forceinline__ int swap23(int m) { return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1); }

struct State {
    floatx16 acc[2][2];     // O^T [feature tile][query tile]: feature 32 dt + 8 (x / 4) + 4 h + x % 4, query 32 nt + n
    float mref[2], l[2];    // reference (log2 units), sum of exp2(s c2 - mref) over this lane's keys
    bool seen[2];           // the query has met a visible key, i.e. mref is set
    int all_seen[2];        // every query of the tile has (the same in all lanes)
};

// Row maximum of this sub-tile's scores of query tile nt; the reference moves up to it and O, l follow (first contact: it is set).
__device__ __forceinline__ void move_reference(State &st, int nt, const floatx16 &s, float c2)
{
    float rmax = -INFINITY;
#pragma unroll
    for (int x = 0; x < 16; ++x) rmax = fmaxf(rmax, s[x]);
    rmax = fmaxf(rmax, __shfl_xor(rmax, 32, 64));
    const bool was = st.seen[nt], now = was || rmax != -INFINITY;
    const float mnew = now ? (was ? fmaxf(rmax * c2, st.mref[nt]) : rmax * c2) : 0.0f;
    const float alpha = was ? __builtin_amdgcn_exp2f(st.mref[nt] - mnew) : 1.0f;
    st.mref[nt] = mnew;
    st.seen[nt] = now;
    st.all_seen[nt] = __builtin_amdgcn_readfirstlane(__all(now));
    if (__any(alpha != 1.0f)) {
        st.l[nt] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int x = 0; x < 16; ++x) st.acc[dt][nt][x] *= alpha;
    }
}

// Probabilities p = exp2(s c2 - mref) of one query tile as three bf16 terms, largest first.
struct Split {
    bf16x8 t[3][2];                                        // [term][16 keys]
};

// Score pairs of a query tile on their way to terms: the upper halves of two numbers are a pair of terms, and what is left of a
// number is an exact difference of 16, then of 8 bits.  Masks, differences and byte moves run under matrix instructions; the
// bf16 dot product that would form a difference in one instruction does not: two beside a matrix instruction make 54 clocks
// of its 32, four masks or differences 34, eight of them 44.
struct Softmax {
    uint32_t upper;                                        // 0xffff0000, in a scalar register
    floatx2 p, r;
    float even, odd;                                       // sums of the fp32 probabilities

    __device__ __forceinline__ void begin()
    {
        upper = 0xffff0000u;
        asm volatile("" : "+s"(upper));
        even = odd = 0.0f;
    }
    template <int Y>
    __device__ __forceinline__ void exponentials(const floatx16 &s, float c2, float mref)
    {
        p = {__builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * Y], c2, -mref)),
             __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * Y + 1], c2, -mref))};
    }
    template <int Y, int TERM>
    __device__ __forceinline__ void put(Split &pf, floatx2 v) const
    {
        const float lo = v[0], hi = v[1];
        uint32_t pair = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo), 0x07060302u);
        asm volatile("" : "+v"(pair));                     // formed here, not where it is used
        const bf16x2 t = __builtin_bit_cast(bf16x2, pair);
        pf.t[TERM][Y >> 2][2 * (Y & 3)] = t[0];
        pf.t[TERM][Y >> 2][2 * (Y & 3) + 1] = t[1];
    }
    __device__ __forceinline__ float rest(float v) const
    {
        return v - __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) & upper);
    }
    template <int Y>
    __device__ __forceinline__ void first_term(Split &pf)
    {
        even += p[0];
        odd += p[1];
        put<Y, 0>(pf, p);
        r = floatx2{rest(p[0]), rest(p[1])};
    }
    template <int Y>
    __device__ __forceinline__ void other_terms(Split &pf) const
    {
        put<Y, 1>(pf, r);
        put<Y, 2>(pf, floatx2{rest(r[0]), rest(r[1])});
    }
};

// f(0), f(1), .. with compile-time arguments
template <typename F, int... M>
__device__ __forceinline__ void unrolled(F &f, std::integer_sequence<int, M...>)
{
    (f(std::integral_constant<int, M>{}), ...);
}

__device__ __forceinline__ float probabilities(const floatx16 &s, float c2, float mref, Split &pf)
{
    Softmax sm;
    sm.begin();
    auto pair = [&](auto yc) __attribute__((always_inline)) {
        constexpr int y = decltype(yc)::value;
        sm.exponentials<y>(s, c2, mref);
        sm.first_term<y>(pf);
        sm.other_terms<y>(pf);
        __builtin_amdgcn_sched_barrier(0);                 // pair by pair: in few registers
    };
    unrolled(pair, std::make_integer_sequence<int, 8>{});
    return sm.even + sm.odd;
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
    __shared__ Tile ring_k0[WAVES], ring_k1[WAVES], ring_v0[WAVES], ring_v1[WAVES];    // separate variables: the compiler can tell them apart
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
    Tile &k0 = ring_k0[wave], &k1 = ring_k1[wave], &v0 = ring_v0[wave], &v1 = ring_v1[wave];
    __shared__ __align__(16) int32_t ring_p[WAVES][2][64];    // positions of the keys of a pair of sub-tiles
    const uint32_t own = wave * (uint32_t)sizeof(Tile);    // in the lanes' offsets of fragment reads
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
        st.all_seen[nt] = 0;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int x = 0; x < 16; ++x) st.acc[dt][nt][x] = 0.0f;
    }

    // Loads: a sub-tile of K' or Vt is 4 instructions of 1 KiB.  Reads past the end of K' give zeros (such slots are masked) and
    // start at the end at the latest (scalar_offset); Vt is zero-filled to whole blocks; a pair's positions start with one of the n keys.
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
    for (int c = 0; c < 4; ++c) kfr[c] = own + (uint32_t)(ln * (D * 2) + (((2 * c + lh) ^ ((ln >> 1) & 7)) << 4));
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) vfr[k2] = own + (uint32_t)(ln * (KS * 2) + (((2 * k2 + lh) ^ ((ln >> 2) & 3)) << 4));
    // load C of the K' rows or the Vt group of the 32 slots from slot0 on
    auto load_k = [&](auto cc, Tile &to, int slot0) __attribute__((always_inline)) {
        constexpr int c = decltype(cc)::value;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lptr_t)(to.b + c * 1024), 16, koff[c & 1],
                                                 scalar_offset((slot0 + (c >> 1) * 16) * (D * 2), g.n * (D * 2)), 0, 0);
    };
    auto load_v = [&](auto cc, Tile &to, int slot0) __attribute__((always_inline)) {
        constexpr int c = decltype(cc)::value;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lptr_t)(to.b + c * 1024), 16, voff, slot0 * (D * 2) + c * 1024, 0, 0);
    };
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(w.kidx), 0, g.n * 4, kRawDword);
    auto load_positions = [&](int which, int slot0) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rp, (lptr_t)(ring_p[wave][which]), 4, lane * 4, slot0 * 4, 0, 0);
    };
    auto load_tile = [&](auto &load, Tile &to, int slot0) __attribute__((always_inline)) {
        auto one = [&](auto cc) __attribute__((always_inline)) { load(cc, to, slot0); };
        unrolled(one, std::make_integer_sequence<int, 4>{});
    };

    // the list as pairs of sub-tiles, this wave's are every WAVES-th: the first slot of its next admitted 64 keys, -1 past
    // the end
    const int halves_log2 = g.block >> 7, total = w.cnt << halves_log2;    // 64-key pieces of a block: one or two
    int u_next = wave;
    auto next_slot = [&]() __attribute__((always_inline)) -> int {
        while (u_next < total) {
            const int j = __builtin_amdgcn_readfirstlane(w.cols[u_next >> halves_log2]);
            const int part = u_next & halves_log2;
            u_next += WAVES;
            const int first = listed_slot(j, part, 64, g.block, w.ni, g.n);
            if (first >= 0) return first;
        }
        return -1;
    };

    auto scores = [&](const bf16x8 (&kf)[4], int nt, floatx16 &s) __attribute__((always_inline)) {
        s = floatx16{0};
#pragma unroll
        for (int x = 0; x < 4; ++x) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[x], qf[nt][x], s, 0, 0, 0);
    };
    // the lane's id formed anew, for the rare paths: what they alone need of it would take registers from the loop
    auto fresh_lane = [&]() __attribute__((always_inline)) {
        uint32_t ones = ~0u;
        asm volatile("" : "+s"(ones));
        return (int)__builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0));
    };
    auto load_kf = [&](bf16x8 (&kf)[4], int slot0) __attribute__((always_inline)) {           // from memory
        const int id = fresh_lane(), at = swap23(id & 31) * (D * 2) + (id >> 5) * 16;
        const int from = scalar_offset(slot0 * (D * 2), g.n * (D * 2));
#pragma unroll
        for (int x = 0; x < 4; ++x)
            kf[x] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rk, at + 32 * x, from, 0));
    };
    auto far_scores = [&](int nt, int slot0, floatx16 &s) __attribute__((always_inline)) {
        bf16x8 kf[4];
        load_kf(kf, slot0);
        scores(kf, nt, s);
    };
    // product I of the 12 that add a sub-tile to O^T of query tile NT: the terms of its first 16 keys, then of the others, so
    // that the registers of the former are free half way
    auto add_value = [&](auto ic, auto nc, const bf16x8 (&vf)[2][2], const Split &pf) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, nt = decltype(nc)::value, k2 = i / 6, dt = i / 3 % 2, term = i % 3;
        st.acc[dt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[dt][k2], pf.t[term][k2], st.acc[dt][nt], 0, 0, 0);
    };
    auto add_values = [&](auto nc, const bf16x8 (&vf)[2][2], const Split &pf) __attribute__((always_inline)) {
        auto one = [&](auto ic) __attribute__((always_inline)) { add_value(ic, nc, vf, pf); };
        unrolled(one, std::make_integer_sequence<int, 12>{});
    };
    // the token-level mask on the scores of query tile nt; s[x]: key 16 (x / 8) + 8 h + x % 8, query 32 nt + n; eight(k8):
    // positions of the eight keys from k8 on, of which `room` of the sub-tile's exist
    auto hide = [&](floatx16 &s, int nt, int room, auto eight) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k8 = 16 * u + 8 * (fresh_lane() >> 5);
            int kp[8];
            eight(k8, kp);
            if (room < KS) {
#pragma unroll
                for (int x = 0; x < 8; ++x)
                    if (k8 + x >= room) kp[x] = 0x7fffffff;
            }
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (kp[x] > qpos[nt]) s[8 * u + x] = -INFINITY;
        }
    };
    // the same with positions that have landed in LDS.  Written in assembly: the compiler would wait for the next pair's as well.
    auto hide_near = [&](floatx16 &s, int nt, int slot0, int which) __attribute__((always_inline)) {
        const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int32_t *)ring_p[wave][which] + (slot0 & 32) * 4;
        hide(s, nt, w.n - slot0, [&](int k8, int (&kp)[8]) __attribute__((always_inline)) {
            int4u a, c;
            asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:16\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(a), "=&v"(c) : "v"(at + 4 * k8) : "memory");
#pragma unroll
            for (int x = 0; x < 4; ++x) { kp[x] = a[x]; kp[4 + x] = c[x]; }
        });
    };

    // Half a sub-tile: the softmax of query tile NT runs under 16 products that do not wait for it, four that form the
    // scores of the other query tile (s_next) and twelve that add the other tile's last probabilities to its O^T.
    // under(m): loads and fragment reads that go out behind product m.
    auto half = [&](auto nc, floatx16 &s, floatx16 &s_next, const bf16x8 (&kf)[4], const bf16x8 (&vf)[2][2], const Split &pf_other,
                    Split &pf, int slot0, int which, bool masked, auto under) __attribute__((always_inline)) {
        constexpr int nt = decltype(nc)::value;
        const int moves = st.all_seen[nt] ^ 1;
        if (__builtin_expect((moves | (int)masked) != 0, 0)) {
            asm volatile("" ::: "memory");                 // stays out of the straight-line code, as the block below
            if (masked) hide_near(s, nt, slot0, which);
            if (moves) move_reference(st, nt, s, c2);      // at least the row maximum: no sum below can be large
        }
        Softmax sm;
        sm.begin();
        __builtin_amdgcn_sched_barrier(0);
        auto slot = [&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value, y = m / 2;
            if constexpr (m == 0) s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], qf[1 - nt][0], floatx16{0}, 0, 0, 0);
            else if constexpr (m < 4) s_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[m], qf[1 - nt][m], s_next, 0, 0, 0);
            else add_value(std::integral_constant<int, m - 4>{}, std::integral_constant<int, 1 - nt>{}, vf, pf_other);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (m % 2 == 0) {
                if constexpr (y > 0) sm.other_terms<y - 1>(pf);
                sm.exponentials<y>(s, c2, st.mref[nt]);
            } else {
                sm.first_term<y>(pf);
            }
            under(mc);
            __builtin_amdgcn_sched_barrier(0);
        };
        unrolled(slot, std::make_integer_sequence<int, 16>{});
        sm.other_terms<7>(pf);
        float rsum = sm.even + sm.odd;
        if (__builtin_expect((moves == 0) & __any(!(rsum <= kBigRowSum)), 0)) {
            asm volatile("" ::: "memory");
            floatx16 again;                                // formed again from K' in memory rather than kept: 16 registers fewer
            far_scores(nt, slot0, again);
            if (masked) hide_near(again, nt, slot0, which);
            move_reference(st, nt, again, c2);
            rsum = probabilities(again, c2, st.mref[nt], pf);
        }
        st.l[nt] += rsum;
    };
    using N0 = std::integral_constant<int, 0>;
    using N1 = std::integral_constant<int, 1>;
    auto read_k = [&](auto xc, const Tile *from, bf16x8 (&kf)[4]) __attribute__((always_inline)) {
        constexpr int x = decltype(xc)::value;
        kf[x] = *reinterpret_cast<const bf16x8 *>(from->b + kfr[x]);
    };

    // Sub-tile t.  On entry: s0 its scores for query tile 0, kf its K' fragments, pf1 and vf the probabilities of query tile 1
    // and the V'^T fragments of sub-tile t - 1.  kt: place of K' of t + 1, which that of t + 3 replaces; vt: place of V'^T of t,
    // which that of t + 2 replaces.  A load has at least 1 1/4 sub-tiles to arrive.
    floatx16 s0, s1;
    bf16x8 kf[4], vf[2][2];
    Split pf0, pf1;
    // partc: which of its pair; which: place of the pair's key positions.  The next pair's are one load in its first half.
    auto subtile = [&](auto partc, Tile *kring, Tile *vring, int which, int slot0, bool masked, int refill_k, int refill_v) __attribute__((always_inline)) {
        Tile &kt = kring[wave], &vt = vring[wave];
        constexpr int part = decltype(partc)::value;
        // K' of t + 1 and V'^T of t have landed (and the pair's positions), the loads of the last sub-tile may still be in flight
        __builtin_amdgcn_s_waitcnt(part == 0 ? 0x0F78 : 0x0F79);    // vmcnt(8), vmcnt(9), gfx9 encoding
        __builtin_amdgcn_sched_barrier(0);
        half(N0{}, s0, s1, kf, vf, pf1, pf0, slot0, which, masked, [&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value;
            if constexpr (m >= 4 && m < 8) read_k(std::integral_constant<int, m - 4>{}, kring, kf);
            if constexpr (m == 11) {
                __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0): K' of t + 1 is in registers and may be replaced
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (m >= 12) load_k(std::integral_constant<int, m - 12>{}, kt, refill_k);
        });
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2) vf[dt][k2] = *reinterpret_cast<const bf16x8 *>(vring->b + vfr[k2] + dt * 2048);
        half(N1{}, s1, s0, kf, vf, pf0, pf1, slot0, which, masked, [&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value;
            if constexpr (m == 4) {
                __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0): the same for V'^T of t
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (m >= 5 && m < 9) load_v(std::integral_constant<int, m - 5>{}, vt, refill_v);
            if constexpr (m == 9 && part == 0) load_positions(which ^ 1, refill_v);
        });
    };

    int p0 = next_slot();
    if (p0 >= 0) {
        load_tile(load_k, k0, p0);
        load_positions(0, p0);
        load_tile(load_v, v0, p0);
        load_tile(load_k, k1, p0 + KS);
        load_tile(load_v, v1, p0 + KS);
        int p1 = next_slot();
        __builtin_amdgcn_s_waitcnt(0x0F7C);                // vmcnt(12), of 17: the first K' sub-tile
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < 4; ++x) kf[x] = *reinterpret_cast<const bf16x8 *>(ring_k0->b + kfr[x]);
        __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        load_tile(load_k, k0, p1 >= 0 ? p1 : p0);
        scores(kf, 0, s0);
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {                   // nothing to add yet
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) vf[dt][k2] = bf16x8{0};
#pragma unroll
            for (int term = 0; term < 3; ++term) pf1.t[term][k2] = bf16x8{0};
        }
        for (int which = 0; p0 >= 0; which ^= 1) {
            const int p2 = p1 >= 0 ? next_slot() : -1;
            const int a1 = p1 >= 0 ? p1 : p0, a2 = p2 >= 0 ? p2 : a1;    // past the end: a pair again (unused)
            const bool masked = p0 >= w.jmask * g.block;
            subtile(N0{}, ring_k1, ring_v0, which, p0, masked, a1 + KS, a1);
            subtile(N1{}, ring_k0, ring_v1, which, p0 + KS, masked, a2, a1 + KS);
            p0 = p1;
            p1 = p2;
        }
        add_values(N1{}, vf, pf1);
        __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the loads issued past the end have landed too
    }

    // A value that is not finite does not come through these products: 0 * inf of a hidden key is NaN, and so is
    // the sum over the terms of a visible one whenever a term is zero.  A wave that finds NaN in its O^T forms it again,
    // relative to the references it has ended with: such values leave the products and are added one key at a time, with the
    // undivided probability, for the queries that see the key.  Nothing is prefetched here; with one infinite value that every
    // query of the call sees, 16 / 4 heads x 12301 tokens take 1.24 ms instead of 0.61.
    bool odd = false;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int x = 0; x < 16; ++x) odd = odd || st.acc[dt][nt][x] != st.acc[dt][nt][x];
    if (__any(odd)) {
        // [key % 16][query], -1: not seen; the first 16 keys of the sub-tile, the others
        float *weight[2] = {reinterpret_cast<float *>(&k0), reinterpret_cast<float *>(&k1)};
        static_assert(sizeof(Tile) == 16 * kQ * sizeof(float), "the probabilities of half a sub-tile");
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) st.acc[dt][nt] = floatx16{0};
        u_next = wave;
        int slot0 = next_slot();
        for (int part = 0; slot0 >= 0; ) {
            bf16x8 kf[4], vf[2][2];
            load_kf(kf, slot0);
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
                    vf[dt][k2] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rv, (32 * dt + ln) * (KS * 2) + (2 * k2 + lh) * 16, slot0 * (D * 2), 0));
            floatx16 s[2];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                scores(kf, nt, s[nt]);
                if (slot0 >= w.jmask * g.block)
                    hide(s[nt], nt, w.n - slot0, [&](int k8, int (&kp)[8]) __attribute__((always_inline)) {
#pragma unroll
                        for (int x = 0; x < 8; ++x) kp[x] = w.kidx[min(slot0 + k8 + x, w.n - 1)];
                    });
#pragma unroll
                for (int x = 0; x < 16; ++x)
                    weight[x >> 3][(8 * lh + (x & 7)) * kQ + 32 * nt + ln] =
                        s[nt][x] == -INFINITY ? -1.0f : __builtin_amdgcn_exp2f(__builtin_fmaf(s[nt][x], c2, -st.mref[nt]));
            }
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
            probabilities(s[0], c2, st.mref[0], pf0);
            probabilities(s[1], c2, st.mref[1], pf1);
            add_values(N0{}, vf, pf0);
            add_values(N1{}, vf, pf1);
            for (; keys; keys &= keys - 1) {
                const int key = __builtin_ctz(keys);
                const float *wk = (key < 16 ? weight[0] : weight[1]) + (key & 15) * kQ;
                const float p[2] = {wk[ln], wk[32 + ln]};
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
        static_assert(WAVES == 4 && sizeof(Tile) == D / WAVES * kQ * sizeof(float), "a quarter of the features of 64 queries");
        float *part[4] = {reinterpret_cast<float *>(&k0), reinterpret_cast<float *>(&k1), reinterpret_cast<float *>(&v0),
                          reinterpret_cast<float *>(&v1)};
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
                    part[2 * dt + (x >> 3)][(8 * (x >> 2 & 1) + 4 * lh + (x & 3)) * kQ + 32 * nt + ln] = st.acc[dt][nt][x];
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
        const Tile *ring = wave == 0 ? ring_k0 : wave == 1 ? ring_k1 : wave == 2 ? ring_v0 : ring_v1;
        bf16x8 out[F / 8];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            float o = 0.0f;
#pragma unroll
            for (int v = 0; v < WAVES; ++v)
                o += reinterpret_cast<const float *>(&ring[v])[f * kQ + q] * scale[v];
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
    // there are two tiles per slot.  Measured, four waves / one, us: every admitted block listed, 768 tiles 84 / 188, 1536
    // 300 / 402, 2048 272 / 325, 3088 590 / 634, 4096 529 / 512 and 1019 / 1001, 8192 3953 / 3934; a tenth of the
    // blocks, 1536 tiles 52 / 64, 2048 55 / 56, 3088 95 / 93, 4096 102 / 81 and 146 / 136, 16384 1830 / 1715.
    if (units * rows < 2 * 2048)
        return launch(d64::attn_d64_kernel<4>, grid, dim3(256), 0, s, (const bf16_t *)Qp, (const bf16_t *)Kp,
                      (const bf16_t *)Vt, qidx, kidx, row_cnt, col_idx, (bf16_t *)Op, lse, g, cohort);
    return launch(d64::attn_d64_kernel<1>, grid, dim3(64), 0, s, (const bf16_t *)Qp, (const bf16_t *)Kp,
                  (const bf16_t *)Vt, qidx, kidx, row_cnt, col_idx, (bf16_t *)Op, lse, g, cohort);
}

}  // namespace pbs

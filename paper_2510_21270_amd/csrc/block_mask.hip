// pbs_block_mask: Algorithm 2 (MeanPooling block selection) on the permuted (Q', K') plus the forced blocks.
//
// Everything that decides the discrete result runs in IEEE fp64 in the order of the definition, so the mask does not
// depend on how a machine rounds lower precision (the logits use fused multiply-adds: the same bits as separate
// operations whenever the products of two block means are exact, which 15 + 15 significant bits plus the exponent
// spread inside a block's column usually are):
//   1. pool_kernel     block means of K' (HBM-bound), stored d-major ([head][e][T]) so that the next kernel reads
//                      them coalesced.  A sum of up to 128 bf16 values is exact in fp64 in any order (8 significant
//                      bits each; the exponents of one column would have to spread over more than 38 binades to lose
//                      a bit), so bf16 inputs are summed in whatever order loads best.  fp32 values have 24 significant
//                      bits and no such slack: they are added one row after the other, in ascending order, which
//                      is the order of the plain definition.
//   2. select_kernel   block means of its own Q' blocks, then logits of up to four query heads of one group against
//                      the allowed columns, softmax, the mass threshold by bisection (one wave per row), forced
//                      blocks, then bit-mask words by wave ballot and the ascending column list by prefix popcount.
#include <type_traits>
#include <utility>

#include "pbs_host.h"

namespace pbs {

// Sum of `rows` values `stride` apart, added in ascending order (fp32 storage); sixteen loads are in flight ahead of their
// additions, so that a block costs a few memory latencies and not one per row.
template <typename E>
__device__ __forceinline__ double ordered_column_sum(const E *x, int rows, int stride)
{
    constexpr int U = 16;
    double s = 0.0;
    int r0 = 0;
    for (; r0 + U <= rows; r0 += U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ElemTraits<E>::to_float(x[(r0 + u) * stride]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) s += (double)v[u];
    }
    for (; r0 < rows; ++r0) s += (double)ElemTraits<E>::to_float(x[r0 * stride]);
    return s;
}

// ---------------------------------------------------------------------------------------------
// grid = (T, heads); E = input element type.  TRANSPOSED: write out[head][e][Ts] (row stride Ts >= T) instead of
// out[head][i][e].
// 256 threads: thread (cg = tid % cpr, rg = tid / cpr) sums its 16-byte column group over rows rg, rg+RG, ...
// ---------------------------------------------------------------------------------------------
template <typename E, bool TRANSPOSED>
__global__ __launch_bounds__(256) void pool_kernel(const E *__restrict__ X, double *__restrict__ out, int n, int d,
                                                   int block, int T, int Ts)
{
    constexpr int VEC = 16 / sizeof(E);
    typedef E vec_t __attribute__((ext_vector_type(VEC)));
    __shared__ double red[256 * VEC];                       // [rg][cg][VEC] flattened as tid * VEC
    const int i = blockIdx.x;
    const size_t head = blockIdx.y;
    const int cpr = d / VEC;                                // 8..32
    const int RG = 256 / cpr;
    const int cg = threadIdx.x % cpr, rg = threadIdx.x / cpr;
    const int lo = i * block, hi = min(n, lo + block);
    if constexpr (sizeof(E) == 4) {
        // fp32 storage: thread e owns column e and adds its rows in ascending order
        if ((int)threadIdx.x < d) {
            const int e = threadIdx.x;
            const double mean = ordered_column_sum(X + (head * n + lo) * (size_t)d + e, hi - lo, d) / (double)(hi - lo);
            if (TRANSPOSED) out[(head * d + e) * (size_t)Ts + i] = mean;
            else out[(head * T + i) * (size_t)d + e] = mean;
        }
        return;
    }
    double acc[VEC];
#pragma unroll
    for (int u = 0; u < VEC; ++u) acc[u] = 0.0;
    // four independent 16-byte loads in flight per thread (bf16: the sums are exact in fp64 whatever the order)
    constexpr int U = 4;
    for (int row = lo + rg; row < hi; row += U * RG) {
        vec_t v[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            v[q] = vec_t{};
            if (row + q * RG < hi)
                v[q] = *reinterpret_cast<const vec_t *>(X + (head * n + row + q * RG) * (size_t)d + cg * VEC);
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (row + q * RG < hi)
#pragma unroll
                for (int u = 0; u < VEC; ++u) acc[u] += (double)ElemTraits<E>::to_float(v[q][u]);
    }
#pragma unroll
    for (int u = 0; u < VEC; ++u) red[threadIdx.x * VEC + u] = acc[u];
    __syncthreads();
    if ((int)threadIdx.x < d) {
        const int e = threadIdx.x, c = e / VEC, u = e % VEC;
        double s = 0.0;
        for (int q = 0; q < RG; ++q) s += red[(q * cpr + c) * VEC + u];
        const double mean = s / (double)(hi - lo);
        if (TRANSPOSED) out[(head * d + e) * (size_t)Ts + i] = mean;
        else out[(head * T + i) * (size_t)d + e] = mean;
    }
}

// ---------------------------------------------------------------------------------------------
// Selection.  One workgroup per (kv head, chunk of RB query heads of its group, QB query blocks): the RB * QB rows share
// the allowed columns and the pooled keys.  The logits run on the fp64 matrix instruction v_mfma_f64_4x4x4 (four
// independent 4 x 4 x 4 products: here 4 rows x 16 columns x 4 features), whose accumulator takes the four products in
// ascending order with one rounding each, i.e. exactly the chain of fused multiply-adds over ascending features that
// defines a logit.  It does 12.8 multiply-adds per clock where v_fma_f64 does 8, and a pooled query comes out of LDS
// once per 64 of them instead of once per 2.  A wave takes 32 columns at a time.  After the logits, wave w owns row w
// and finishes it alone (no workgroup barriers): softmax, then the smallest probability v* that is still kept, found by
// bisection instead of a sort, with the row in registers.
// Bound: vector issue (pooling Q': a conversion and an fp64 addition per value, 3 us of a wave's time per block; the
// bisection about as much) and the phases' latencies, which only other waves of the SIMD hide.  Measured, same masks bit
// for bit, against logits on v_fma_f64 with every multiply-add's query operand read from LDS and two workgroups to a
// compute unit: 28 / 4 heads x 65536 179 -> 134 us, 32 / 8 heads x 2048 25.5 -> 15.9 us, x 8147 31.9 -> 22.4 us,
// x 131072 443 -> 386 us.
//
// The kept set of Algorithm 2 is the shortest prefix of the order (probability descending, column ascending)
// whose mass reaches tau.  With M(v) = sum of the probabilities >= v, v* is the largest v with M(v) >= tau:
// every probability above v* is kept, and of the columns that tie at v* the first m by column index, m being
// the number of additions of v* to M(> v*) that reach tau.  The bisection runs over the bit patterns of the
// non-negative doubles between the smallest and the largest probability and stops as soon as a single
// element, or a single bit pattern, is left in the bracket.
// ---------------------------------------------------------------------------------------------
struct MassCount {
    double mass;
    int cnt;
};

constexpr int kPanel = 512;                                // columns whose logits go through LDS at a time

template <int... I, typename F>
__device__ __forceinline__ void for_each_index(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// One row in registers, 64 columns per chunk, lane = column, up to NC chunks.  Columns past the row's own count are padded
// by the caller.
template <int NC>
struct RowProbs {
    double x[NC];
    int chunks;
    __device__ __forceinline__ explicit RowProbs(int ni) : chunks((ni + 63) >> 6) {}
    // the chunks of panel p (kPanel columns, compile-time p) from the panel's row in LDS
    template <int P>
    __device__ __forceinline__ void take(const double *pr, int lane)
    {
#pragma unroll
        for (int c = 0; c < kPanel / 64; ++c)
            if (P * (kPanel / 64) + c < chunks) x[P * (kPanel / 64) + c] = pr[64 * c + lane];
    }
    template <typename F>
    __device__ __forceinline__ void each(F f)              // f(chunk, value), in ascending order
    {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (c < chunks) f(c, x[c]);
    }
};

// mass and number of the row's probabilities >= v (padding is negative)
template <int NC>
__device__ __forceinline__ MassCount mass_at_least(RowProbs<NC> &row, double v)
{
    double acc = 0.0;
    int cnt = 0;
    row.each([&](int, double &x) {
        const bool ge = x >= v;
        acc += ge ? x : 0.0;
        cnt += __popcll(__ballot(ge));
    });
    return {wave_sum_dpp(acc), cnt};
}

// QB query blocks (i0 = QB * blockIdx.x and the next ones) of RB query heads per workgroup: RT = RB * QB rows, one wave
// each.  Neighbouring query blocks see the same pooled keys (the later ones a few more columns), so that pooled keys once
// loaded feed QB times the multiply-adds and the logits need that much fewer round trips to L2.
// Query blocks are taken from the last one down: the long rows start first, the short ones fill the tail.
// The registers of a row of at most 512 columns (NC = 8) leave room for eight waves per SIMD, of 1024 for six, of 2048 for
// four, of 4096 for two; the more there are, the more they hide of each other's phases.
// FEW (at most 512 columns, bf16 blocks of 128 x 128): no more workgroups than compute units, so that no other wave hides a phase's
// latencies; with registers for two waves per SIMD a whole query block and twice the pooled keys are on their way at a time.
constexpr int select_waves(int nc, bool few) { return few ? 2 : nc == 8 ? 8 : nc == 16 ? 6 : nc == 32 ? 4 : 2; }

template <int RB, int QB, int NC, bool FEW, typename E>
__global__ __launch_bounds__(64 * RB * QB) __attribute__((amdgpu_waves_per_eu(select_waves(NC, FEW), select_waves(NC, FEW))))
void select_kernel(const E *__restrict__ Qp,           // [bhq][n][d]
                   const double *__restrict__ KbarT,   // [bhkv][d][Ts]
                   uint64_t *__restrict__ mask_bits, int32_t *__restrict__ row_cnt, int32_t *__restrict__ col_idx,
                   Geo g, int chunks, int Tpad, int Ts)
{
    constexpr int RT = RB * QB;                                      // rows (= waves) of the workgroup
    constexpr int NG = (RT + 3) / 4;                                 // groups of four rows
    constexpr int FS = FEW ? 8 : 4;                                  // steps of four features per register buffer
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double *prob = reinterpret_cast<double *>(smem_raw);             // [RT][kPanel, or Tpad if less]
    __shared__ __align__(16) double qs[128][RT];                     // block means of the RT query rows, feature-major

    const int i0 = (g.T - 1) / QB * QB - QB * (int)blockIdx.x;       // first query block of this workgroup
    const int bhk = blockIdx.y / chunks, chunk = blockIdx.y % chunks;
    const int b = bhk / g.h_kv, hk = bhk % g.h_kv;
    const int rows = min(RB, g.r - chunk * RB);                      // query heads handled here
    const int bhq0 = b * g.h_q + hk * g.r + chunk * RB;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wq = w / RB, wh = w % RB;                              // this wave's query block (i0 + wq) and head
    const int i = i0 + wq;
    const bool active = i < g.T && wh < rows;
    const int nblk = min(QB, g.T - i0);                              // query blocks present
    const int ni_all = allowed_cols(i0 + nblk - 1, g);               // the last one sees the most columns

    // Block mean of query block i of head wh, by wave w (sums of storage values in fp64; 16-byte column groups,
    // U loads in flight per lane, then the row groups of the wave are added up).  Pooling Q' here instead of in
    // a kernel of its own lets the 1 GiB read of Q' overlap with the arithmetic of other workgroups.
    // fp32 storage: every lane owns columns and adds their rows in ascending order (see the note at the top).
    if constexpr (sizeof(E) == 4) {
        const int lo = i * g.block, hi = min(g.n, lo + g.block);
        if (active) {
            const E *X = Qp + (size_t)(bhq0 + wh) * g.n * g.d;
            for (int e = lane; e < g.d; e += 64) {
                qs[e][w] = ordered_column_sum(X + (size_t)lo * g.d + e, hi - lo, g.d) / (double)(hi - lo);
            }
        }
    } else {
        constexpr int VEC = 16 / sizeof(E);
        typedef E vec_t __attribute__((ext_vector_type(VEC)));
        const int cpr = g.d / VEC;                                   // 8 .. 32 column groups
        const int RG = 64 / cpr;                                     // row groups of a wave
        const int cg = lane % cpr, rg = lane / cpr;
        const int lo = i * g.block, hi = min(g.n, lo + g.block);
        double acc[VEC];
#pragma unroll
        for (int u = 0; u < VEC; ++u) acc[u] = 0.0;
        if (active) {
            // A register is requested again as soon as it is added up, so that the additions (a conversion and an fp64
            // addition per value) run under the loads of the others.  Buffer loads: rows past the block lie past
            // the descriptor's end and read as zeros, without a branch per load.  The way into the block is part of the lane's offset:
            // a scalar offset may not lie behind the descriptor's end (see scalar_offset).
            constexpr int U = FEW ? 32 : 4, kNonTemporal = 2;        // FEW: blocks of 32 pieces
            const int row_bytes = g.d * (int)sizeof(E);
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<E *>(Qp + ((size_t)(bhq0 + wh) * g.n + lo) * g.d), 0, (hi - lo) * row_bytes, 0x00020000);
            const int voff = lane * 16;                              // row rg, column group cg of a piece of 1 KiB = RG rows
            static_assert(VEC * sizeof(E) == 16, "one load of 16 bytes per lane");
            const int pieces = (g.block + RG - 1) / RG;
            vec_t v[U];
#pragma unroll
            for (int q = 0; q < U; ++q)
                v[q] = __builtin_bit_cast(vec_t, __builtin_amdgcn_raw_buffer_load_b128(r, voff + q * 1024, 0, kNonTemporal));
            __builtin_amdgcn_sched_barrier(0);
            auto add = [&](int q) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < VEC; ++u) acc[u] += (double)ElemTraits<E>::to_float(v[q][u]);
                __builtin_amdgcn_sched_barrier(0);
            };
            if constexpr (FEW) {
#pragma unroll
                for (int q = 0; q < U; ++q) add(q);
            } else {
                for (int q0 = 0; q0 < pieces; q0 += U)
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        add(q);
                        v[q] = __builtin_bit_cast(vec_t, __builtin_amdgcn_raw_buffer_load_b128(r, voff + (q0 + U + q) * 1024, 0, kNonTemporal));
                        __builtin_amdgcn_sched_barrier(0);
                    }
            }
        }
        for (int o = cpr; o < 64; o <<= 1)
#pragma unroll
            for (int u = 0; u < VEC; ++u) acc[u] += __shfl_xor(acc[u], o, 64);
        if (rg == 0 && active)
#pragma unroll
            for (int u = 0; u < VEC; ++u) qs[cg * VEC + u][w] = acc[u] / (double)(hi - lo);
    }
    __syncthreads();

    // logits: A operand: lane holds the mean of row lane % 4 (of its group), feature 4 step + lane / 16; B operand: column
    // lane % 16, same feature; accumulator: row lane / 16, column lane % 16.  Rows that are not there compute whatever
    // qs holds, columns past the row end the last one's; neither is stored.  Two register buffers of FS steps, filled
    // alternately: the loads of one are in flight while the other is multiplied (scheduling barriers keep the compiler
    // from moving a buffer's loads down to its use).
    const double *kt = KbarT + (size_t)bhk * g.d * Ts;
    auto logits = [&](int first, int end, int stride) {              // columns first .. end - 1 into prob rows of `stride`
      for (int c0 = first + 32 * w; c0 < end; c0 += 32 * RT) {
        const double *src[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) src[t] = kt + (size_t)(lane >> 4) * Ts + min(c0 + 16 * t + (lane & 15), Ts - 1);
        double acc[2][NG];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int y = 0; y < NG; ++y) acc[t][y] = 0.0;
        double ka[FS][2], kb[FS][2];
        const int steps = g.d / 4;                                   // 16 or 32
        auto fetch = [&](double (&k)[FS][2], int s0) {
            const int sc = s0 < steps ? s0 : 0;                      // past the end: the first features again (unused)
#pragma unroll
            for (int u = 0; u < FS; ++u)
#pragma unroll
                for (int t = 0; t < 2; ++t) k[u][t] = src[t][(size_t)(4 * (sc + u)) * Ts];
        };
        auto multiply = [&](const double (&k)[FS][2], int s0) {
#pragma unroll
            for (int u = 0; u < FS; ++u)
#pragma unroll
                for (int y = 0; y < NG; ++y) {
                    const double q = qs[4 * (s0 + u) + (lane >> 4)][min(4 * y + (lane & 3), RT - 1)];
#pragma unroll
                    for (int t = 0; t < 2; ++t) acc[t][y] = __builtin_amdgcn_mfma_f64_4x4x4f64(q, k[u][t], acc[t][y], 0, 0, 0);
                }
        };
        fetch(ka, 0);
        for (int s0 = 0; s0 < steps; s0 += 2 * FS) {
            fetch(kb, s0 + FS);
            __builtin_amdgcn_sched_barrier(0);
            multiply(ka, s0);
            __builtin_amdgcn_sched_barrier(0);
            fetch(ka, s0 + 2 * FS);
            __builtin_amdgcn_sched_barrier(0);
            multiply(kb, s0 + FS);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int y = 0; y < NG; ++y) {
            const int row = 4 * y + (lane >> 4);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int col = c0 + 16 * t + (lane & 15);
                if (row < RT && col < end) prob[row * stride + col - first] = __dmul_rn(acc[t][y], g.scale64);
            }
        }
      }
    };
    // A row gets into its wave's registers in panels of kPanel columns, so that LDS holds one panel of every row.
    const int ni = allowed_cols(active ? i : i0, g);
    RowProbs<NC> row(ni);
    const int stride = min(Tpad, kPanel);
    auto panel = [&](auto p_) {
        constexpr int P = decltype(p_)::value;
        if (P * kPanel >= ni_all) return;                            // uniform over the workgroup
        if (P > 0) __syncthreads();                                  // the panel before is in registers everywhere
        logits(P * kPanel, min(ni_all, (P + 1) * kPanel), stride);
        __syncthreads();
        row.template take<P>(prob + w * stride, lane);
    };
    for_each_index(std::make_integer_sequence<int, NC * 64 / kPanel>{}, panel);

    // from here on wave w works alone on its row
    if (!active) return;
    double lmax = -INFINITY;
    row.each([&](int c, double &x) {
        if (64 * c + lane >= ni) x = -INFINITY;
        lmax = fmax(lmax, x);
    });
    lmax = wave_max(lmax);
    double lsum = 0.0, emin = INFINITY;
    row.each([&](int c, double &x) {
        if (64 * c + lane < ni) {
            x = exp(x - lmax);
            lsum += x;
            emin = fmin(emin, x);
        }
    });
    lsum = wave_sum_dpp(lsum);
    emin = -wave_max(-emin);
    row.each([&](int c, double &x) { x = 64 * c + lane < ni ? x / lsum : -1.0; });      // padding never counts
    const double pmax = 1.0 / lsum, pmin = emin / lsum;      // exp(0) = 1 is the largest numerator

    // vstar: smallest kept probability; above: mass and count of the probabilities > vstar; ties: columns at vstar
    double vstar, above = 0.0;
    int n_above = 0, n_tie;
    int m;                                                   // ties kept, lowest columns first
    if (!(g.tau > 0.0)) {                                    // the first cumulative sum already reaches tau
        vstar = pmax;
        n_tie = mass_at_least(row, pmax).cnt;
        m = 1;
    } else {
        const MassCount all = mass_at_least(row, pmin);
        if (all.mass < g.tau) {                              // never reached: everything is kept
            vstar = -0.5;
            n_above = ni;
            n_tie = 0;
            m = 0;
        } else {
            // invariant: M(lo) >= tau > M(hi); lo and hi are bit patterns of non-negative doubles
            long long lo = __double_as_longlong(pmin), hi = __double_as_longlong(pmax) + 1;
            int cnt_lo = all.cnt;
            while (hi - lo > 1 && cnt_lo - n_above > 1) {
                const long long mid = lo + ((hi - lo) >> 1);
                const MassCount mc = mass_at_least(row, __longlong_as_double(mid));
                if (mc.mass >= g.tau) { lo = mid; cnt_lo = mc.cnt; }
                else { hi = mid; n_above = mc.cnt; above = mc.mass; }
            }
            n_tie = cnt_lo - n_above;
            if (hi - lo > 1) {                               // one element left in [lo, hi): it is vstar
                const double hid = __longlong_as_double(hi);
                double best = -1.0;
                row.each([&](int, double &x) { best = fmax(best, x < hid ? x : -1.0); });
                vstar = wave_max(best);
            } else {
                vstar = __longlong_as_double(lo);
            }
            double c = above;
            m = 0;
            do { c += vstar; ++m; } while (c < g.tau && m < n_tie);
        }
    }

    // forced blocks and output: mask words by ballot, ascending column list by prefix popcount
    const int seg = i / g.R;
    const int flo = seg < g.G ? seg * g.R : i;
    const int W = (g.T + 63) >> 6;
    const size_t orow = (size_t)(bhq0 + wh) * g.T + i;
    uint64_t *mrow = mask_bits + orow * W;
    int32_t *crow = col_idx + orow * g.T;
    const uint64_t below = (1ull << lane) - 1ull;
    int base = 0, ties_seen = 0;
    row.each([&](int c, double &x) {
        const int j = 64 * c + lane;
        const uint64_t tie_word = __ballot(x == vstar);
        const int tie_rank = ties_seen + __popcll(tie_word & below);
        ties_seen += __popcll(tie_word);
        bool on = false;
        if (j < ni)
            on = x > vstar || (x == vstar && tie_rank < m) || j >= flo ||
                 (j == 0 && (g.flags & PBS_FLAG_FORCE_FIRST_BLOCK));
        const uint64_t word = __ballot(on);
        if (lane == 0) mrow[c] = word;
        if (on) crow[base + __popcll(word & below)] = j;
        base += __popcll(word);
    });
    for (int c = row.chunks + lane; c < W; c += 64) mrow[c] = 0;     // columns past the allowed ones
    if (lane == 0) row_cnt[orow] = base;
}

template <int RB, int QB, int NC, bool FEW, typename E>
static pbs_status launch_select_nc(const E *Qp, const double *KbarT, uint64_t *mask_bits, int32_t *row_cnt,
                                   int32_t *col_idx, const Geo &g, hipStream_t s)
{
    const int chunks = (g.r + RB - 1) / RB;
    const int Tpad = (g.T + 63) & ~63;
    const size_t lds = (size_t)RB * QB * (Tpad > kPanel ? kPanel : Tpad) * sizeof(double);           // at most 32 KiB
    return launch((select_kernel<RB, QB, NC, FEW, E>), dim3((g.T + QB - 1) / QB, g.batch * g.h_kv * chunks), dim3(64 * RB * QB),
                  lds, s, Qp, KbarT, mask_bits, row_cnt, col_idx, g, chunks, Tpad, kbar_stride(g.T));
}

// Rows stay in registers up to the largest T: more than 1024 columns, heads x tokens, block 32: 8 / 2 x 65536 294 us,
// 8 / 4 x 131072 1.57 ms, block 128: 32 / 8 x 139264 499 us.  With the rows in LDS, one query block to a workgroup and
// the logits on v_fma_f64 that took 433 us, 2.73 ms and 513 us; with the rows in LDS and the logits on the matrix instruction
// 504 us, 3.82 ms and 562 us.
constexpr int kFewWgs = 256;
template <int RB, int QB, typename E>
static pbs_status launch_select_qb(const E *Qp, const double *KbarT, uint64_t *mask_bits, int32_t *row_cnt,
                                   int32_t *col_idx, const Geo &g, hipStream_t s)
{
    static_assert(kMaxT <= 4096, "columns of a row");
    // Whole query blocks on their way at a time, where no workgroup shares a compute unit.  Stage, four pieces / a block of 32, us: 32 / 8
    // heads x 1024 14.4 / 12.5, x 2048 16.1 / 14.1, x 8147 20.0 / 18.8, 4 / 2 x 8192 13.1 / 11.2, 28 / 4 x 4000 16.7 / 14.9; blocks of fewer
    // pieces, whose other loads are idle: 16 / 4 x 3000 x 64, block 64 11.5 / 12.9, 8 / 8 x 2000 x 64, block 128 8.9 / 9.4, 8 / 8 x 3000
    // x 128, block 64 10.4 / 10.5.  Where the line lies, the same two: workgroups of eight waves (three heads and more to a kv head), 256
    // of them 17.9 / 19.0 and 19.9 / 21.1, 288 29.8 / 26.0, 316 32.0 / 29.1, 512 39.0 / 33.5.  Those of four waves (one or two heads) share
    // a compute unit before its registers are full and gain somewhat further, 256 14.0 / 15.2, 320 18.6 / 19.0, 384 17.3 / 17.5, 512
    // 27.8 / 28.4, 768 47.7 / 38.7; the line is the same for them.
    if (sizeof(E) == 2 && g.T <= 512 && g.block * g.d == 128 * 128 &&
        (long long)ceil_div(g.T, QB) * g.batch * g.h_kv * ceil_div(g.r, RB) <= kFewWgs)
        return launch_select_nc<RB, QB, 8, sizeof(E) == 2>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
    if (g.T <= 512) return launch_select_nc<RB, QB, 8, false>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
    if (g.T <= 1024) return launch_select_nc<RB, QB, 16, false>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
    if (g.T <= 2048) return launch_select_nc<RB, QB, 32, false>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
    return launch_select_nc<RB, QB, 64, false>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
}

// A matrix instruction takes four rows: with one query head to a kv head two query blocks leave half of it empty, so four come to
// a workgroup except in the shortest rows; with two heads two blocks fill it and four only halve the reads of pooled keys, which
// pays once every compute unit has a workgroup.  Measured, four query blocks / two, us: one head, T = 64 12.1 / 10.9 and 11.2 / 11.0,
// 100 13.3 / 16.2, 128 11.1 / 12.9, 256 15.7 / 19.0, 1024 43 / 56, 8 / 8 heads x 131072 155 / 222, 32 / 32 x 131072 493 / 766; two heads, 32
// workgroups of four blocks 14.7 / 11.7, 89 22.5 / 20.3, 128 16.2 / 12.6, 200 19.1 / 19.7, 256 48 / 51, 512 54 / 66.  (Logits on
// v_fma_f64, two query blocks: 8 / 8 x 131072 175, 32 / 32 x 131072 581, two heads at 512 workgroups 62.)
template <typename E>
static pbs_status launch_select(const E *Qp, const double *KbarT, uint64_t *mask_bits, int32_t *row_cnt,
                                int32_t *col_idx, const Geo &g, hipStream_t s)
{
    if (g.r >= 3) return launch_select_qb<4, 2>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
    if (g.r == 2)
        return (long long)g.batch * g.h_kv * ceil_div(g.T, 4) >= 256 ? launch_select_qb<2, 4>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s)
                                                                     : launch_select_qb<2, 2>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
    return g.T > 64 ? launch_select_qb<1, 4>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s)
                    : launch_select_qb<1, 2>(Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
}

// Block means of K' into KbarT ([kv head][feature][kbar_stride(T)] fp64).
static pbs_status launch_pool_keys(const pbs_problem *p, const Geo &g, const void *Kp, double *KbarT, hipStream_t s)
{
    const int nk = g.batch * g.h_kv;
    if (p->dtype == PBS_BF16)
        return launch((pool_kernel<bf16_t, true>), dim3(g.T, nk), dim3(256), 0, s, (const bf16_t *)Kp, KbarT, g.n, g.d,
                      g.block, g.T, kbar_stride(g.T));
    return launch((pool_kernel<float, true>), dim3(g.T, nk), dim3(256), 0, s, (const float *)Kp, KbarT, g.n, g.d, g.block,
                  g.T, kbar_stride(g.T));
}

// Block means of the keys K, row-major ([kv head][block][feature] fp64): the centroids of the query permutation.
pbs_status launch_pool_keys_rowmajor(const pbs_problem *p, const Geo &g, const void *K, double *Kbar, hipStream_t s)
{
    const int nk = g.batch * g.h_kv;
    if (p->dtype == PBS_BF16)
        return launch((pool_kernel<bf16_t, false>), dim3(g.T, nk), dim3(256), 0, s, (const bf16_t *)K, Kbar, g.n, g.d,
                      g.block, g.T, g.T);
    return launch((pool_kernel<float, false>), dim3(g.T, nk), dim3(256), 0, s, (const float *)K, Kbar, g.n, g.d, g.block,
                  g.T, g.T);
}

size_t ws_block_mask(const pbs_problem *p)
{
    const Geo g = make_geo(p);
    // pooled K', fp64, feature-major, rows padded to kbar_stride(T) columns
    return align_up((size_t)g.batch * g.h_kv * kbar_stride(g.T) * g.d * sizeof(double), kWsAlign);
}

}  // namespace pbs

using namespace pbs;

extern "C" pbs_status pbs_block_mask(const pbs_problem *p, const void *Qp, const void *Kp, uint64_t *mask_bits,
                                     int32_t *row_cnt, int32_t *col_idx, void *ws, size_t ws_bytes, void *stream)
{
    pbs_status st = validate(p);
    if (st != PBS_OK) return st;
    if (!Qp || !Kp || !mask_bits || !row_cnt || !col_idx) return PBS_ERR_NULL;
    if (!aligned16(Qp) || !aligned16(Kp)) return PBS_ERR_SHAPE;
    if ((st = check_ws(p, PBS_STAGE_BLOCK_MASK, ws, ws_bytes)) != PBS_OK) return st;
    const Geo g = make_geo(p);
    hipStream_t s = (hipStream_t)stream;
    double *KbarT = reinterpret_cast<double *>(ws);
    if (!(p->flags & PBS_FLAG_KBAR_IN_WS) && (st = launch_pool_keys(p, g, Kp, KbarT, s)) != PBS_OK) return st;
    return p->dtype == PBS_BF16 ? launch_select((const bf16_t *)Qp, KbarT, mask_bits, row_cnt, col_idx, g, s)
                                : launch_select((const float *)Qp, KbarT, mask_bits, row_cnt, col_idx, g, s);
}

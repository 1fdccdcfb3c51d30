// Segmented permutation (Eq. 5 + Algorithm 1's first and last steps): per-segment stable descending
// argsort of the key scores, row gathers for K' and Q', the block-transposed gather for V', and the
// inverse row scatter for the output.  Pure integer/compare and copy work: bound by HBM.
#include "pbs_host.h"

namespace pbs {

// ---------------------------------------------------------------------------------------------
// One workgroup sorts one segment (or several short ones).  Key = (~orderable(score)) << 32 | position-in-segment, so an ascending 64-bit
// bitonic sort yields descending score with ties in ascending position.  -0.0 is folded onto +0.0 first so that the bit
// order agrees with the arithmetic order.
// The keys stay in registers, kSortPer = 4 neighbouring ones per lane (a padded segment of 4096 keys is 1024 threads):
// compare-exchange partners at strides 1 and 2 sit in the same lane, at strides 4 .. 128 in the same wave (lane ^ 1 ..
// 32, by DPP moves and the row swaps), and only at strides from 256 on do waves exchange keys through LDS, one barrier
// each (two buffers alternate).  Of the 55 stages of 1024 keys 19 touch no other lane and 3 meet at a barrier.
// Bound: instruction issue, ~10 vector instructions per key and stage.  Measured at 1024 keys a segment: 16 segments
// 15.0 -> 9.8 us, 1024 segments 26.5 -> 16.6 us against the same network with the keys in LDS (two LDS round trips and
// the index arithmetic of a generic loop per stage).
// Segments of at most 128 keys lie side by side in a wave, 256 keys (padded) of them: 8 x 65536 keys in segments of 16 take
// 4.2 us, of 64 5.5, of 128 7.3 (a wave to a segment padded to 256: 40.5, 13.3 and 9.4; keys in LDS 18.0, 10.9 and 10.3).
// grid = (ceil(G / segments of a workgroup) + 1, batch*h_kv); the last workgroup writes the identity for the unpermuted tail.
// ---------------------------------------------------------------------------------------------
constexpr int kSortPer = 4;
typedef int int4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned long long u64;

// Both values of the pair a lane forms with lane ^ X, in registers of their own; which of the two is the lane's own one
// does not matter for a compare-exchange.  X = 16, 32: the row swaps of a value with itself; below: DPP moves.
template <int X>
__device__ __forceinline__ void lane_pair(uint32_t v, uint32_t &a, uint32_t &b)
{
    if constexpr (X >= 16) {
        const auto sw = X == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false) : __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = sw[0];
        b = sw[1];
    } else {
        a = v;
        if constexpr (X == 1) b = __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, false);            // quad_perm [1,0,3,2]
        else if constexpr (X == 2) b = __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, false);       // quad_perm [2,3,0,1]
        else if constexpr (X == 8) b = __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, false);      // row_ror:8
        else b = __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, false),   // row_half_mirror: 7 - i,
                                          0x1B, 0xf, 0xf, false);                                // quad_perm [3,2,1,0]
    }
}

// this lane keeps the smaller (or the larger) key of the pair it forms with lane ^ X
template <int X>
__device__ __forceinline__ void exchange_lanes(u64 (&key)[kSortPer], bool smaller)
{
#pragma unroll
    for (int e = 0; e < kSortPer; ++e) {
        uint32_t ah, al, bh, bl;
        lane_pair<X>((uint32_t)(key[e] >> 32), ah, bh);
        lane_pair<X>((uint32_t)key[e], al, bl);
        const u64 a = ((u64)ah << 32) | al, b = ((u64)bh << 32) | bl;
        key[e] = (b < a) == smaller ? b : a;
    }
}

__device__ __forceinline__ void exchange_in_lane(u64 &a, u64 &b, bool asc)
{
    const bool swap = (b < a) == asc;
    const u64 t = a;
    a = swap ? b : a;
    b = swap ? t : b;
}

// the bits of a score (INT_KEYS: an int32 key) as an unsigned number in the order of the sort
template <bool INT_KEYS>
__device__ __forceinline__ uint32_t sort_key(int raw)
{
    if (INT_KEYS) return (uint32_t)raw ^ 0x80000000u;        // signed order
    const uint32_t u = __float_as_uint(__int_as_float(raw) + 0.0f);
    return ~((u & 0x80000000u) ? ~u : (u | 0x80000000u));    // descending in u == ascending in the score
}

// identity != NULL: the positions 0 .. n-1 are written there as well (the kidx of a token-order copy).
// INT_KEYS: `scores` holds int32 keys instead, sorted ascending (equal keys in ascending position).
// p2: the segment padded to a power of two; blockDim.x = max(p2, 256) / kSortPer.
template <bool INT_KEYS>
__global__ __launch_bounds__(1024) void segment_argsort_kernel(const float *__restrict__ scores,
                                                               int32_t *__restrict__ kidx,
                                                               int32_t *__restrict__ identity, int n, int segment,
                                                               int G, int p2)
{
    extern __shared__ __align__(16) u64 keys[];              // two buffers of p2 keys (segments of more than one wave)
    const int tid = threadIdx.x, p2_log2 = 31 - __builtin_clz(p2);
    const int per = (int)(blockDim.x * kSortPer) >> p2_log2;  // segments of this workgroup
    const int g0 = blockIdx.x * per;
    const size_t base = (size_t)blockIdx.y * n;
    if (identity) {
        const int lo = min(g0, G) * segment, hi = blockIdx.x == gridDim.x - 1 ? n : min(g0 + per, G) * segment;
        for (int p = lo + tid; p < hi; p += blockDim.x) identity[base + p] = p;
    }
    if (blockIdx.x == gridDim.x - 1) {
        for (int p = G * segment + tid; p < n; p += blockDim.x) kidx[base + p] = p;
        return;
    }
    // this lane's segment and place in it; a segment is a multiple of 16 keys
    const int g = g0 + (tid * kSortPer >> p2_log2), t0 = tid * kSortPer & (p2 - 1);
    const bool mine = g < G && t0 < segment;
    const float *s = scores + base + (size_t)min(g, G - 1) * segment;
    u64 key[kSortPer];
    if (mine) {
        const int4u raw = *reinterpret_cast<const int4u *>(s + t0);
#pragma unroll
        for (int e = 0; e < kSortPer; ++e) {
            key[e] = ((u64)sort_key<INT_KEYS>(raw[e]) << 32) | (uint32_t)(t0 + e);
        }
    } else {
#pragma unroll
        for (int e = 0; e < kSortPer; ++e) key[e] = ~0ull;
    }
    int buffer = 0;
    for (int k = 2; k <= p2; k <<= 1) {
        const bool asc4 = (t0 & k) == 0;                     // direction of this lane's keys for k >= 8 (and k = 4)
        for (int j = k >> 1; j >= 256; j >>= 1) {            // other waves
            u64 *buf = keys + buffer * p2;
            buffer ^= 1;
#pragma unroll
            for (int e = 0; e < kSortPer; ++e) buf[t0 + e] = key[e];
            __syncthreads();
            const bool smaller = ((t0 & j) == 0) == asc4;
            const u64 *from = buf + (t0 ^ j);
#pragma unroll
            for (int e = 0; e < kSortPer; ++e) {
                const u64 other = from[e];
                key[e] = (other < key[e]) == smaller ? other : key[e];
            }
        }
#define PBS_LANES(X)                                                            \
        if (k >= 8 * X) exchange_lanes<X>(key, ((tid & X) == 0) == asc4);
        PBS_LANES(32) PBS_LANES(16) PBS_LANES(8) PBS_LANES(4) PBS_LANES(2) PBS_LANES(1)
#undef PBS_LANES
        if (k >= 4) {
            exchange_in_lane(key[0], key[2], asc4);
            exchange_in_lane(key[1], key[3], asc4);
            exchange_in_lane(key[0], key[1], asc4);
            exchange_in_lane(key[2], key[3], asc4);
        } else {                                             // k = 2
            exchange_in_lane(key[0], key[1], true);
            exchange_in_lane(key[2], key[3], false);
        }
    }
    if (mine) {
        int4u out;
#pragma unroll
        for (int e = 0; e < kSortPer; ++e) out[e] = g * segment + (int32_t)(key[e] & 0xffffffffu);
        *reinterpret_cast<int4u *>(kidx + base + (size_t)g * segment + t0) = out;
    }
}

// ---------------------------------------------------------------------------------------------
// The same order by counting, for calls whose segments are too few to fill the chip: a key's place is the number of keys
// in front of it, so 64 keys of a segment (one per lane) are placed by a workgroup of their own.  The segment's keys lie
// in LDS and are read as broadcasts, 64-key chunk by chunk, the chunks dealt out to the waves; equal keys count
// where they come from an earlier position.  Bound by launch and load latency where it is used: no chain of exchanges.
// grid = (G * chunks + 1, heads), the last workgroup for the tail; scores and kidx must not overlap.
// ---------------------------------------------------------------------------------------------
constexpr int kRankWaves = 8;

template <bool INT_KEYS>
__global__ __launch_bounds__(64 * kRankWaves) void segment_rank_kernel(const float *__restrict__ scores, int32_t *__restrict__ kidx,
                                                           int32_t *__restrict__ identity, int n, int segment, int G,
                                                           int chunks)
{
    extern __shared__ __align__(16) uint32_t rank_lds[];     // chunks * 64 keys, then kRankWaves * 64 counts
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t base = (size_t)blockIdx.y * n;
    const int g = blockIdx.x / chunks, own = blockIdx.x - g * chunks;
    if (g >= G) {
        for (int p = G * segment + tid; p < n; p += 64 * kRankWaves) {
            kidx[base + p] = p;
            if (identity) identity[base + p] = p;
        }
        return;
    }
    const float *s = scores + base + (size_t)g * segment;
    for (int t0 = tid * 4; t0 < chunks * 64; t0 += 256 * kRankWaves) {   // a segment is a multiple of 16 keys
        uintx4 u = {~0u, ~0u, ~0u, ~0u};                     // behind the segment: in front of nothing
        if (t0 < segment) {
            const int4u raw = *reinterpret_cast<const int4u *>(s + t0);
#pragma unroll
            for (int e = 0; e < 4; ++e) u[e] = sort_key<INT_KEYS>(raw[e]);
        }
        *reinterpret_cast<uintx4 *>(rank_lds + t0) = u;
    }
    __syncthreads();
    const uint32_t mine = rank_lds[own * 64 + lane];
    uint32_t before = 0;
    for (int c = wave; c < chunks; c += kRankWaves) {
        const uintx4 *k = reinterpret_cast<const uintx4 *>(rank_lds + c * 64);
        if (c < own) {
#pragma unroll
            for (int q = 0; q < 16; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) before += k[q][e] <= mine;
        } else if (c > own) {
#pragma unroll
            for (int q = 0; q < 16; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) before += k[q][e] < mine;
        } else {
#pragma unroll 2
            for (int q = 0; q < 16; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) before += k[q][e] < mine || (k[q][e] == mine && q * 4 + e < lane);
        }
    }
    uint32_t *counts = rank_lds + chunks * 64;
    counts[tid] = before;
    __syncthreads();
    const int i = own * 64 + lane;
    if (wave != 0 || i >= segment) return;
    int at = 0;
#pragma unroll
    for (int w = 0; w < kRankWaves; ++w) at += (int)counts[w * 64 + lane];
    kidx[base + (size_t)g * segment + at] = g * segment + i;
    if (identity) identity[base + (size_t)g * segment + i] = g * segment + i;
}

// launch shape of the sort: padded segment, threads, dynamic LDS
struct SortShape {
    int p2, threads;
    size_t lds;
};
static SortShape sort_shape(int segment)
{
    int p2 = 16;
    while (p2 < segment) p2 <<= 1;
    const int keys = p2 > 64 * kSortPer ? p2 : 64 * kSortPer;
    return {p2, keys / kSortPer, p2 > 64 * kSortPer ? 2 * (size_t)p2 * sizeof(u64) : 0};
}

// Counting costs a segment's square, the network hardly more than its own depth until it fills the chip: up to 32768 keys
// in all counting is ahead (us, counting / network: 64 segments of 512 keys 6.1 / 6.8, 32 of 1024 7.2 / 9.0, 16 of 2048
// 10.5 / 11.4, 8 of 4096 16.8 / 20.6; 16 of 1024 6.5 / 8.8), past it no longer (64 of 1024 9.0 / 9.0, 128 of 1024
// 14.1 / 9.0); below 256 keys a segment is one wave's network, or part of one.
constexpr int kRankKeys = 32768, kRankMinSegment = 256;

template <bool INT_KEYS>
static pbs_status launch_sort(const Geo &g, int heads, const float *scores, int32_t *idx, int32_t *identity, hipStream_t s)
{
    const int chunks = (g.segment + 63) / 64;
    const uintptr_t in = reinterpret_cast<uintptr_t>(scores), out = reinterpret_cast<uintptr_t>(idx),
                    bytes = (uintptr_t)heads * g.n * sizeof(float);
    if (g.segment >= kRankMinSegment && (long long)heads * g.G * g.segment <= kRankKeys && (in + bytes <= out || out + bytes <= in))
        return launch(segment_rank_kernel<INT_KEYS>, dim3(g.G * chunks + 1, heads), dim3(64 * kRankWaves),
                      ((size_t)chunks + kRankWaves) * 64 * sizeof(uint32_t), s, scores, idx, identity, g.n, g.segment, g.G, chunks);
    const SortShape sh = sort_shape(g.segment);
    static std::atomic<unsigned long long> lds_raised{0};
    if (sh.lds > 32 * 1024) {
        const pbs_status st = raise_lds_limit(reinterpret_cast<const void *>(&segment_argsort_kernel<INT_KEYS>), 64 * 1024, lds_raised);
        if (st != PBS_OK) return st;
    }
    const int per = sh.threads * kSortPer / sh.p2;
    return launch(segment_argsort_kernel<INT_KEYS>, dim3(ceil_div(g.G, per) + 1, heads), dim3(sh.threads), sh.lds, s, scores, idx,
                  identity, g.n, g.segment, g.G, sh.p2);
}

__global__ __launch_bounds__(256) void iota_kernel(int32_t *__restrict__ idx, int32_t *__restrict__ idx2, int n,
                                                   size_t total)
{
    for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < total; p += (size_t)gridDim.x * blockDim.x) {
        idx[p] = (int32_t)(p % (size_t)n);
        if (idx2) idx2[p] = (int32_t)(p % (size_t)n);
    }
}

// A 16-byte load of a source row.  Rows that are read once are read past the caches' retention (non-temporal); with
// the token-order copy every row is read twice, by neighbouring workgroups, and the second read should find it.
template <bool TWICE, typename T>
__device__ inline T load_once_or_twice(const T *ptr)
{
    if constexpr (TWICE) return *ptr;
    else return __builtin_nontemporal_load(ptr);
}

// ---------------------------------------------------------------------------------------------
// Row gather / scatter in 16-byte chunks; cpr = chunks per row (a power of two).
// SCATTER = false: dst[row] = src[head(row), idx[row]]     (X' = P X)
// SCATTER = true : dst[head(row), idx[row]] = src[row]     (O = P^T O')
// idx == NULL is the identity.  An index outside [0, n) gives a zero row (gather) or is dropped (scatter).
// ---------------------------------------------------------------------------------------------
// copy_stride > 0 (gather only): the grid is twice as wide; odd workgroups write a plain copy of the same range of
// rows copy_stride chunks behind dst (the token-order copy), right next in time to the even workgroup that gathers
// rows of the same segments, so that most of what they read is still in the last-level caches.
template <bool SCATTER, bool TWICE = false>
__global__ __launch_bounds__(256) void move_rows_kernel(const uintx4 *__restrict__ src,
                                                        const int32_t *__restrict__ idx,
                                                        uintx4 *__restrict__ dst, int n, int cpr_log2,
                                                        size_t copy_stride)
{
    // grid = (x, nbh): blockIdx.y is the head; workgroup x owns a contiguous range of that head's n * cpr chunks and
    // moves it in batches of U x 256 chunks: all index loads of a batch, then all data loads, then all stores, so
    // that every thread keeps U independent 16-byte loads in flight.
    constexpr int U = 4;
    const size_t head = (size_t)blockIdx.y * n;
    const uint32_t chunks = (uint32_t)n << cpr_log2;
    const uint32_t cmask = (1u << cpr_log2) - 1u;
    const bool plain = copy_stride != 0 && (blockIdx.x & 1);
    const uint32_t wg = copy_stride ? blockIdx.x >> 1 : blockIdx.x, nwg = copy_stride ? gridDim.x >> 1 : gridDim.x;
    const uintx4 *hsrc = src + (head << cpr_log2);
    uintx4 *hdst = dst + (head << cpr_log2) + (plain ? copy_stride : 0);
    const int32_t *hidx = (idx && !plain) ? idx + head : nullptr;
    const uint32_t batch = U * 256;
    const uint32_t per = ((chunks + nwg - 1) / nwg + batch - 1) / batch * batch;
    const uint32_t begin = min(wg * per, chunks), end = min(begin + per, chunks);
    for (uint32_t c0 = begin + threadIdx.x; c0 < end; c0 += batch) {
        int32_t other[U];
        uintx4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t c = c0 + u * 256;
            other[u] = c < end ? (hidx ? hidx[c >> cpr_log2] : (int32_t)(c >> cpr_log2)) : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t c = c0 + u * 256;
            const bool ok = other[u] >= 0 && other[u] < n;
            v[u] = uintx4{0u, 0u, 0u, 0u};
            if (SCATTER ? c < end : ok)
                v[u] = load_once_or_twice<TWICE>(hsrc + (SCATTER ? c : ((uint32_t)other[u] << cpr_log2) + (c & cmask)));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t c = c0 + u * 256;
            const bool ok = other[u] >= 0 && other[u] < n;
            if (SCATTER ? ok : c < end)
                __builtin_nontemporal_store(v[u], hdst + (SCATTER ? ((uint32_t)other[u] << cpr_log2) + (c & cmask) : c));
        }
    }
}

// ---------------------------------------------------------------------------------------------
// The row gather of K' for 2-byte storage (move_rows_kernel<false> with the same grid, ranges and token-order copy)
// that also leaves the block means of K' behind, as Algorithm 2 needs them next: kbarT[head][feature][Ts] fp64.
// A workgroup owns whole key blocks (its range is a multiple of block * cpr chunks, and a block is a whole number of
// 1024-chunk batches), a thread always meets the same 16-byte column group, so it adds up its rows' eight features in
// fp64 registers while the rows pass through (sums of bf16 values are exact in fp64 in any order), and at the end of
// every block the 256 / cpr row slots of a column meet in LDS.  dst == NULL: only the block means are produced (index
// remapping: the attention kernel gathers the rows itself and no K' is written).
// ---------------------------------------------------------------------------------------------
template <bool TWICE>
__device__ __forceinline__ void gather_pool(const uintx4 *__restrict__ src, const int32_t *__restrict__ idx,
                                            uintx4 *__restrict__ dst, int n, int cpr_log2, size_t copy_stride,
                                            double *__restrict__ kbarT, int block, int Ts, uint32_t bx, uint32_t gx,
                                            double *red /* 256 * 8, LDS */)
{
    constexpr int U = 4;
    const size_t head = (size_t)blockIdx.y * n;
    const uint32_t chunks = (uint32_t)n << cpr_log2;
    const uint32_t cpr = 1u << cpr_log2, cmask = cpr - 1u;
    const bool plain = copy_stride != 0 && (bx & 1);
    const uint32_t wg = copy_stride ? bx >> 1 : bx, nwg = copy_stride ? gx >> 1 : gx;
    const uintx4 *hsrc = src + (head << cpr_log2);
    uintx4 *hdst = dst + (head << cpr_log2) + (plain ? copy_stride : 0);
    const int32_t *hidx = (idx && !plain) ? idx + head : nullptr;
    const uint32_t batch = U * 256;
    const uint32_t cpb = (uint32_t)block << cpr_log2;        // chunks per key block, a multiple of batch
    const uint32_t per = ((chunks + nwg - 1) / nwg + cpb - 1) / cpb * cpb;
    const uint32_t begin = min(wg * per, chunks), end = min(begin + per, chunks);
    const int d = 8 << cpr_log2;
    double acc[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) acc[x] = 0.0;
    for (uint32_t base = begin; base < end; base += batch) {
        int32_t other[U];
        uintx4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t c = base + threadIdx.x + u * 256;
            other[u] = c < end ? (hidx ? hidx[c >> cpr_log2] : (int32_t)(c >> cpr_log2)) : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t c = base + threadIdx.x + u * 256;
            v[u] = uintx4{0u, 0u, 0u, 0u};
            if (other[u] >= 0 && other[u] < n)
                v[u] = load_once_or_twice<TWICE>(hsrc + ((uint32_t)other[u] << cpr_log2) + (c & cmask));
        }
        if (dst) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t c = base + threadIdx.x + u * 256;
                if (c < end) __builtin_nontemporal_store(v[u], hdst + c);
            }
        }
        if (plain) continue;                                  // uniform: the token-order copy is not pooled
#pragma unroll
        for (int u = 0; u < U; ++u)                           // rows past the end were loaded as zeros
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                acc[2 * x] += (double)__uint_as_float(v[u][x] << 16);
                acc[2 * x + 1] += (double)__uint_as_float(v[u][x] & 0xffff0000u);
            }
        const uint32_t done = base + batch - begin;
        if (done % cpb == 0 || base + batch >= end) {         // uniform: a key block is complete
            const int blk = (int)((base >> cpr_log2) / (uint32_t)block);
            const int rows = min(block, n - blk * block);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                red[threadIdx.x * 8 + x] = acc[x];
                acc[x] = 0.0;
            }
            __syncthreads();
            if ((int)threadIdx.x < d) {
                const int e = threadIdx.x;
                double s = 0.0;
                for (uint32_t q = 0; q < 256 / cpr; ++q) s += red[(q * cpr + (e >> 3)) * 8 + (e & 7)];
                kbarT[((size_t)blockIdx.y * d + e) * Ts + blk] = s / (double)rows;
            }
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------------------------
// V' in the block-transposed layout Vt[bh][j][e][c] = V[bh][kidx[j*block + c]][e] (zero for slots >= n).
// One workgroup per (key block j, bh): gathered rows go to LDS with coalesced 16-byte reads, the tile is
// read back column-wise in 4-byte words and leaves as 16-byte pieces of Vt rows (VEC keys of one feature),
// neighbouring lanes writing neighbouring pieces of a key group, then the next feature.  LDS row r starts at word
// r * (row words) + (r / VEC) * (64 / gpp) with gpp pieces per Vt row: the lanes of a wave read gpp pieces x
// 64 / gpp word columns, which then fall into 64 different banks.
// E = storage type (2 or 4 bytes); VEC = elements per 16-byte chunk.
// ---------------------------------------------------------------------------------------------
// copy_stride > 0: the grid is twice as wide; odd workgroups transpose the same key block without the permutation
// into the copy copy_stride elements behind Vt (see move_rows_kernel).
template <typename E, bool TWICE>
__device__ __forceinline__ void gather_vt(const E *__restrict__ V, const int32_t *__restrict__ kidx, E *__restrict__ Vt,
                                          int n, int d, int block, int T, size_t copy_stride, uint32_t bx,
                                          uint32_t *tile /* LDS */)
{
    constexpr int VEC = 16 / sizeof(E);
    const int roww = d * (int)sizeof(E) / 4;               // 4-byte words per row
    const bool plain = copy_stride != 0 && (bx & 1);
    const int j = copy_stride ? bx >> 1 : bx;
    const size_t bh = blockIdx.y;
    if (plain) kidx = nullptr;
    const int cpr = d / VEC;
    const int G = vt_group(block);                         // keys per transposed group
    const int gpp = G / VEC;                               // 16-byte pieces per Vt row
    const int skew = 64 / gpp;                             // words; gpp is 2, 4 or 8
    typedef E vec_t __attribute__((ext_vector_type(VEC)));
    // batches of U chunks per thread: index loads, then row loads, then the LDS stores
    constexpr int U = 4;
    const int total = block * cpr;
    for (int c0 = threadIdx.x; c0 < total; c0 += U * 256) {
        int32_t from[U];
        vec_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * 256;
            const int slot = j * block + c / cpr;
            from[u] = (c < total && slot < n) ? (kidx ? kidx[bh * n + slot] : slot) : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * 256;
            v[u] = vec_t{};
            if (from[u] >= 0 && from[u] < n)
                v[u] = load_once_or_twice<TWICE>(reinterpret_cast<const vec_t *>(V + (bh * n + from[u]) * (size_t)d + (c % cpr) * VEC));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * 256;
            const int row = c / cpr;
            if (c < total) *reinterpret_cast<vec_t *>(tile + row * roww + (row / VEC) * skew + (c % cpr) * 4) = v[u];
        }
    }
    __syncthreads();
    E *out = Vt + (bh * T + j) * (size_t)d * block + (plain ? copy_stride : 0);
    for (int c = threadIdx.x; c < roww * (block / VEC); c += blockDim.x) {
        const int kgi = c % gpp, w = (c / gpp) % roww, gi = c / (gpp * roww);
        const int kg = gi * gpp + kgi;                     // word column w of the rows kg*VEC .. kg*VEC+VEC-1
        uint32_t x[VEC];
#pragma unroll
        for (int u = 0; u < VEC; ++u) x[u] = tile[(kg * VEC + u) * roww + kg * skew + w];
        E *og = out + (size_t)gi * d * G + kgi * VEC;      // feature e of this piece: og + e * G
        if (sizeof(E) == 4) {
            uintx4 v;
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = x[u];
            __builtin_nontemporal_store(v, reinterpret_cast<uintx4 *>(og + (size_t)w * G));
        } else {                                           // word w holds elements 2w (low half) and 2w + 1
            uintx4 lo, hi;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                lo[u] = __builtin_amdgcn_perm(x[(2 * u + 1) % VEC], x[(2 * u) % VEC], 0x05040100u);
                hi[u] = __builtin_amdgcn_perm(x[(2 * u + 1) % VEC], x[(2 * u) % VEC], 0x07060302u);
            }
            __builtin_nontemporal_store(lo, reinterpret_cast<uintx4 *>(og + (size_t)(2 * w) * G));
            __builtin_nontemporal_store(hi, reinterpret_cast<uintx4 *>(og + (size_t)(2 * w + 1) * G));
        }
    }
}

template <typename E, bool TWICE>
__global__ __launch_bounds__(256) void gather_vt_kernel(const E *__restrict__ V, const int32_t *__restrict__ kidx,
                                                        E *__restrict__ Vt, int n, int d, int block, int T,
                                                        size_t copy_stride)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    gather_vt<E, TWICE>(V, kidx, Vt, n, d, block, T, copy_stride, blockIdx.x, reinterpret_cast<uint32_t *>(smem_raw));
}

// Both gathers of a head in one launch: workgroups 0 .. kwgs - 1 move K rows, the rest key blocks of V.  They do not
// depend on each other, and a launch of its own costs each of them its ramp and its tail: 159 + 164 -> 311 us at
// 8 x 131072 keys with the token-order copies (7 TB/s), 6.4 + 5.9 -> 7.9 us at 8 x 2048.
// LDS (dynamic): what either of the two needs.
template <bool TWICE>
__global__ __launch_bounds__(256) void gather_both_kernel(const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
                                                          const int32_t *__restrict__ kidx, uint16_t *__restrict__ Kp,
                                                          uint16_t *__restrict__ Vt, int n, int d, int cpr_log2,
                                                          size_t kcopy, size_t vcopy, double *__restrict__ kbarT,
                                                          int block, int T, int Ts, uint32_t kwgs)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if (blockIdx.x < kwgs)
        gather_pool<TWICE>(reinterpret_cast<const uintx4 *>(K), kidx, reinterpret_cast<uintx4 *>(Kp), n, cpr_log2, kcopy, kbarT, block, Ts, blockIdx.x, kwgs,
                           reinterpret_cast<double *>(smem_raw));
    else
        gather_vt<uint16_t, TWICE>(V, kidx, Vt, n, d, block, T, vcopy, blockIdx.x - kwgs,
                                   reinterpret_cast<uint32_t *>(smem_raw));
}

// The rows of one key block of K and their mean, for storage and blocks that gather_pool does not take (float; 2-byte blocks of
// fewer than 1024 chunks): the workgroup owns the block whole.  bf16 values are summed on the way, as there; float rows
// are kept in LDS and added in ascending order, column by column.  Odd workgroups write the token-order copy, as everywhere.
template <typename E, bool TWICE>
__device__ __forceinline__ void gather_block(const uintx4 *__restrict__ src, const int32_t *__restrict__ idx,
                                             uintx4 *__restrict__ dst, int n, int cpr_log2, size_t copy_stride,
                                             double *__restrict__ kbarT, int block, int Ts, uint32_t bx, unsigned char *lds)
{
    constexpr int U = 4;
    constexpr bool wide = sizeof(E) == 4;
    const bool plain = copy_stride != 0 && (bx & 1);
    const int j = (int)(copy_stride ? bx >> 1 : bx), row0 = j * block, rows = min(block, n - row0);
    const int cpr = 1 << cpr_log2, total = rows << cpr_log2, d = cpr * (16 / (int)sizeof(E));
    const size_t head = (size_t)blockIdx.y * n;
    const uintx4 *hsrc = src + (head << cpr_log2);
    uintx4 *hdst = dst + ((head + row0) << cpr_log2) + (plain ? copy_stride : 0);
    const int32_t *hidx = plain ? nullptr : idx + head + row0;
    uintx4 *tile = reinterpret_cast<uintx4 *>(lds);        // float: the block's rows
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};            // bf16: this thread's column group
    for (int c0 = threadIdx.x; c0 < total; c0 += U * 256) {
        int32_t from[U];
        uintx4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = (c0 + u * 256) >> cpr_log2;
            from[u] = row < rows ? (hidx ? hidx[row] : row0 + row) : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = uintx4{0u, 0u, 0u, 0u};
            if (from[u] >= 0 && from[u] < n)
                v[u] = load_once_or_twice<TWICE>(hsrc + ((size_t)from[u] << cpr_log2) + ((c0 + u * 256) & (cpr - 1)));
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c0 + u * 256 < total) {
                __builtin_nontemporal_store(v[u], hdst + c0 + u * 256);
                if (wide && !plain) tile[c0 + u * 256] = v[u];
            }
        if (!wide && !plain) {
#pragma unroll
            for (int u = 0; u < U; ++u)                    // rows past the end were loaded as zeros
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    acc[2 * x] += (double)__uint_as_float(v[u][x] << 16);
                    acc[2 * x + 1] += (double)__uint_as_float(v[u][x] & 0xffff0000u);
                }
        }
    }
    if (plain) return;
    double *red = reinterpret_cast<double *>(lds);         // 256 * 8
    if (!wide) {
#pragma unroll
        for (int x = 0; x < 8; ++x) red[threadIdx.x * 8 + x] = acc[x];
    }
    __syncthreads();
    const int e = threadIdx.x;
    if (e >= d) return;
    double s = 0.0;
    if (wide) {
        const float *column = reinterpret_cast<const float *>(lds) + e;
        int r = 0;
        for (; r + 16 <= rows; r += 16) {                  // the reads of sixteen rows go out ahead of their additions
            float v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = column[(r + u) * d];
#pragma unroll
            for (int u = 0; u < 16; ++u) s += (double)v[u];
        }
        for (; r < rows; ++r) s += (double)column[r * d];
    } else {
        for (int q = 0; q < 256 / cpr; ++q) s += red[(q * cpr + (e >> 3)) * 8 + (e & 7)];
    }
    kbarT[((size_t)blockIdx.y * d + e) * Ts + j] = s / (double)rows;
}

// gather_both_kernel for the blocks of gather_block.  One launch in the place of three (rows, means, V'): short ones were mostly their
// own start and end, and long ones read K' once more for its means.  Whole stage, three launches / this, us: float, 2 heads x 2048
// x 64 14.3 / 10.0, 8 x 131072 x 64 244 / 190, 8 x 131072 x 128, block 128 (64 KiB of LDS) 517 / 425, with the token-order copies 788 /
// 694, 8 x 65536 x 128, block 16 274 / 209; bf16, 4 x 12288 x 64, block 64 20.4 / 13.6, 8 x 131072 141 / 109, with copies 205 / 178,
// 8 x 65536 x 64, block 16 (a workgroup of 2 KiB) 119 / 109, block 32 92 / 71.
template <typename E, bool TWICE>
__global__ __launch_bounds__(256) void gather_blocks_kernel(const E *__restrict__ K, const E *__restrict__ V,
                                                            const int32_t *__restrict__ kidx, E *__restrict__ Kp,
                                                            E *__restrict__ Vt, int n, int d, int cpr_log2, size_t kcopy,
                                                            size_t vcopy, double *__restrict__ kbarT, int block, int T, int Ts,
                                                            uint32_t kwgs)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if (blockIdx.x < kwgs)
        gather_block<E, TWICE>(reinterpret_cast<const uintx4 *>(K), kidx, reinterpret_cast<uintx4 *>(Kp), n, cpr_log2, kcopy,
                               kbarT, block, Ts, blockIdx.x, smem_raw);
    else
        gather_vt<E, TWICE>(V, kidx, Vt, n, d, block, T, vcopy, blockIdx.x - kwgs, reinterpret_cast<uint32_t *>(smem_raw));
}

static int ilog2(int v) { int l = 0; while ((1 << l) < v) ++l; return l; }

static int grid_for(size_t items, int per_block)
{
    size_t b = (items + per_block - 1) / per_block;
    const size_t cap = 256 * 32;                          // 32 workgroups per CU is plenty for a copy
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (int)b;
}

// grid for move_rows_kernel and the K half of gather_both_kernel: one batch of 4 x 256 chunks (16 KiB) per workgroup -- or `unit`
// chunks where a workgroup has to own whole key blocks --, so that the workgroups in flight at any time sweep one
// narrow window of addresses (measured on a plain 1 GiB copy: 5.3 TB/s read + write with 1024 long ranges, 6.3 with
// 65536 short ones and non-temporal accesses)
static dim3 move_grid(int n, int cpr, int nbh, size_t unit = 256 * 4)
{
    const size_t chunks = (size_t)n * cpr;
    size_t bx = (chunks + unit - 1) / unit;
    if (bx < 1) bx = 1;
    return dim3((unsigned)bx, (unsigned)nbh);
}

// idx[head][g*S + t] = position of the query with the t-th smallest (key, position) of segment g; the tail keeps its place.
pbs_status launch_segment_sort_by_int_key(const Geo &g, int heads, const int32_t *keys, int32_t *idx, hipStream_t s)
{
    return launch_sort<true>(g, heads, reinterpret_cast<const float *>(keys), idx, nullptr, s);
}

size_t ws_block_mask(const pbs_problem *p);

}  // namespace pbs

using namespace pbs;

extern "C" pbs_status pbs_segment_permute(const pbs_problem *p, const float *scores, const void *K, const void *V,
                                          int32_t *kidx, void *Kp, void *Vt, void *ws, size_t ws_bytes,
                                          void *stream)
{
    pbs_status st = validate(p);
    if (st != PBS_OK) return st;
    if (!kidx) return PBS_ERR_NULL;
    const bool remap = (p->flags & PBS_FLAG_INDEX_REMAP) != 0;    // no K' is written: Kp is ignored and may be NULL
    if (remap) {
        if (p->flags & PBS_FLAG_TOKEN_ORDER_COPY) return PBS_ERR_UNSUPPORTED;
        if (Vt && !Kp) Kp = Vt;                                   // "both or none" below is about Vt alone then
        if (!Vt) Kp = nullptr;
    }
    if ((Kp == nullptr) != (Vt == nullptr)) return PBS_ERR_NULL;
    if (ws && Kp && ((reinterpret_cast<uintptr_t>(ws) & (kWsAlign - 1)) != 0 || ws_bytes < ws_block_mask(p)))
        return PBS_ERR_WORKSPACE;
    if (Kp && (!K || !V)) return PBS_ERR_NULL;
    if (Kp && (!aligned16(K) || !aligned16(V) || !aligned16(Kp) || !aligned16(Vt))) return PBS_ERR_SHAPE;
    void *kdst = remap ? nullptr : Kp;
    const Geo g = make_geo(p);
    hipStream_t s = (hipStream_t)stream;
    const int nbh = g.batch * g.h_kv;
    const bool token_copy = (p->flags & PBS_FLAG_TOKEN_ORDER_COPY) != 0;
    const size_t tok_rows = (size_t)nbh * g.T * g.block;   // the token-order copies start this many rows in
    int32_t *kidx_tok = token_copy ? kidx + tok_rows : nullptr;
    if (scores) {
        st = launch_sort<false>(g, nbh, scores, kidx, kidx_tok, s);
    } else {
        const size_t total = (size_t)nbh * g.n;
        st = launch(iota_kernel, dim3(grid_for(total, 256)), dim3(256), 0, s, kidx, kidx_tok, g.n, total);
    }
    if (st != PBS_OK) return st;
    if (!Kp) return PBS_OK;
    const size_t es = elem_size(p->dtype);
    const int cpr = (int)(g.d * es / 16);
    const size_t vt_half = (size_t)nbh * g.T * g.d * g.block;           // elements

    // with a workspace, the block means of K' are left there for pbs_block_mask by the gather itself: gather_pool where a key
    // block is a whole number of its 1024-chunk batches (2-byte storage), gather_block otherwise
    double *kbarT = reinterpret_cast<double *>(ws);
    const bool pool_on_the_way = kbarT && p->dtype == PBS_BF16 && (g.block * cpr) % 1024 == 0;
    dim3 mg = pool_on_the_way ? move_grid(g.n, cpr, nbh, (size_t)g.block * cpr) : move_grid(g.n, cpr, nbh);
    if (token_copy) mg.x *= 2;
    if (remap && kbarT && !pool_on_the_way) return PBS_ERR_UNSUPPORTED;   // means without K' only from the gather kernel
    const size_t kcopy = token_copy ? tok_rows * cpr : (size_t)0;
    const int Tsk = kbar_stride(g.T), cl = ilog2(cpr);
    const dim3 vg(token_copy ? 2 * g.T : g.T, nbh);
    const size_t vcopy = token_copy ? vt_half : (size_t)0;
    const size_t vlds = p->dtype == PBS_BF16                              // tile + skew
                            ? (size_t)g.block * g.d * 2 + (size_t)(g.block / 8) * (64 / (vt_group(g.block) / 8)) * 4
                            : (size_t)g.block * g.d * 4 + (size_t)(g.block / 4) * (64 / (vt_group(g.block) / 4)) * 4;
    if (kbarT) {
        // V' may take the place of K, which nothing needs once K' is gathered: then one after the other
        const uintptr_t k0 = reinterpret_cast<uintptr_t>(K), v0 = reinterpret_cast<uintptr_t>(Vt);
        const bool in_place = v0 < k0 + (size_t)nbh * g.n * g.d * es && k0 < v0 + pbs_vt_bytes(p);
        const unsigned kwgs = pool_on_the_way ? mg.x : vg.x;                // by blocks: as many workgroups as V' takes
        const size_t klds = p->dtype == PBS_BF16 ? 256 * 8 * sizeof(double) : (size_t)g.block * g.d * 4;
        const size_t lds = vlds > klds ? vlds : klds;
        auto gather = [&](auto kernel, auto *element, unsigned kw, unsigned vw) {
            typedef std::remove_pointer_t<decltype(element)> E;
            return launch(kernel, dim3(kw + vw, nbh), dim3(256), lds, s, (const E *)K, (const E *)V, (const int32_t *)kidx, (E *)kdst,
                          (E *)Vt, g.n, g.d, cl, kcopy, vcopy, kbarT, g.block, g.T, Tsk, kw);
        };
        auto part = [&](unsigned kw, unsigned vw) {
            uint16_t *two = nullptr;
            uint32_t *four = nullptr;
            if (p->dtype != PBS_BF16)
                return token_copy ? gather(gather_blocks_kernel<uint32_t, true>, four, kw, vw)
                                  : gather(gather_blocks_kernel<uint32_t, false>, four, kw, vw);
            if (pool_on_the_way)
                return token_copy ? gather(gather_both_kernel<true>, two, kw, vw) : gather(gather_both_kernel<false>, two, kw, vw);
            return token_copy ? gather(gather_blocks_kernel<uint16_t, true>, two, kw, vw)
                              : gather(gather_blocks_kernel<uint16_t, false>, two, kw, vw);
        };
        if (!in_place) return part(kwgs, vg.x);
        st = part(kwgs, 0);
        return st == PBS_OK ? part(0, vg.x) : st;
    }
    if (kdst)
        st = token_copy ? launch((move_rows_kernel<false, true>), mg, dim3(256), 0, s, (const uintx4 *)K,
                                 (const int32_t *)kidx, (uintx4 *)kdst, g.n, cl, kcopy)
                        : launch((move_rows_kernel<false, false>), mg, dim3(256), 0, s, (const uintx4 *)K,
                                 (const int32_t *)kidx, (uintx4 *)kdst, g.n, cl, kcopy);
    if (st != PBS_OK) return st;
    if (p->dtype == PBS_BF16)
        st = token_copy ? launch((gather_vt_kernel<uint16_t, true>), vg, dim3(256), vlds, s, (const uint16_t *)V,
                                 (const int32_t *)kidx, (uint16_t *)Vt, g.n, g.d, g.block, g.T, vcopy)
                        : launch((gather_vt_kernel<uint16_t, false>), vg, dim3(256), vlds, s, (const uint16_t *)V,
                                 (const int32_t *)kidx, (uint16_t *)Vt, g.n, g.d, g.block, g.T, vcopy);
    else
        st = token_copy ? launch((gather_vt_kernel<uint32_t, true>), vg, dim3(256), vlds, s, (const uint32_t *)V,
                                 (const int32_t *)kidx, (uint32_t *)Vt, g.n, g.d, g.block, g.T, vcopy)
                        : launch((gather_vt_kernel<uint32_t, false>), vg, dim3(256), vlds, s, (const uint32_t *)V,
                                 (const int32_t *)kidx, (uint32_t *)Vt, g.n, g.d, g.block, g.T, vcopy);
    return st;
}

extern "C" pbs_status pbs_permute_rows(const pbs_problem *p, int32_t heads, const void *X, const int32_t *idx,
                                       void *Xp, void *stream)
{
    pbs_status st = validate(p);
    if (st != PBS_OK) return st;
    if (!X || !idx || !Xp) return PBS_ERR_NULL;
    if (heads < 1) return PBS_ERR_SHAPE;
    if ((long long)p->batch * heads > 65535) return PBS_ERR_UNSUPPORTED;   // heads ride on gridDim.y
    if (!aligned16(X) || !aligned16(Xp) || X == Xp) return PBS_ERR_SHAPE;
    const int cpr = (int)(p->d * elem_size(p->dtype) / 16);
    return launch(move_rows_kernel<false>, move_grid(p->n, cpr, p->batch * heads), dim3(256), 0,
                       (hipStream_t)stream, (const uintx4 *)X, idx, (uintx4 *)Xp, p->n, ilog2(cpr), (size_t)0);
}

extern "C" pbs_status pbs_unpermute(const pbs_problem *p, const void *Op, const int32_t *qidx, void *O, void *stream)
{
    pbs_status st = validate(p);
    if (st != PBS_OK) return st;
    if (!Op || !O) return PBS_ERR_NULL;
    if (!aligned16(Op) || !aligned16(O)) return PBS_ERR_SHAPE;
    if (Op == O) return qidx ? PBS_ERR_SHAPE : PBS_OK;     // in place only for the identity
    const int cpr = (int)(p->d * elem_size(p->dtype) / 16);
    return launch(move_rows_kernel<true>, move_grid(p->n, cpr, p->batch * p->h_q), dim3(256), 0,
                       (hipStream_t)stream, (const uintx4 *)Op, qidx, (uintx4 *)O, p->n, ilog2(cpr), (size_t)0);
}

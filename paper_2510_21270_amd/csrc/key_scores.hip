// pbs_key_scores: Eq. 4 with group-averaged queries (appendix "GQA Handling").
//
//   scores[j] = (1/B') * sum_r softmax_j( Qhat[r] . K[j] * scale ),   r over the last B' = min(block, n) rows
//
// The row softmax needs the global maximum and normaliser of each of the B' rows over all n keys, so K is
// swept twice: sweep 1 produces per-row (max, sum-exp) partials, a tiny kernel merges them into one
// constant c[r] = -max_r - log2(B' * sumexp_r) (log2 domain), and sweep 2 evaluates
// scores[j] = sum_r exp2(logit2[r][j] + c[r]).  Sweep 2 walks the key tiles in reverse so that it starts
// on what sweep 1 left in the last-level cache.
//
// bf16, d = 128: both sweeps form the 128 x keys logit tile on the matrix cores (32x32x16 bf16 MFMA, fp32
// accumulator).  Qhat is an fp32 mean, not a bf16 value, so it is pre-multiplied by scale*log2(e) and split
// into two bf16 terms hi + lo; each tile takes two MFMAs per fragment.  A wave keeps the fragments of its rows
// of Qhat in registers (64 rows for long inputs, 32 for short ones) and the K tiles go through LDS, shared by the waves of
// a workgroup.  Both forms compute a logit, and the sums of a range of keys, with the same operations in the same order.  How
// long the ranges are is a matter of a head's length up to 262144 keys in all, and of the keys of all heads from there on
// (sweep_range_keys).
// Everything else (fp32 inputs, d = 64): the same two sweeps on the fp64 matrix instruction.
#include <utility>

#include "pbs_host.h"

namespace pbs {

constexpr int kQRows = 128;            // logit tile rows (>= B')
constexpr int kSweepWgs = 512;         // workgroups of the MFMA sweeps that the chip holds: two on each of 256 compute units
constexpr int kMaxRangeKeys = 1024;                        // keys of a range at most (sweep_range_keys)
constexpr long long kLongKeys = 327680;                    // keys of all heads from which on the long sweeps run (long_sweeps)
constexpr float kLog2e = 1.4426950408889634f;

// ------------------------------------------------------------------ MFMA path: prep
// qsplit[bh][row tile][feature step][term][lane][8]: the operand fragments of the 32 x 32 x 16 instruction one after the other
// (lane = row % 32 + 32 h holds d = 16 step + 8 h .. + 8 of its row), so that a wave loads each as 1 KiB of consecutive
// bytes.  Rows >= bl are zero.
// qrows: positions of the bl query rows (device memory), or NULL for the last bl rows of the sequence (Eq. 4);
// positions outside [0, n) are clamped.  qavg != NULL instead: one query row, the fp64 mean over all positions.
__device__ inline int query_row_position(const int32_t *qrows, int row, int bl, int n)
{
    if (!qrows) return n - bl + row;
    const int pos = qrows[row];
    return pos < 0 ? 0 : (pos >= n ? n - 1 : pos);
}

__device__ __forceinline__ size_t qfrag_offset(int bh, int row_tile, int step, int term)
{
    return (size_t)bh * 2 * kQRows * 128 + ((row_tile * 8 + step) * 2 + term) * 512;
}

__global__ __launch_bounds__(256) void qhat_split_kernel(const bf16_t *__restrict__ Q, bf16_t *__restrict__ qsplit,
                                                         Geo g, int bl, const int32_t *__restrict__ qrows,
                                                         const double *__restrict__ qavg)
{
    // grid = (kQRows / 8, batch * h_kv): each workgroup converts 8 rows x 128 columns, 4 elements per thread
    const int bh = blockIdx.y;
    const int b = bh / g.h_kv, h = bh % g.h_kv;
    const float mul = g.scale * kLog2e / (float)g.r;
    const int row = blockIdx.x * 8 + (threadIdx.x >> 5);
    const int e0 = (threadIdx.x & 31) * 4;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float mul_row = mul;
    if (row < bl) {
        if (qavg) {                                           // already the mean over heads and positions
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[x] = (float)qavg[(size_t)bh * 128 + e0 + x];
            mul_row = g.scale * kLog2e;
        } else {
            const int pos = query_row_position(qrows, row, bl, g.n);
            for (int t = 0; t < g.r; ++t) {
                const bf16x4 v = *reinterpret_cast<const bf16x4 *>(
                    Q + (((size_t)b * g.h_q + h * g.r + t) * g.n + pos) * 128 + e0);
#pragma unroll
                for (int x = 0; x < 4; ++x) acc[x] += (float)v[x];
            }
        }
    }
    bf16x4 vh, vl;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const float v = acc[x] * mul_row;
        vh[x] = (bf16_t)v;
        vl[x] = (bf16_t)(v - (float)vh[x]);
    }
    bf16_t *dst = qsplit + qfrag_offset(bh, row >> 5, e0 >> 4, 0) + ((row & 31) + 32 * ((e0 >> 3) & 1)) * 8 + (e0 & 7);
    *reinterpret_cast<bf16x4 *>(dst) = vh;
    *reinterpret_cast<bf16x4 *>(dst + 512) = vl;
}

// ------------------------------------------------------------------ MFMA path: tiles and fragments
// Both sweeps multiply the 128 rows of Qhat with every key, two bf16 terms each: 64 matrix instructions of 32 x 32 x 16
// per 32 keys.  A workgroup is two waves; wave w owns the rows 64 w .. 64 w + 63 (two row tiles) and keeps their fragments in
// registers (2 row tiles x 8 feature steps x 2 terms x 4 registers), so that a K fragment read from LDS feeds four
// MFMAs and one wave runs per SIMD.  A wave issues in order, so the two halves of the work are interleaved by hand:
//     iteration t:  MFMAs 0..31: logits of tile t + 1, row tile 0, then row tile 1;  all along: exponentials and sums of
//                   tile t, one logit per MFMA, in the same order
//                   K fragments of tile t + 2 under MFMAs 18, 20 .. 30 (and 0), as tile t + 1 is done with theirs;
//                   after MFMA 8 the waves meet, then the loads of tile t + 5 go out
// Tiles travel to LDS asynchronously, through a ring of four; a load has three iterations to arrive.
// Bound by the matrix work under the chip's power limit and, close behind, by the stream of K: 8 heads of 131072 keys (two sweeps
// of 69 GFLOP and 268 MB each) 136 -> 125.5 us for the stage against four waves of 32 rows, two to a SIMD, whose staging,
// exponentials and products took turns.  (The 16 x 16 x 32 instruction, which the power limit favours, was seen at 110 us in
// a form of these sweeps that adds a logit's products in another order; the short form would have to change with it.)
constexpr int kTileKeys = 32;
constexpr int kTileB = kTileKeys * 256;

typedef __attribute__((address_space(3))) void *lptr_t;

// 32 keys x 256 bytes; the 16-byte piece c of key r sits at r * 256 + ((c ^ (r & 15)) << 4): conflict-free for the
// fragment reads (16 lanes = 16 keys, one piece each).  The ring's tiles are separate variables, so that the compiler can
// tell a read of one from an asynchronous load into another.
struct __align__(16) KTile {
    unsigned char b[kTileB];
};

// Descriptor of a workgroup's keys (bytes of them) and byte offsets of this lane: dma[j]: in memory, of the piece it moves in
// load j of its wave, ahead of 1024 j (the instruction's own offset, which counts in memory and in LDS); kfr[x]: in LDS, of
// its piece of feature step x.
struct KSource {
    __amdgpu_buffer_rsrc_t keys;
    int bytes;
    uint32_t dma[4], kfr[8];
};

// Scalar offset of what wave w moves of tile t.  The hardware compares a lane's own offset with the descriptor's size less the
// scalar offset, a difference that must not fall below zero: a tile past the last key starts at the end, where every lane
// is out of range.
__host__ __device__ constexpr int tile_offset(int t, int wave, int bytes)
{
    const int first = t * kTileB + wave * (kTileB / 2);
    return first < bytes ? first : bytes;
}
constexpr bool tile_offsets_hold()
{
    for (int keys = 1; keys <= 3 * kTileKeys; ++keys)
        for (int t = 0; t <= 3 + 32; ++t)                  // what is loaded past the end starts up to a range of tiles behind it
            for (int wave = 0; wave < 2; ++wave) {
                const int at = tile_offset(t, wave, keys * 256);
                if (at > keys * 256 || (t * kTileKeys + wave * 16 < keys && at != (t * kTileKeys + wave * 16) * 256)) return false;
            }
    return true;
}
static_assert(tile_offsets_hold(), "no load starts behind the descriptor's end, and every key is loaded from its place");

__device__ __forceinline__ KSource key_source(const bf16_t *first, int keys, int lane)
{
    KSource k;
    k.bytes = keys * 256;
    k.keys = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(first), 0, k.bytes, 0x00020000);
    const int row = lane >> 4, place = lane & 15, key = lane & 31;
#pragma unroll
    for (int j = 0; j < 4; ++j) k.dma[j] = (uint32_t)(row * 256 + ((place ^ (4 * j + row)) << 4));
#pragma unroll
    for (int x = 0; x < 8; ++x) k.kfr[x] = (uint32_t)(key * 256 + (((2 * x + (lane >> 5)) ^ (key & 15)) << 4));
    return k;
}

// Wave w moves keys 16 w .. 16 w + 15 of tile t (past the last key: zeros, without a memory access)
__device__ __forceinline__ void issue_tile(KTile &tile, const KSource &src, int t, int wave)
{
    const lptr_t dst = (lptr_t)((__attribute__((address_space(3))) unsigned char *)tile.b + wave * 4096);
    const int soff = tile_offset(t, wave, src.bytes);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src.keys, dst, 16, src.dma[0], soff, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src.keys, dst, 16, src.dma[1], soff, 1024, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src.keys, dst, 16, src.dma[2], soff, 2048, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src.keys, dst, 16, src.dma[3], soff, 3072, 0);
}

// The order in which a workgroup goes through its tiles: each starts elsewhere in its share.  All of them move at one pace, and
// where shares begin at multiples of a power of two (8 heads of 65536, 131072, 262144 keys) workgroups in step were slow to get
// keys that are not in the caches.  Stage, us, behind a kernel that has written 1 GiB, on five machines, all from their first
// tile on / each from another: 65536 keys 91 .. 109 / 90 .. 97, 131072 163 .. 188 / 160 .. 172, 262144 282 .. 337 / 291 .. 304,
// 66000 112 .. 115 / 99 .. 100; with the keys in the caches 131072 takes 125.9 / 125.7, 262144 272 / 266, 66000 82.5 / 83.2.
// Sweep 1 walks a range from the tile on that only the range's place in its head decides, so that a row's sums, which a range
// adds up, do not depend on the other heads of a call (and from its first tile on where a call of fewer heads takes the short
// form, with ranges of the same length); it takes the ranges of its share in turn from any one on.  Sweep 2 walks its whole
// share from any tile on.  Tiles go in groups of four, as the loops do: the groups in turn and the tiles of a group in turn.
// A range, and a share of sweep 2, that is not full keeps its order.  Past the end both go on behind the last key.
__device__ __forceinline__ uint32_t spread32(uint32_t i) { return i * 0x9E3779B1u; }       // 2^32 / golden ratio

// a place in 0 .. count - 1 for this workgroup
__device__ __forceinline__ int own_place(int count)
{
    return (int)((spread32(blockIdx.y * gridDim.x + blockIdx.x) >> 16) * (uint32_t)count >> 16);
}

struct RangeWalk {
    int tiles;             // of a range, a power of two
    int ranges, turned;    // of the share; those that do not start with their first tile
    int first, place;      // the range it starts with; number in its head of the share's range 0
    int begun;             // ranges begun
    int base, at, left;    // range's first tile, group's first tile in it, groups of it that are left
    int in[4];             // tile of a group at each step

    // the share's keys from range first_range of a head of n keys on
    __device__ __forceinline__ RangeWalk(int first_range, int keys, int range_keys, int n)
    {
        const int full = keys >> (31 - __builtin_clz(range_keys));
        tiles = range_keys / kTileKeys;
        // 2048 keys in ranges of 1024: at least 349525 keys in all, so that no call with such heads takes the short form
        static_assert(kLongKeys <= kSweepWgs * (long long)kMaxRangeKeys * 2 / 3, "3 ranges at most for each 2 that are full");
        turned = range_keys == kMaxRangeKeys && n >= 2 * kMaxRangeKeys ? full : 0;
        ranges = (keys & (range_keys - 1)) == 0 ? full : full + 1;
        first = full == ranges ? own_place(ranges) : 0;
        place = first_range;
        begun = 0;
        open();
    }
    // the range that is the k-th to be taken
    __device__ __forceinline__ int range(int k) const { return k + first >= ranges && k < ranges ? k + first - ranges : k + first; }
    __device__ __forceinline__ void open()
    {
        const int r = range(begun), phase = r < turned ? (int)(spread32(place + r) >> 27) : 0;       // 0 .. 31
        static_assert(kMaxRangeKeys / kTileKeys == 32, "a phase is a tile of a range");
        base = r * tiles;
        at = phase & ~3;
        left = tiles / 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) in[i] = (i + phase) & 3;
        ++begun;
    }
    __device__ __forceinline__ void next_group()
    {
        at = (at + 4) & (tiles - 1);
        if (__builtin_expect(--left == 0, 0)) open();
    }
    __device__ __forceinline__ int tile(int i) const { return base + at + in[i]; }
};

struct ShareWalk {
    int groups, group, left, in[4];

    __device__ __forceinline__ explicit ShareWalk(int keys)
    {
        const bool full = keys % (4 * kTileKeys) == 0;
        groups = (keys + 4 * kTileKeys - 1) / (4 * kTileKeys);
        group = full ? own_place(groups) : 0;
        left = groups;
#pragma unroll
        for (int i = 0; i < 4; ++i) in[i] = (i + (full ? (int)blockIdx.x : 0)) & 3;
    }
    __device__ __forceinline__ void next_group()
    {
        group = group + 1 == groups ? 0 : group + 1;
        if (--left == 0) group = groups;
    }
    __device__ __forceinline__ int tile(int i) const { return 4 * group + in[i]; }
};

// Feature step x: lane (key = lane & 31, h = lane >> 5) holds d = 16 x + 8 h .. + 8 of its key.
__device__ __forceinline__ bf16x8 k_fragment(const KTile &tile, const KSource &src, int x)
{
    return *reinterpret_cast<const bf16x8 *>(tile.b + src.kfr[x]);
}

// The wave's 64 rows of the split Qhat: qf[rt][x][term], row 64 wave + 32 rt + (lane & 31), the features of k_fragment.
__device__ __forceinline__ void load_qfrags(bf16x8 (&qf)[2][8][2], const bf16_t *qsplit, int bh, int wave, int lane)
{
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int x = 0; x < 8; ++x)
#pragma unroll
            for (int term = 0; term < 2; ++term)
                qf[rt][x][term] = *reinterpret_cast<const bf16x8 *>(qsplit + qfrag_offset(bh, 2 * wave + rt, x, term) + lane * 8);
}

// More wait states than a matrix result needs before a vector instruction reads it; no read of s moves up across
__device__ __forceinline__ void mfma_fence(floatx16 &s) { asm volatile("s_nop 15\n\ts_nop 15" : "+v"(s)::"memory"); }

// Logit MFMA m of the 32 of a tile, a chain of sixteen for each row tile.  KEYS_BY_ROWS: s[rt][i] belongs to key
// 8 (i / 4) + 4 h + i % 4 and row 32 rt + (lane & 31), and starts at 0; otherwise to key lane & 31 and that row, and starts at
// c[rt].  Assembly statements: the compiler's own would move accumulators about.  It does not see inside, so the one hazard
// (results read by vector instructions) is covered by distance, or by mfma_fence().
template <int M, bool KEYS_BY_ROWS>
__device__ __forceinline__ void logit_mfma(floatx16 (&s)[2], const bf16x8 (&kf)[8], const bf16x8 (&qf)[2][8][2],
                                           const floatx16 (&c)[2])
{
    constexpr int rt = M >> 4, x = (M >> 1) & 7, term = M & 1;
    const bf16x8 &k = kf[x], &q = qf[rt][x][term];
    if constexpr (KEYS_BY_ROWS) {
        if constexpr ((M & 15) == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s[rt]) : "v"(k), "a"(q));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s[rt]) : "v"(k), "a"(q));
    } else {
        if constexpr ((M & 15) == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(s[rt]) : "a"(q), "v"(k), "v"(c[rt]));
        else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s[rt]) : "a"(q), "v"(k));
    }
}

// f(0), f(1), .. with compile-time arguments
template <typename F, int... M>
__device__ __forceinline__ void unrolled(F &&f, std::integer_sequence<int, M...>)
{
    (f(std::integral_constant<int, M>{}), ...);
}

// One iteration: logits of tile t + 1 into s_nxt; score(m) does the vector work under MFMA m.  tile1: LDS tile of t + 1, which
// tile t + 5 takes, number `later` of the share; tile2: of t + 2.
template <bool KEYS_BY_ROWS, typename Score>
__device__ __forceinline__ void sweep_step(floatx16 (&s_nxt)[2], bf16x8 (&kf)[8], const bf16x8 (&qf)[2][8][2],
                                           const floatx16 (&c)[2], KTile &tile1, const KTile &tile2, const KSource &src,
                                           int later, int wave, Score score)
{
    __builtin_amdgcn_sched_barrier(0);
    unrolled([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        logit_mfma<m, KEYS_BY_ROWS>(s_nxt, kf, qf, c);
        __builtin_amdgcn_sched_barrier(0);                 // what goes out under an MFMA follows it
        if constexpr (m == 0) kf[7] = k_fragment(tile1, src, 7);
        if constexpr (m >= 18 && m % 2 == 0) kf[(m - 18) / 2] = k_fragment(tile2, src, (m - 18) / 2);
        score(mc);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (m == 8) {
            // this wave's reads of tile1 are done and its loads of tile t + 2 have landed (those of the two tiles behind may be
            // on their way); after the barrier that is so for the other wave as well
            __builtin_amdgcn_s_waitcnt(0x0078);            // vmcnt(8) lgkmcnt(0), gfx9 encoding
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            issue_tile(tile1, src, later, wave);
        }
    }, std::make_integer_sequence<int, 32>{});
}

// Everything ahead of the loop: four tiles on their way, Qhat in registers, the logits of tile 0 in s.
template <bool KEYS_BY_ROWS, typename Walk>
__device__ __forceinline__ void sweep_start(floatx16 (&s)[2], bf16x8 (&kf)[8], bf16x8 (&qf)[2][8][2], const floatx16 (&c)[2],
                                            KTile &t0, KTile &t1, KTile &t2, KTile &t3, const KSource &src,
                                            Walk &walk, const bf16_t *qsplit, int bh, int wave, int lane)
{
    issue_tile(t0, src, walk.tile(0), wave);
    issue_tile(t1, src, walk.tile(1), wave);
    issue_tile(t2, src, walk.tile(2), wave);
    issue_tile(t3, src, walk.tile(3), wave);
    walk.next_group();
    load_qfrags(qf, qsplit, bh, wave, lane);
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0), gfx9 encoding
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 8; ++x) kf[x] = k_fragment(t0, src, x);
    unrolled([&](auto mc) __attribute__((always_inline)) { logit_mfma<decltype(mc)::value, KEYS_BY_ROWS>(s, kf, qf, c); },
             std::make_integer_sequence<int, 32>{});
    mfma_fence(s[0]);
    mfma_fence(s[1]);
#pragma unroll
    for (int x = 0; x < 7; ++x) kf[x] = k_fragment(t1, src, x);
    __syncthreads();                                       // both waves have read tile 0
    issue_tile(t0, src, walk.tile(0), wave);
}

// ------------------------------------------------------------------ MFMA path: sweep 1
// partial[bh][range][row] = (max2, sumexp2) over the keys of a range, log2 domain; a workgroup takes `ranges` of them.
// The maximum of a row tile is known before its first exponential: that of row tile 1 is formed under the exponentials of row
// tile 0, that of row tile 0 under those of row tile 1 of the tile before.
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(1, 1))) void scores_sweep1_kernel(
    const bf16_t *__restrict__ K, const bf16_t *__restrict__ qsplit, float2 *__restrict__ partial, Geo g, int range_keys,
    int ranges)
{
    __shared__ KTile tile0, tile1, tile2, tile3;
    const int bh = blockIdx.y, parts = ceil_div(g.n, range_keys);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first_range = blockIdx.x * ranges;
    const int key_begin = first_range * range_keys, keys = min(g.n - key_begin, range_keys * ranges);
    const int ntiles = ceil_div(keys, kTileKeys), range_tiles = range_keys / kTileKeys;
    const KSource src = key_source(K + ((size_t)bh * g.n + key_begin) * 128, keys, lane);
    RangeWalk walk(first_range, keys, range_keys, g.n);         // tiles to load
    bf16x8 qf[2][8][2], kf[8];
    floatx16 sa[2], sb[2];
    sweep_start<true>(sa, kf, qf, sa, tile0, tile1, tile2, tile3, src, walk, qsplit, bh, wave, lane);
    float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.0f, 0.0f};   // row 32 rt + (lane & 31), this lane's half of the keys
    // keys of tile t that do not exist weigh nothing
    auto cut = [&](floatx16 &s, int t) __attribute__((always_inline)) {
        if (__builtin_expect((t + 1) * kTileKeys > keys, 0)) {
            mfma_fence(s);
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (t * kTileKeys + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3) >= keys) s[i] = -INFINITY;
        }
    };
    float top0;                                            // maximum of the current tile's row tile 0
    cut(sa[0], 0);
    top0 = sa[0][0];
#pragma unroll
    for (int i = 1; i < 16; ++i) top0 = fmaxf(top0, sa[0][i]);
    auto step = [&](floatx16 (&s)[2], floatx16 (&nxt)[2], KTile &u1, const KTile &u2, int t, int later) __attribute__((always_inline)) {
        cut(s[1], t);
        float p[2], sum[2], mn[2], less[2], top1 = -INFINITY;
        // arguments are <= 0: the bare instruction (no denormal rescue) loses nothing that a sum near 1 would see
        auto add = [&](auto uc) __attribute__((always_inline)) {         // logit u joins its row tile's sum
            constexpr int u = decltype(uc)::value, rt = u >> 4;
            if constexpr ((u & 15) == 0) sum[rt] = p[u & 1];
            else sum[rt] += p[u & 1];
            if constexpr ((u & 15) != 0) asm volatile("" : "+v"(sum[rt]));
            if constexpr ((u & 15) == 15) {
                const float joined = l[rt] * __builtin_amdgcn_exp2f(m[rt] - mn[rt]) + sum[rt];   // exp2(-inf) = 0 on the first tile
                l[rt] = mn[rt] != -INFINITY ? joined : l[rt];
                m[rt] = mn[rt];
            }
        };
        sweep_step<true>(nxt, kf, qf, nxt, u1, u2, src, later, wave, [&](auto mc) __attribute__((always_inline)) {
            constexpr int mm = decltype(mc)::value, rt = mm >> 4, i = mm & 15;
            if constexpr (i == 0) {
                mn[rt] = fmaxf(m[rt], rt == 0 ? top0 : top1);
                less[rt] = mn[rt] == -INFINITY ? 0.0f : mn[rt];
            }
            const float x = s[rt][i] - less[rt];
            if constexpr (mm > 0) add(std::integral_constant<int, mm - 1>{});
            p[mm & 1] = __builtin_amdgcn_exp2f(x);
            // the other row tile's maximum, two logits at a time
            if constexpr (rt == 0 && i >= 4 && i < 12) {
                constexpr int z = 2 * (i - 4);
                asm volatile("v_max3_f32 %0, %1, %2, %0" : "+v"(top1) : "v"(s[1][z]), "v"(s[1][z + 1]));
            }
            if constexpr (mm == 21) cut(nxt[0], t + 1);
            if constexpr (rt == 1 && i >= 6 && i < 14) {
                constexpr int z = 2 * (i - 6);
                if constexpr (z == 0) top0 = -INFINITY;
                asm volatile("v_max3_f32 %0, %1, %2, %0" : "+v"(top0) : "v"(nxt[0][z]), "v"(nxt[0][z + 1]));
            }
        });
        add(std::integral_constant<int, 31>{});
    };
    int done = 0;                                          // ranges
    for (int t = 0; t < ntiles; t += 4) {                  // (tiles past the last one hold no keys)
        step(sa, sb, tile1, tile2, t, walk.tile(1));
        step(sb, sa, tile2, tile3, t + 1, walk.tile(2));
        step(sa, sb, tile3, tile0, t + 2, walk.tile(3));
        walk.next_group();
        step(sb, sa, tile0, tile1, t + 3, walk.tile(0));
        if ((t + 4) % range_tiles == 0 || t + 4 >= ntiles) {         // the end of a range
            const int range = first_range + walk.range(done++);
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {               // merge the two lane halves; the rows of a wave are its own
                const float mo = __shfl_xor(m[rt], 32, 64), lo = __shfl_xor(l[rt], 32, 64);
                const float mn = fmaxf(m[rt], mo);
                float ln = 0.0f;
                if (mn != -INFINITY) ln = l[rt] * exp2f(m[rt] - mn) + lo * exp2f(mo - mn);
                if (lane < 32) partial[((size_t)bh * parts + range) * kQRows + 64 * wave + 32 * rt + lane] = make_float2(mn, ln);
                m[rt] = -INFINITY;
                l[rt] = 0.0f;
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // the loads issued past the end have landed
}

// c[bh][row] = -max - log2(bl * sumexp) for row < bl, -inf for the padding rows.
// 1024 threads: thread (grp, row) folds the partials grp, grp+8, ... of its row, then the 8 groups meet in LDS.
__global__ __launch_bounds__(1024) void scores_merge_kernel(const float2 *__restrict__ partial,
                                                            float *__restrict__ cvec, int nwg, int bl)
{
    __shared__ float2 red[8][kQRows];
    const int bh = blockIdx.x, row = threadIdx.x & (kQRows - 1), grp = threadIdx.x >> 7;
    float mn = -INFINITY, ln = 0.0f;
    for (int w0 = grp; w0 < nwg; w0 += 32) {                 // four independent loads per round trip
        float2 pr[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int w = w0 + 8 * q;
            pr[q] = w < nwg ? partial[((size_t)bh * nwg + w) * kQRows + row] : make_float2(-INFINITY, 0.0f);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (pr[q].x != -INFINITY) {
                const float m2 = fmaxf(mn, pr[q].x);
                ln = ln * exp2f(mn - m2) + pr[q].y * exp2f(pr[q].x - m2);
                mn = m2;
            }
    }
    red[grp][row] = make_float2(mn, ln);
    __syncthreads();
    if (grp == 0) {
        float m2 = -INFINITY;
        for (int q = 0; q < 8; ++q) m2 = fmaxf(m2, red[q][row].x);
        float l2 = 0.0f;
        for (int q = 0; q < 8; ++q)
            if (red[q][row].x != -INFINITY) l2 += red[q][row].y * exp2f(red[q][row].x - m2);
        cvec[(size_t)bh * kQRows + row] = row < bl ? -m2 - log2f((float)bl * l2) : -INFINITY;
    }
}

// ------------------------------------------------------------------ MFMA path: sweep 2
// scores[key] = sum over the 128 rows of exp2(logit2 + c[row]): each wave sums its 64 rows per key; what the lane halves and
// the waves have of a tile's keys is put together under the next tile.
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(1, 1))) void scores_sweep2_kernel(
    const bf16_t *__restrict__ K, const bf16_t *__restrict__ qsplit, const float *__restrict__ cvec,
    float *__restrict__ scores, Geo g, int kpw)
{
    __shared__ KTile tile0, tile1, tile2, tile3;
    __shared__ float psum[4][2][kTileKeys];                  // of the last tiles, by wave
    const int bh = blockIdx.y;
    const int wg = gridDim.x - 1 - blockIdx.x;               // reverse order: reuse what sweep 1 left in cache
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int key_begin = wg * kpw, keys = min(g.n - key_begin, kpw), ntiles = ceil_div(keys, kTileKeys);
    const KSource src = key_source(K + ((size_t)bh * g.n + key_begin) * 128, keys, lane);
    ShareWalk walk(keys);                                    // tiles to load
    float *out = scores + (size_t)bh * g.n + key_begin;
    bf16x8 qf[2][8][2], kf[8];
    // the accumulators start at c[row]; row = 64 wave + 32 rt + 8 (i / 4) + 4 (lane >> 5) + (i % 4)
    floatx16 sa[2], sb[2], c[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            c[rt][i] = cvec[(size_t)bh * kQRows + 64 * wave + 32 * rt + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3)];
    const int group0 = walk.group;
    sweep_start<false>(sa, kf, qf, c, tile0, tile1, tile2, tile3, src, walk, qsplit, bh, wave, lane);
    float done[2] = {0.0f, 0.0f};                            // this lane's sums of the tile before
    auto halves = [&](int rt) __attribute__((always_inline)) {
        const uint32_t own = __builtin_bit_cast(uint32_t, done[rt]);
        const auto sw = __builtin_amdgcn_permlane32_swap(own, own, false, false);
        const uint32_t lower = sw[0], upper = sw[1];
        done[rt] = __builtin_bit_cast(float, lower) + __builtin_bit_cast(float, upper);
    };
    // 16 keys of the tile before for each wave (behind a barrier that psum of both waves is ahead of)
    const int mine = 16 * wave + (lane & 15);
    auto leave = [&](int t, int number) __attribute__((always_inline)) {
        const int at = number * kTileKeys + mine;
        if (lane < 16 && at >= 0 && at < keys) out[at] = psum[t & 3][0][mine] + psum[t & 3][1][mine];
    };
    auto step = [&](floatx16 (&s)[2], floatx16 (&nxt)[2], KTile &u1, const KTile &u2, int t, int before, int later)
                    __attribute__((always_inline)) {
        float p[2], sum[2];
        auto add = [&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value, rt = u >> 4;
            if constexpr ((u & 15) == 0) sum[rt] = p[u & 1];
            else sum[rt] += p[u & 1];
            if constexpr ((u & 15) != 0) asm volatile("" : "+v"(sum[rt]));
        };
        sweep_step<false>(nxt, kf, qf, c, u1, u2, src, later, wave, [&](auto mc) __attribute__((always_inline)) {
            constexpr int mm = decltype(mc)::value;
            if constexpr (mm > 0) add(std::integral_constant<int, mm - 1>{});
            p[mm & 1] = __builtin_amdgcn_exp2f(s[mm >> 4][mm & 15]);
            if constexpr (mm == 1) halves(0);
            if constexpr (mm == 2) halves(1);
            if constexpr (mm == 3) psum[(t - 1) & 3][wave][lane & 31] = done[0] + done[1];     // the same from both halves
            if constexpr (mm == 12) leave(t - 1, before);
        });
        add(std::integral_constant<int, 31>{});
        done[0] = sum[0];
        done[1] = sum[1];
    };
    int t = 0, before = -1;                                  // number of tile t - 1
    int own = 4 * group0;                                    // first tile of its group
    for (; t < ntiles; t += 4) {                             // (tiles past the last one hold no keys)
        const int later = 4 * walk.group;
        step(sa, sb, tile1, tile2, t, before, walk.tile(1));
        step(sb, sa, tile2, tile3, t + 1, own + walk.in[0], walk.tile(2));
        step(sa, sb, tile3, tile0, t + 2, own + walk.in[1], walk.tile(3));
        walk.next_group();
        step(sb, sa, tile0, tile1, t + 3, own + walk.in[2], walk.tile(0));
        before = own + walk.in[3];
        own = later;
    }
    halves(0);
    halves(1);
    psum[(t - 1) & 3][wave][lane & 31] = done[0] + done[1];
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // the loads issued past the end have landed
    __syncthreads();
    leave(t - 1, before);
}

// ------------------------------------------------------------------ MFMA path, short inputs
// Where there are too few keys for every SIMD to have a wave of 64 rows: four waves to a workgroup, 32 rows each, two to
// a SIMD.  The logits, their maxima and their sums are formed in the same order as above.
namespace short_input {

// Wave w of a workgroup owns the logit rows 32 w .. 32 w + 31 and keeps their split Qhat fragments in registers
// (8 k-steps x 2 terms x 4 registers); the K tiles of 32 keys go through LDS, where all four waves read them, so a
// fragment read feeds two MFMAs and the tile is fetched from memory once.  A tile travels global -> registers ->
// LDS; kTilesAhead tiles per workgroup are in flight in registers, and two LDS copies alternate so that one
// barrier per tile suffices.
constexpr int kTileKeys = 32;
constexpr int kTilesAhead = 2;

// 32 keys x 256 bytes; the 16-byte piece c of row r sits at r * 256 + ((c ^ (r & 15)) << 4): conflict-free for the
// stores (16 lanes = the 16 pieces of a row) and for the fragment reads (16 lanes = 16 rows, one piece each).
struct KTile {
    unsigned char b[kTileKeys * 256];
};

// Thread tid moves pieces tid and tid + 256 of the 512 pieces of a tile (row = piece / 16, c = piece % 16).
__device__ inline void ktile_fetch(uintx4 (&v)[2], const bf16_t *Kh, int key0, int n, int tid)
{
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int piece = tid + 256 * u;
        int key = key0 + (piece >> 4);
        if (key >= n) key = n - 1;                            // clamped; masked by the caller
        v[u] = *reinterpret_cast<const uintx4 *>(Kh + (size_t)key * 128 + (piece & 15) * 8);
    }
}

__device__ inline void ktile_store(KTile &t, const uintx4 (&v)[2], int tid)
{
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int piece = tid + 256 * u;
        const int row = piece >> 4, c = piece & 15;
        *reinterpret_cast<uintx4 *>(t.b + row * 256 + ((c ^ (row & 15)) << 4)) = v[u];
    }
}

// MFMA operand of k-step ks: lane (key = lane & 31, h = lane >> 5) holds d = 16 ks + 8 h .. + 8 of its key.
__device__ inline bf16x8 kfrag(const KTile &t, int ks, int lane)
{
    const int row = lane & 31, c = 2 * ks + (lane >> 5);
    return *reinterpret_cast<const bf16x8 *>(t.b + row * 256 + ((c ^ (row & 15)) << 4));
}

// The wave's 32 rows of one term of the split Qhat (same d range per lane as kfrag).
__device__ inline void load_qfrags(bf16x8 (&qf)[8], const bf16_t *qsplit, int bh, int term, int wave, int lane)
{
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(qsplit + qfrag_offset(bh, wave, ks, term) + lane * 8);
}

// Runs body(t, tile) for the tiles t = 0 .. ntiles - 1 of the keys from key_begin on, the tile being complete in
// LDS.  The loops over the tiles in flight are fully unrolled, so their register copies have compile-time indices.
template <typename Body>
__device__ __forceinline__ void sweep_tiles(KTile (&kt)[2], const bf16_t *Kh, int key_begin, int ntiles, int n, int tid,
                                            Body body)
{
    uintx4 pre[kTilesAhead][2];
#pragma unroll
    for (int a = 0; a < kTilesAhead; ++a) ktile_fetch(pre[a], Kh, min(key_begin + a * kTileKeys, n - 1), n, tid);
    ktile_store(kt[0], pre[0], tid);
    ktile_fetch(pre[0], Kh, min(key_begin + kTilesAhead * kTileKeys, n - 1), n, tid);
    __syncthreads();
    for (int t0 = 0; t0 < ntiles; t0 += kTilesAhead) {
#pragma unroll
        for (int a = 0; a < kTilesAhead; ++a) {
            const int t = t0 + a;
            if (t < ntiles) {                                  // uniform
                // tile t + 1 leaves its registers for the LDS copy that tile t - 1 used, and its registers take
                // tile t + 1 + kTilesAhead (reads past the range are clamped to the last key and never used)
                ktile_store(kt[(a + 1) & 1], pre[(a + 1) % kTilesAhead], tid);
                ktile_fetch(pre[(a + 1) % kTilesAhead], Kh, min(key_begin + (t + 1 + kTilesAhead) * kTileKeys, n - 1),
                            n, tid);
                body(t, kt[a & 1]);
                __syncthreads();                               // tile t consumed, tile t + 1 visible
            }
        }
    }
}

// partial[bh][range][row] = (max2, sumexp2) over the keys of a range, log2 domain; a workgroup takes kpw keys, a whole number of
// ranges of range_keys (a multiple of a tile).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void sweep1_kernel(
    const bf16_t *__restrict__ K, const bf16_t *__restrict__ qsplit, float2 *__restrict__ partial, Geo g, int kpw, int range_keys)
{
    __shared__ __align__(16) KTile kt[2];
    const int bh = blockIdx.y, wg = blockIdx.x, parts = ceil_div(g.n, range_keys);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    bf16x8 qh[8], ql[8];
    load_qfrags(qh, qsplit, bh, 0, wave, lane);
    load_qfrags(ql, qsplit, bh, 1, wave, lane);
    const bf16_t *Kh = K + (size_t)bh * g.n * 128;
    const int key_begin = wg * kpw, key_end = min(g.n, key_begin + kpw);
    const int ntiles = ceil_div(key_end - key_begin, kTileKeys);
    float2 *first = partial + ((size_t)bh * parts + key_begin / range_keys) * kQRows + wave * 32 + lane;
    float m = -INFINITY, l = 0.0f;                           // row 32 wave + (lane & 31), this lane's half of the keys
    sweep_tiles(kt, Kh, key_begin, ntiles, g.n, tid, [&](int t, const KTile &tile) {
        floatx16 acc = {0};
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 kf = kfrag(tile, ks, lane);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qh[ks], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, ql[ks], acc, 0, 0, 0);
        }
        // acc[i]: key = key0 + 8 (i / 4) + 4 (lane >> 5) + (i % 4), query row = 32 wave + (lane & 31)
        const int key0 = key_begin + t * kTileKeys;
        if (key0 + kTileKeys > g.n) {                          // the ragged last tile of the sequence
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (key0 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3) >= g.n) acc[i] = -INFINITY;
        }
        float tmax = acc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, acc[i]);
        const float mn = fmaxf(m, tmax);
        if (mn != -INFINITY) {
            // arguments are <= 0: the bare instruction (no denormal rescue) loses nothing that a sum near 1 would see
            float sum = 0.0f;
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(acc[i] - mn);
            l = l * __builtin_amdgcn_exp2f(m - mn) + sum;    // exp2(-inf) = 0 on the first tile
            m = mn;
        }
        if (((t + 1) * kTileKeys & (range_keys - 1)) != 0 && t + 1 < ntiles) return;
        // the end of a range: merge the two lane halves; the rows of a wave are its own.  (Without LDS and without a rescue of
        // denormals, which next to the half that holds the maximum count for nothing: a range may end every other tile.)
        const uint32_t mb = __builtin_bit_cast(uint32_t, m), lb = __builtin_bit_cast(uint32_t, l);
        const auto ms = __builtin_amdgcn_permlane32_swap(mb, mb, false, false), ls = __builtin_amdgcn_permlane32_swap(lb, lb, false, false);
        const uint32_t ml = ms[0], mh = ms[1], ll = ls[0], lh = ls[1];       // of the lower and of the upper half
        const float m0 = __builtin_bit_cast(float, ml), m1 = __builtin_bit_cast(float, mh), both = fmaxf(m0, m1);
        float ln = 0.0f;
        if (both != -INFINITY)
            ln = __builtin_bit_cast(float, ll) * __builtin_amdgcn_exp2f(m0 - both) + __builtin_bit_cast(float, lh) * __builtin_amdgcn_exp2f(m1 - both);
        if (lane < 32) first[(size_t)(t * kTileKeys / range_keys) * kQRows] = make_float2(both, ln);
        m = -INFINITY;
        l = 0.0f;
    });
}

// scores[key] = sum over the 128 rows of exp2(logit2 + c[row]): each wave sums its 32 rows per key into LDS, the
// four partial sums of a key meet once at the end of the workgroup's range.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void sweep2_kernel(
    const bf16_t *__restrict__ K, const bf16_t *__restrict__ qsplit, const float *__restrict__ cvec,
    float *__restrict__ scores, Geo g, int kpw)
{
    __shared__ __align__(16) KTile kt[2];
    __shared__ float psum[4][kMaxRangeKeys];
    const int bh = blockIdx.y;
    const int wg = gridDim.x - 1 - blockIdx.x;               // reverse order: reuse what sweep 1 left in cache
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    bf16x8 qh[8], ql[8];
    load_qfrags(qh, qsplit, bh, 0, wave, lane);
    load_qfrags(ql, qsplit, bh, 1, wave, lane);
    // the accumulator starts at c[row]; row = 32 wave + 8 (i / 4) + 4 (lane >> 5) + (i % 4)
    floatx16 cinit;
#pragma unroll
    for (int i = 0; i < 16; ++i)
        cinit[i] = cvec[(size_t)bh * kQRows + 32 * wave + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3)];
    const bf16_t *Kh = K + (size_t)bh * g.n * 128;
    const int key_begin = wg * kpw, key_end = min(g.n, key_begin + kpw);
    const int ntiles = ceil_div(key_end - key_begin, kTileKeys);
    sweep_tiles(kt, Kh, key_begin, ntiles, g.n, tid, [&](int t, const KTile &tile) {
        floatx16 acc = cinit;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 kf = kfrag(tile, ks, lane);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qh[ks], kf, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ql[ks], kf, acc, 0, 0, 0);
        }
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(acc[i]);
        sum += __shfl_xor(sum, 32, 64);
        if (lane < 32) psum[wave][t * kTileKeys + lane] = sum;      // key = key_begin + 32 t + lane
    });
    // the loop's last barrier has made every partial sum visible
    for (int k = tid; k < key_end - key_begin; k += 256)
        scores[(size_t)bh * g.n + key_begin + k] = (psum[0][k] + psum[1][k]) + (psum[2][k] + psum[3][k]);
}

}  // namespace short_input

// ------------------------------------------------------------------ generic path (fp64 accumulation)
// one thread per element of Qhat; grid = (ceil(bl * d / 256), batch * h_kv)
template <typename E>
__global__ __launch_bounds__(256) void qhat_f64_kernel(const E *__restrict__ Q, double *__restrict__ qhat, Geo g,
                                                       int bl, const int32_t *__restrict__ qrows,
                                                       const double *__restrict__ qavg)
{
    const int bh = blockIdx.y;
    const int b = bh / g.h_kv, h = bh % g.h_kv;
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= bl * g.d) return;
    const int row = idx / g.d, e = idx % g.d;
    if (qavg) {
        qhat[(size_t)bh * bl * g.d + idx] = qavg[(size_t)bh * 128 + e];
        return;
    }
    const int pos = query_row_position(qrows, row, bl, g.n);
    double acc = 0.0;
    for (int t = 0; t < g.r; ++t)
        acc += (double)ElemTraits<E>::to_float(Q[(((size_t)b * g.h_q + h * g.r + t) * g.n + pos) * g.d + e]);
    qhat[(size_t)bh * bl * g.d + idx] = acc / (double)g.r;
}

// ------------------------------------------------------------------ the average query (one proxy of the ablations)
// partial[bh][chunk][e] = fp64 sum over the chunk's positions and the group's r heads of Q[.., pos, e];
// grid = (kAvgChunks, nbh), 256 threads: thread (e = tid % d, slot = tid / d) walks the positions slot, slot + 256/d, ..
constexpr int kAvgChunks = 128;

template <typename E>
__global__ __launch_bounds__(256) void qavg_partial_kernel(const E *__restrict__ Q, double *__restrict__ partial, Geo g)
{
    __shared__ double red[256];
    const int bh = blockIdx.y, chunk = blockIdx.x;
    const int b = bh / g.h_kv, h = bh % g.h_kv;
    const int per = ceil_div(g.n, kAvgChunks);
    const int lo = chunk * per, hi = min(g.n, lo + per);
    const int e = threadIdx.x % g.d, slot = threadIdx.x / g.d, slots = 256 / g.d;
    double acc = 0.0;
    for (int t = 0; t < g.r; ++t) {
        const E *Qh = Q + ((size_t)b * g.h_q + h * g.r + t) * (size_t)g.n * g.d;
        for (int pos = lo + slot; pos < hi; pos += slots) acc += (double)ElemTraits<E>::to_float(Qh[(size_t)pos * g.d + e]);
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    if ((int)threadIdx.x < g.d) {
        double s = 0.0;
        for (int q = 0; q < slots; ++q) s += red[q * g.d + threadIdx.x];
        partial[((size_t)bh * kAvgChunks + chunk) * 128 + threadIdx.x] = s;
    }
}

// qavg[bh][e] = (sum of the partials) / (r * n)
__global__ __launch_bounds__(128) void qavg_final_kernel(const double *__restrict__ partial, double *__restrict__ qavg,
                                                         Geo g)
{
    const int bh = blockIdx.x, e = threadIdx.x;
    if (e >= g.d) return;
    double s = 0.0;
    for (int c = 0; c < kAvgChunks; ++c) s += partial[((size_t)bh * kAvgChunks + c) * 128 + e];
    qavg[(size_t)bh * 128 + e] = s / ((double)g.r * (double)g.n);
}

// Both sweeps form 16 keys x 16 query rows of logits at a time on the fp64 matrix instruction (v_mfma_f64_16x16x4:
// the arithmetic of fp64 fused multiply-adds).  A operand: lane (key = lane % 16, grp = lane / 16) holds
// K[key][16 u + 4 grp + c] of step (u, c), a 16-byte load for float; B operand: the same features of query row
// lane % 16, kept in registers; accumulator: keys grp + 4 x (x = 0..3) of query row lane % 16.  So a lane owns a query row
// (its statistics are per lane) and what a wave needs of K comes straight from memory, without LDS.
// The four waves of a workgroup divide the 16-row tiles of Qhat among them (at most two each) and, where there are
// fewer than three, the key tiles as well.
// Bound: the exponentials (one fp64 exp per logit and sweep, about 30 fp64 instructions) and the latency of a few short
// launches.  Measured, stage: float32, 2 heads x 2048 keys x 64 12.4 us, bf16 d = 64, 4 kv heads x 12301 keys 46 us (541 and 757 us with
// one thread per key, or per key and row, walking its K row alone).
struct WaveShare {
    int rw, kg;                        // waves that share the rows, waves that share the keys; rw * kg = 4
};
__host__ __device__ inline WaveShare wave_share(int bl)
{
    const int tiles = ceil_div(bl, 16);
    return tiles > 2 ? WaveShare{4, 1} : (tiles == 2 ? WaveShare{2, 2} : WaveShare{1, 4});
}

template <typename E, int D>
struct F64Logits {
    double q[2][D / 4];                // query rows 16 (wr + rw t) + lane % 16, t = 0, 1
    int row[2];                        // those rows' indices
    int tiles;                         // row tiles of this wave

    // qhat: what qhat_f64_kernel has left, or NULL: formed here from Q in the same way, for one or two query heads, by which a
    // division is a multiplication
    __device__ __forceinline__ void load_rows(const double *qhat, const E *Q, const int32_t *qrows, const Geo &g, int bh, int bl,
                                              int wr, int rw, int lane)
    {
        tiles = wr * 16 >= bl ? 0 : ((wr + rw) * 16 >= bl ? 1 : 2);
        const int b = bh / g.h_kv, h = bh % g.h_kv;
        if (qhat) qhat += (size_t)bh * bl * D;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            row[t] = 16 * (wr + rw * t) + (lane & 15);
            if (!qhat) {
                if (t >= tiles) continue;
                const int pos = query_row_position(qrows, min(row[t], bl - 1), bl, g.n);
                const E *from = Q + (((size_t)b * g.h_q + h * g.r) * g.n + pos) * (size_t)D + 4 * (lane >> 4);
#pragma unroll
                for (int e = 0; e < D / 4; ++e) q[t][e] = 0.0;
#pragma unroll 1
                for (int head = 0; head < g.r; ++head) {
                    floatx4 v[D / 16];
#pragma unroll
                    for (int u = 0; u < D / 16; ++u) v[u] = load4(from + (size_t)head * g.n * D + 16 * u);
#pragma unroll
                    for (int e = 0; e < D / 4; ++e) q[t][e] += (double)v[e >> 2][e & 3];
                }
                const double mean = 1.0 / (double)g.r;
#pragma unroll
                for (int e = 0; e < D / 4; ++e) q[t][e] *= mean;
                continue;
            }
            const double *src = qhat + (size_t)min(row[t], bl - 1) * D + 4 * (lane >> 4);
            if (t < tiles)
#pragma unroll
                for (int e = 0; e < D / 4; ++e) q[t][e] = src[16 * (e >> 2) + (e & 3)];
        }
    }
    // logits of the 16 keys from key0 on (keys past n are clamped: the caller masks them) against row tile t
    __device__ __forceinline__ void load_keys(floatx4 (&k)[D / 16], const E *Kh, int key0, int n, int lane) const
    {
        const E *src = Kh + (size_t)min(key0 + (lane & 15), n - 1) * D + 4 * (lane >> 4);
#pragma unroll
        for (int u = 0; u < D / 16; ++u) k[u] = load4(src + 16 * u);
    }
    __device__ __forceinline__ doublex4 operator()(const floatx4 (&k)[D / 16], int t) const
    {
        doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < D / 4; ++e)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)k[e >> 2][e & 3], q[t][e], acc, 0, 0, 0);
        return acc;
    }
};

// Sweep 1.  grid = (ceil(chunks / per), nbh): (max, sum of exp) of every query row over a chunk of keys and one key share, for `per`
// chunks one after the other; partial[bh][row][part], part = chunk * kg + key share.
template <typename E, int D>
__global__ __launch_bounds__(256) void scores_stats_f64_kernel(const E *__restrict__ K,
                                                               const double *__restrict__ qhat, const E *__restrict__ Q,
                                                               const int32_t *__restrict__ qrows,
                                                               double2 *__restrict__ partial, Geo g, int bl,
                                                               int keys_per_chunk, int per)
{
    const int bh = blockIdx.y, chunks = ceil_div(g.n, keys_per_chunk);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const WaveShare ws = wave_share(bl);
    const int wr = wave % ws.rw, wk = wave / ws.rw;
    F64Logits<E, D> logits;
    logits.load_rows(qhat, Q, qrows, g, bh, bl, wr, ws.rw, lane);
    const E *Kh = K + (size_t)bh * g.n * D;
    const int parts = chunks * ws.kg;
    for (int chunk = blockIdx.x * per; chunk < min(chunks, ((int)blockIdx.x + 1) * per); ++chunk) {
        const int end = min(g.n, (chunk + 1) * keys_per_chunk);
        double m[2] = {-INFINITY, -INFINITY}, l[2] = {0.0, 0.0};
        for (int key0 = chunk * keys_per_chunk + 16 * wk; key0 < end; key0 += 16 * ws.kg) {
            floatx4 k[D / 16];
            logits.load_keys(k, Kh, key0, g.n, lane);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if (t >= logits.tiles) break;
                doublex4 v = logits(k, t);
                double top = -INFINITY;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    v[x] = key0 + (lane >> 4) + 4 * x < end ? v[x] * g.scale64 : -INFINITY;
                    top = fmax(top, v[x]);
                }
                if (__any(top > m[t])) {                       // rare after the first tiles
                    const double mn = fmax(m[t], top);
                    if (mn != -INFINITY) l[t] *= exp(m[t] - mn);
                    m[t] = mn;
                }
#pragma unroll
                for (int x = 0; x < 4; ++x)                    // (a logit that is not a number counts, whatever m is)
                    if (v[x] != -INFINITY) l[t] += exp(v[x] - m[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t >= logits.tiles) break;
            // the four lane groups hold different keys of the same row
#pragma unroll
            for (int o = 16; o < 64; o <<= 1) {
                const double mo = __shfl_xor(m[t], o, 64), lo = __shfl_xor(l[t], o, 64);
                const double mn = fmax(m[t], mo);
                l[t] = mn == -INFINITY ? l[t] + lo : l[t] * exp(m[t] - mn) + lo * exp(mo - mn);
                m[t] = mn;
            }
            if (lane < 16 && logits.row[t] < bl)
                partial[((size_t)bh * bl + logits.row[t]) * parts + chunk * ws.kg + wk] = make_double2(m[t], l[t]);
        }
    }
}

// One wave per row: stats[bh][row] = (max, 1 / sum of exp) over all parts.  grid = (ceil(bl / 4), nbh)
__global__ __launch_bounds__(256) void scores_merge_f64_kernel(const double2 *__restrict__ partial,
                                                               double2 *__restrict__ stats, int bl, int parts)
{
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), bh = blockIdx.y, lane = threadIdx.x & 63;
    if (row >= bl) return;
    const double2 *pr = partial + ((size_t)bh * bl + row) * parts;
    double mn = -INFINITY, ln = 0.0;
    for (int c = lane; c < parts; c += 64) {
        const double2 v = pr[c];
        const double m2 = fmax(mn, v.x);
        ln = m2 == -INFINITY ? ln + v.y : ln * exp(mn - m2) + v.y * exp(v.x - m2);
        mn = m2;
    }
    const double wm = wave_max(mn);
    const double wl = wave_sum(mn == -INFINITY ? ln : ln * exp(mn - wm));
    if (lane == 0) stats[(size_t)bh * bl + row] = make_double2(wm, 1.0 / wl);
}

// Sweep 2.  grid = (ceil(n / keys), nbh), keys <= kF64Keys: scores[key] = (1 / bl) sum_row exp(logit - max_row) / sum_row
constexpr int kF64Keys = 256;

template <typename E, int D>
__global__ __launch_bounds__(256) void scores_final_f64_kernel(const E *__restrict__ K,
                                                               const double *__restrict__ qhat, const E *__restrict__ Q,
                                                               const int32_t *__restrict__ qrows,
                                                               const double2 *__restrict__ stats,
                                                               float *__restrict__ scores, Geo g, int bl, int keys)
{
    __shared__ double psum[4][kF64Keys];
    const int bh = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const WaveShare ws = wave_share(bl);
    const int wr = wave % ws.rw, wk = wave / ws.rw;
    F64Logits<E, D> logits;
    logits.load_rows(qhat, Q, qrows, g, bh, bl, wr, ws.rw, lane);
    double mrow[2], inv[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const double2 st = stats[(size_t)bh * bl + min(logits.row[t], bl - 1)];
        mrow[t] = st.x;
        inv[t] = st.y;
    }
    const E *Kh = K + (size_t)bh * g.n * D;
    const int begin = blockIdx.x * keys, end = min(g.n, begin + keys);
    for (int key0 = begin + 16 * wk; key0 < end; key0 += 16 * ws.kg) {
        floatx4 k[D / 16];
        logits.load_keys(k, Kh, key0, g.n, lane);
        double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (t >= logits.tiles) break;
            const doublex4 v = logits(k, t);
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (logits.row[t] < bl) sum[x] += exp(v[x] * g.scale64 - mrow[t]) * inv[t];
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            sum[x] = row_sum_dpp(sum[x]);                  // over the 16 query rows of the lane group
            if ((lane & 15) == 0) psum[wr][key0 - begin + (lane >> 4) + 4 * x] = sum[x];
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < end - begin; j += 256) {
        double acc = psum[0][j];
        for (int w = 1; w < ws.rw; ++w) acc += psum[w][j];
        scores[(size_t)bh * g.n + begin + j] = (float)(acc / (double)bl);
    }
}

static bool use_mfma(const pbs_problem *p) { return p->dtype == PBS_BF16 && p->d == 128; }

// The generic path's workspace holds the statistics of one chunk per 4096 keys and the average-query region; the
// partial sums of that region are dead once Qhat is formed, so sweep 1 may use both.
constexpr int kGenericKeysPerChunk = 4096;
// Query heads of a kv head up to which both sweeps form Qhat from Q instead of reading what qhat_f64_kernel has left: a launch less,
// but every workgroup reads Q's last block once per head.  Stage, own launch / formed, us: one head, float32 2 x 2048 x 64 21.1 / 18.5,
// 2 x 4096 x 128 42.7 / 36.3, bf16 8 x 12288 x 64 104 / 97.7; two, float32 4/2 x 2048 x 64 21.2 / 19.5, x 128 42.7 / 39.6, bf16 4/2 x
// 4000 x 64 21.2 / 19.1; four, float32 8/2 x 2048 x 64 21.3 / 21.1, x 128 42.8 / 46.5, bf16 16/4 x 12301 x 64 46.0 / 50.0.
constexpr int kFormF64Heads = 2;

static size_t ws_avg_query(size_t nbh);

// Keys that a workgroup of either sweep takes at least (sweep 1: in chunks of their own): 64, and fewer where every workgroup has a
// compute unit then.  Stage, 64 keys / 32 / 16, us: float32 2 heads x 2048 x 64 18.6 / 13.7 / 12.7, 8/2 x 2048 x 128 42.6 / 30.2 /
// 27.0, 2 x 4096 x 128 36.3 / 30.4 / 31.7 (256 workgroups of 32), bf16 4/2 x 4000 x 64 19.2 / 15.1 / 15.3, 8 x 4000 x 64 (500 of 64)
// 41.0 / 42.3 / 45.5.  Every share of the keys gets a tile of 16 (few query rows: wave_share): without that, with 16 rows, float32
// 2 x 2048 x 64 14.3 / 12.5, x 128 16.1 / 13.9, bf16 4/2 x 2048 x 64 15.1 / 12.7 with 64 keys to a workgroup.
static int min_f64_keys(const Geo &g, int bl)
{
    const int least = 16 * wave_share(bl).kg;
    int keys = 64;
    while (keys > least && (long long)ceil_div(g.n, keys / 2) * g.batch * g.h_kv <= 256) keys >>= 1;
    return keys;
}

// Keys per chunk of sweep 1: as many chunks as the workspace has room for, of at least 16, 32 or 64 keys.  That is a matter of a head's
// length and the query rows alone, so that a head's sums do not depend on the other heads of a call; where a workgroup is to
// take more keys it takes several chunks.  By the heads of a call / this, stage, us: float32 2 x 2048 x 64 12.3 / 12.4, 8 x 2048 18.6 /
// 19.2, 32 x 1024 26.3 / 28.5, 32 x 2048 43.1 / 44.5, 8/2 x 1024 x 128 23.8 / 23.6 (26.5 with 32 keys), 16 x 2048 x 128 60.8 / 62.0.
static int f64_keys_per_chunk(const Geo &g, int bl)
{
    const size_t nbh = (size_t)g.batch * g.h_kv;
    const size_t room = nbh * kQRows * ceil_div(g.n, kGenericKeysPerChunk) * sizeof(double2) + ws_avg_query(nbh);
    const size_t parts = room / (nbh * bl * sizeof(double2)) / wave_share(bl).kg;
    const size_t keys = (g.n + parts - 1) / parts;
    const int shortest = g.n <= 1024 ? 16 : g.n <= 4096 ? 32 : 64, tiles = 16 * wave_share(bl).kg;
    const size_t least = shortest > tiles ? shortest : tiles;
    return (int)(keys < least ? least : (keys + 15) / 16 * 16);
}

// Keys of a range of sweep 1, which leaves one (max, sum) per row: 1024 for long inputs; halved while there would be fewer
// than kSweepWgs ranges, so that short inputs still spread over all compute units.  From 256 keys down a range's length depends on
// its head's length alone, so that a head's sums do not depend on the other heads of a call.  Ranges of 256 keys / this, whole
// stage, us: 8 heads x 1024 18.7 / 15.5, x 2048 19.4 / 14.7, x 4096 20.4 / 16.9, x 8147 21.4 / 22.4, 2 x 8192 18.9 / 15.7, 4 x 8000
// 20.1 / 17.4, 32 x 2048 24.4 / 25.6 (four ranges to a workgroup), 32 x 4096 28.6 / 29.2; with 64 keys up to 4096 8 x 4096 17.5,
// with 128 up to 16384 2 x 16384 20.5 -> 17.7, but 4 x 16000 22.7 -> 24.4 and 8 x 16384 26.7 -> 28.5.
constexpr int kShortHead = 8192;       // keys of a head up to which its ranges are shorter than 256
static int long_range_keys(const Geo &g)
{
    int keys = kMaxRangeKeys;
    while (keys > 256 && (long long)ceil_div(g.n, keys) * g.batch * g.h_kv < kSweepWgs) keys >>= 1;
    return keys;
}
static int sweep_range_keys(const Geo &g)
{
    const int keys = long_range_keys(g);
    return keys > 256 || g.n > kShortHead ? keys : g.n > kShortHead / 4 ? 128 : 64;
}

// Keys of a workgroup of the short sweeps: 256 at least, where a workgroup's start weighs little, and fewer, down to one range, while
// every workgroup has a compute unit.
static int short_sweep_keys(const Geo &g, int range_keys)
{
    int keys = range_keys < 256 ? 256 : range_keys;
    while (keys > range_keys && (long long)ceil_div(g.n, keys / 2) * g.batch * g.h_kv <= 256) keys >>= 1;
    return keys;
}

// The long sweeps need their 512 workgroups busy for a while.  Whole stage, short / long sweeps, us: 65176 keys in all 21.7 / 23.9,
// 131072 30.0 / 32.4, 262144 45.0 / 45.0, 400000 71.5 / 60.6, 1048576 135.8 / 125.5, 1600000 233.9 / 206.3.
static bool long_sweeps(const Geo &g) { return (long long)g.n * g.batch * g.h_kv >= kLongKeys; }

// bytes of the average-query region at the end of the workspace: the partial sums and the mean itself
static size_t ws_avg_query(size_t nbh) { return align_up(nbh * (kAvgChunks + 1) * 128 * sizeof(double), kWsAlign); }

// bytes set aside for the partial results of ranges of 256 keys and more; shorter ones run on into the average-query region
// behind it, whose contents are dead once Qhat is split: a head of up to kShortHead keys has room there
static size_t partial_room(const Geo &g)
{
    static_assert(kShortHead / 128 * kQRows * sizeof(float2) <= kAvgChunks * 128 * sizeof(double), "partial results of a head");
    return align_up((size_t)g.batch * g.h_kv * ceil_div(g.n, long_range_keys(g)) * kQRows * sizeof(float2), kWsAlign);
}

// The generic path sizes its workspace for up to kQRows query rows (the block size may be smaller).
size_t ws_key_scores(const pbs_problem *p)
{
    const Geo g = make_geo(p);
    const size_t nbh = (size_t)g.batch * g.h_kv;
    if (use_mfma(p)) {
        return align_up(nbh * 2 * kQRows * 128 * sizeof(bf16_t), kWsAlign) + align_up(nbh * kQRows * sizeof(float), kWsAlign) +
               partial_room(g) + ws_avg_query(nbh);
    }
    const size_t chunks = ceil_div(g.n, kGenericKeysPerChunk);
    const size_t rows = kQRows;
    return align_up(nbh * rows * g.d * sizeof(double), kWsAlign) + align_up(nbh * rows * chunks * sizeof(double2), kWsAlign) +
           align_up(nbh * rows * sizeof(double2), kWsAlign) + ws_avg_query(nbh);
}

// The average query of every kv head into qavg (fp64, 128 doubles per head), through `partial`.
template <typename E>
static pbs_status run_qavg(const Geo &g, const void *Q, double *partial, double *qavg, hipStream_t s)
{
    const int nbh = g.batch * g.h_kv;
    pbs_status st;
    if ((st = launch(qavg_partial_kernel<E>, dim3(kAvgChunks, nbh), dim3(256), 0, s, (const E *)Q, partial, g)) != PBS_OK)
        return st;
    return launch(qavg_final_kernel, dim3(nbh), dim3(128), 0, s, (const double *)partial, qavg, g);
}

// bl query rows: the last bl of the sequence (qrows == NULL), the listed ones, or (avg) the one average query.
template <typename E, int D>
static pbs_status run_generic(const Geo &g, const void *Q, const void *K, float *scores,
                              char *ws, int bl, const int32_t *qrows, bool avg, hipStream_t s)
{
    const int nbh = g.batch * g.h_kv;
    const int kpc = f64_keys_per_chunk(g, bl), chunks = ceil_div(g.n, kpc);
    double *qhat = reinterpret_cast<double *>(ws);
    ws += align_up((size_t)nbh * kQRows * g.d * sizeof(double), kWsAlign);
    double2 *stats = reinterpret_cast<double2 *>(ws);
    ws += align_up((size_t)nbh * kQRows * sizeof(double2), kWsAlign);
    double2 *partial = reinterpret_cast<double2 *>(ws);    // runs on into the average-query region behind it
    ws += align_up((size_t)nbh * kQRows * ceil_div(g.n, kGenericKeysPerChunk) * sizeof(double2), kWsAlign);
    double *avg_partial = reinterpret_cast<double *>(ws), *qavg = avg_partial + (size_t)nbh * kAvgChunks * 128;
    pbs_status st;
    if (avg && (st = run_qavg<E>(g, Q, avg_partial, qavg, s)) != PBS_OK) return st;
    static_assert(kFormF64Heads <= 2, "a division by the number of heads has to be exact as a multiplication");
    const bool form = !avg && g.r <= kFormF64Heads;
    const double *given = form ? nullptr : qhat;
    if (!form && (st = launch(qhat_f64_kernel<E>, dim3(ceil_div(bl * g.d, 256), nbh), dim3(256), 0, s, (const E *)Q, qhat, g, bl,
                              qrows, (const double *)(avg ? qavg : nullptr))) != PBS_OK) return st;
    // chunks to a workgroup of sweep 1
    const int least = min_f64_keys(g, bl), per = kpc < least ? least / kpc : 1;
    if ((st = launch((scores_stats_f64_kernel<E, D>), dim3(ceil_div(chunks, per), nbh), dim3(256), 0, s, (const E *)K, given,
                     (const E *)Q, qrows, partial, g, bl, kpc, per)) != PBS_OK) return st;
    if ((st = launch(scores_merge_f64_kernel, dim3(ceil_div(bl, 4), nbh), dim3(256), 0, s, partial, stats, bl,
                     chunks * wave_share(bl).kg)) != PBS_OK) return st;
    // Short ranges until there are workgroups enough for eight per compute unit.  Measured, 256 keys / 64, us: d = 64, 49204 keys in
    // all 23.5 / 19.3, 98304 37.9 / 31.4, 131072 40.3 / 41.8, 196608 55.0 / 60.2; d = 128, 32768 keys 38.0 / 19.9,
    // 98304 58.8 / 57.9, 131072 61.2 / 74.9, 262144 116 / 147 (a workgroup reads Qhat, 128 KiB, before its first key).
    const int keys = (long long)g.n * nbh >= 256LL * 8 * 64 ? kF64Keys : least;
    return launch((scores_final_f64_kernel<E, D>), dim3(ceil_div(g.n, keys), nbh), dim3(256), 0, s, (const E *)K, given,
                  (const E *)Q, qrows, (const double2 *)stats, scores, g, bl, keys);
}

}  // namespace pbs

using namespace pbs;

// Everything after the argument checks: the launches of one scoring call with its scratch memory at `ws`.
// proxy: which query rows stand for all queries (pbs_proxy); qrows / m only for PBS_PROXY_QUERY_ROWS.
static pbs_status enqueue_key_scores(const pbs_problem *p, int proxy, const int32_t *qrows, int m, const void *Q,
                                     const void *K, float *scores, void *ws, hipStream_t s)
{
    pbs_status st;
    const Geo g = make_geo(p);
    char *w = reinterpret_cast<char *>(ws);
    const bool avg = proxy == PBS_PROXY_AVG_QUERY;
    const int bl = avg ? 1 : (proxy == PBS_PROXY_QUERY_ROWS ? m : (g.block < g.n ? g.block : g.n));
    if (proxy != PBS_PROXY_QUERY_ROWS) qrows = nullptr;
    if (!use_mfma(p)) {
        if (p->dtype == PBS_BF16) return run_generic<bf16_t, 64>(g, Q, K, scores, w, bl, qrows, avg, s);
        return p->d == 128 ? run_generic<float, 128>(g, Q, K, scores, w, bl, qrows, avg, s)
                           : run_generic<float, 64>(g, Q, K, scores, w, bl, qrows, avg, s);
    }
    const int nbh = g.batch * g.h_kv;
    const int range = sweep_range_keys(g), parts = ceil_div(g.n, range), short_keys = short_sweep_keys(g, range);
    bf16_t *qsplit = reinterpret_cast<bf16_t *>(w);
    w += align_up((size_t)nbh * 2 * kQRows * 128 * sizeof(bf16_t), kWsAlign);
    float *cvec = reinterpret_cast<float *>(w);
    w += align_up((size_t)nbh * kQRows * sizeof(float), kWsAlign);
    float2 *partial = reinterpret_cast<float2 *>(w);       // may run on into the average-query region (partial_room)
    w += partial_room(g);
    double *avg_partial = reinterpret_cast<double *>(w), *qavg = avg_partial + (size_t)nbh * kAvgChunks * 128;
    if (avg && (st = run_qavg<bf16_t>(g, Q, avg_partial, qavg, s)) != PBS_OK) return st;
    if ((st = launch(qhat_split_kernel, dim3(kQRows / 8, nbh), dim3(256), 0, s, (const bf16_t *)Q, qsplit, g, bl, qrows,
                     (const double *)(avg ? qavg : nullptr))) != PBS_OK) return st;
    const bool in_long = long_sweeps(g);
    // one round of workgroups, each with one share of a head's ranges (sweep 1) or keys (sweep 2)
    const int ranges = (int)(((long long)parts * nbh + kSweepWgs - 1) / kSweepWgs);
    const int keys = (int)(((long long)g.n * nbh + kSweepWgs - 1) / kSweepWgs + 4 * kTileKeys - 1) / (4 * kTileKeys) * (4 * kTileKeys);
    if (in_long)
        st = launch(scores_sweep1_kernel, dim3(ceil_div(parts, ranges), nbh), dim3(128), 0, s, (const bf16_t *)K, qsplit, partial, g,
                    range, ranges);
    else
        st = launch(short_input::sweep1_kernel, dim3(ceil_div(g.n, short_keys), nbh), dim3(256), 0, s, (const bf16_t *)K, qsplit, partial,
                    g, short_keys, range);
    if (st != PBS_OK) return st;
    if ((st = launch(scores_merge_kernel, dim3(nbh), dim3(1024), 0, s, partial, cvec, parts, bl)) != PBS_OK) return st;
    if (in_long)
        return launch(scores_sweep2_kernel, dim3(ceil_div(g.n, keys), nbh), dim3(128), 0, s, (const bf16_t *)K, qsplit, cvec,
                      scores, g, keys);
    return launch(short_input::sweep2_kernel, dim3(ceil_div(g.n, short_keys), nbh), dim3(256), 0, s, (const bf16_t *)K, qsplit, cvec,
                  scores, g, short_keys);
}

extern "C" pbs_status pbs_key_scores(const pbs_problem *p, const void *Q, const void *K, float *scores, void *ws,
                                     size_t ws_bytes, void *stream)
{
    pbs_status st = validate(p);
    if (st != PBS_OK) return st;
    if (!Q || !K || !scores) return PBS_ERR_NULL;
    if (!aligned16(Q) || !aligned16(K)) return PBS_ERR_SHAPE;
    if ((st = check_ws(p, PBS_STAGE_KEY_SCORES, ws, ws_bytes)) != PBS_OK) return st;
    return enqueue_key_scores(p, PBS_PROXY_LAST_BLOCK, nullptr, 0, Q, K, scores, ws, (hipStream_t)stream);
}

extern "C" pbs_status pbs_key_scores_proxy(const pbs_problem *p, int proxy, const int32_t *qrows, int32_t m,
                                           const void *Q, const void *K, float *scores, void *ws, size_t ws_bytes,
                                           void *stream)
{
    pbs_status st = validate(p);
    if (st != PBS_OK) return st;
    if (!Q || !K || !scores) return PBS_ERR_NULL;
    if (proxy != PBS_PROXY_LAST_BLOCK && proxy != PBS_PROXY_QUERY_ROWS && proxy != PBS_PROXY_AVG_QUERY)
        return PBS_ERR_UNSUPPORTED;
    if (proxy == PBS_PROXY_QUERY_ROWS && !qrows) return PBS_ERR_NULL;
    if (proxy == PBS_PROXY_QUERY_ROWS && (m < 1 || m > kQRows)) return PBS_ERR_SHAPE;
    if (!aligned16(Q) || !aligned16(K)) return PBS_ERR_SHAPE;
    if ((st = check_ws(p, PBS_STAGE_KEY_SCORES, ws, ws_bytes)) != PBS_OK) return st;
    return enqueue_key_scores(p, proxy, qrows, m, Q, K, scores, ws, (hipStream_t)stream);
}

// ------------------------------------------------------------------ the entry point that allocates nothing
// pbs_key_scores with its scratch memory (split Qhat, per-workgroup row statistics, merged constants) in a
// file-scope device array instead of a caller-supplied workspace.  Every GPU holds its own copy of the array at its
// own address; the address is looked up once per device, with that device current, and host code only ever uses
// that address, never the array's name.
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static void *static_scratch_of_current_device()
{
    constexpr int kMaxDevices = 64;
    static std::atomic<void *> ptr_of[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    void *ptr = ptr_of[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        ptr_of[dev].store(ptr, std::memory_order_release);   // racing first calls look up the same address
    }
    return ptr;
}

extern "C" size_t pbs_key_scores_static_scratch_bytes(void) { return kStaticScratchBytes; }

extern "C" pbs_status pbs_key_scores_static(const pbs_problem *p, const void *Q, const void *K, float *scores,
                                            void *stream)
{
    pbs_status st = validate(p);
    if (st != PBS_OK) return st;
    if (!Q || !K || !scores) return PBS_ERR_NULL;
    if (!aligned16(Q) || !aligned16(K)) return PBS_ERR_SHAPE;
    if (pbs_workspace_bytes(p, PBS_STAGE_KEY_SCORES) > kStaticScratchBytes) return PBS_ERR_WORKSPACE;
    void *ws = static_scratch_of_current_device();
    if (!ws) return PBS_ERR_HIP;
    return enqueue_key_scores(p, PBS_PROXY_LAST_BLOCK, nullptr, 0, Q, K, scores, ws, (hipStream_t)stream);
}

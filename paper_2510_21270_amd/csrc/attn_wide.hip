// pbs_attn_fwd for bf16, d = 128, block = 128: the "wide" matrix-core kernel of Algorithm 1's main loop.
//
// Same transposed formulation as the kernel in attn_fwd.hip (S^T = K' Q'^T, O^T += V'^T P^T, one lane owns one query
// of each 32-query tile), but every wave owns 64 queries (two 32-query tiles) and a workgroup is two waves, so that
// one wave runs per SIMD, and the softmax reference of a query is fixed at its first visible key (see kBigRowSum):
//   * every K' / V'^T fragment read from LDS feeds two MFMAs instead of one;
//   * the softmax arithmetic of a wave is interleaved, in its own instruction stream, with independent MFMAs (the
//     scores of the NEXT sub-tile, the O^T update with the PREVIOUS one), so the matrix pipe does not depend on a
//     second wave happening to be in the opposite phase.
// Key blocks are consumed in sub-tiles of 32 keys.  Sub-tile u of a list chunk covers keys [32 p, 32 p + 32),
// p = u % 4, of listed block u / 4.  A wave has a single instruction stream to itself, so the loop is a three-deep
// software pipeline in which no MFMA of an iteration depends on the vector arithmetic of the same iteration, and that
// arithmetic is spread evenly over the iteration's 32 MFMAs.  Iteration t:
//     MFMAs  0..15:  S(t + 1) = K'(t + 1) Q'^T, both query tiles
//     MFMAs 16..31:  O^T += V'^T(t - 1) P^T(t - 1), both query tiles
//     all along:     P^T(t) = softmax arithmetic on S(t), one score pair per two MFMAs
//     LDS traffic:   V'^T(t - 1) fragment reads under MFMAs 0..7; after MFMA 11 the waves meet (every load issued
//                    two or more iterations ago has landed, the V'^T part just read is free); the loads of K'(t + 4),
//                    V'^T(t + 3) and the key positions of sub-tile t + 4 go out under MFMAs 13, 15 .. 29; K'(t + 2)
//                    fragment reads under MFMAs 16, 18 .. 30
// A wave issues in order and has its SIMD to itself, so whatever stands between two iterations is paid in full: whether
// all queries have their reference is one scalar, the check of the row sums waits for the end of the row, the block for
// sub-tiles that are not plain lies outside the loop, and the operands of the loads are formed ahead of the barrier.  That
// is 1447 -> 1219 clocks per iteration (dense lists, 32768 tokens; the MFMAs alone take 1024); the clock granted under
// the chip's power limit falls with it, 1686 -> 1519 MHz, so that layers gain 3 .. 5 %.
// LDS holds a 4-deep ring of stages filled by asynchronous buffer->LDS loads; stage p holds the K' part p and the
// V'^T part (p + 3) % 4 of their blocks, which is what iteration t = p (mod 4) frees and refills.
// A sub-tile that is not plain (token-level mask, queries without a visible key so far) first rewrites its scores
// and references in a separate block, then goes through the same code.
// The block list of a query block is staged in LDS in chunks, each entry as (block to load, keys that exist, mask
// bit).  When K', Vt and kidx carry a token-order copy behind the permuted tensors (tok_delta > 0), the R own-segment
// blocks at the end of a list are replaced, while staged, by the token-order blocks up to the diagonal; the loop
// itself does not know the difference (a token-order block is just a block index beyond the permuted ones).
// Large problems run on as many workgroups as the chip holds, which take query blocks from queues and prepare the next
// one under the current one.  Measured against one workgroup per query block, whole call: 32 / 8 heads, lists of a tenth
// of the causal blocks, 65536 tokens 3.57 -> 3.48 ms; masks of an eighth, 131072 tokens 14.1 -> 13.7 ms (layer); dense
// masks, where the chip's power and not its idle time is what runs out, 102.0 -> 100.1 ms (layer, 131072 tokens).
#include <limits.h>

#include <utility>

#include "pbs_host.h"

namespace pbs {
namespace wide {

constexpr int BLOCK = 128, D = 128;
constexpr int KS = 32;                                     // keys per sub-tile
constexpr int kStageB = 8192;                              // K' sub-tile: 32 rows x 256 B; V'^T sub-tile: 128 rows x 64 B
constexpr int kLoadsPerWave = 8;                           // 16-byte-per-lane loads a wave issues per stage
constexpr int kList = 1024;                                // listed blocks staged in LDS at a time
constexpr int kXcds = 8, kCohortLog2 = 6;
constexpr int kResident = 512;                             // workgroups the chip holds: two on each of 256 compute units
constexpr int kSplitRows = 256;                            // rows up to which each has four waves
constexpr int kTicketStride = 32;                          // queue heads lie 128 bytes apart
constexpr int kQueueRows = 8 * kResident;                  // rows from which on workgroups take them from queues
constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f;
// The softmax reference of a query is the row maximum of the sub-tile that holds its first visible key and is never
// updated: any reference gives the same softmax as long as nothing overflows, and fp32 / bf16 have room for
// probabilities up to 2^64 relative to it (64 log2 units = 44 nats above the first sub-tile's maximum).  A partial
// row sum beyond that, infinite or NaN marks the whole query block as "bad"; the caller recomputes such blocks with
// the rescaling kernel.  This keeps every vector-ALU write away from the O^T accumulators.
constexpr float kBigRowSum = 1.8446744e19f;                // 2^64

typedef __attribute__((address_space(3))) void *lptr_t;

// One ring stage.  Each stage is a separate __shared__ variable so that the compiler can tell a fragment read of
// one stage from an asynchronous load into another.  Rows are not padded; instead the 16-byte pieces of a row are
// stored XOR-permuted so that the fragment reads below (16 lanes = 16 rows at one logical column) fall into 16
// different bank groups:
//   k: row r (256 B) holds key swap23(r) of the sub-tile, its logical piece c (of 16) at place c ^ (r % 16);
//   v: row e (64 B) holds V'^T[e][32 keys], its logical piece c (of 4) at place c ^ ((e / 4) % 4).
struct __align__(16) Stage {
    unsigned char k[kStageB];
    unsigned char v[kStageB];
    int pos[2 * KS];                                       // original positions of the keys in k (and of the next 32)
};

__device__ __forceinline__ int swap23(int m) { return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1); }

// Descriptors of one kv head: what this wave loads (wave 0: K', wave 1: V'^T), with its size (a sub-tile behind the n-th key starts
// at the end, see scalar_offset), and the key positions; ring: byte offset of this wave's stages behind those of the first
// half of a split row.
struct TileBuffers {
    __amdgpu_buffer_rsrc_t tile, pos;
    int tile_bytes;
    int ring;
};

// A stage is 16 chunks of 1 KiB, one load instruction each (64 lanes x 16 bytes, consecutive in LDS).  Both waves
// execute the same eight instructions with per-wave operands: wave 0 brings the K' sub-tile, wave 1 the V'^T one.
// dma[c]: byte offset inside one key block (K': inside the sub-tile) of the piece this lane moves in load c.
// kfr[x], vfr[k2]: byte offsets inside a stage's k / v array of this lane's fragment reads.
struct LaneOffsets {
    uint32_t dma[kLoadsPerWave];
    uint32_t kfr[8], vfr[2];
};

__device__ __forceinline__ uint32_t k_lane_offset(int chunk, int lane)
{
    const int row = chunk * 4 + (lane >> 4), place = lane & 15;
    return (uint32_t)(swap23(row) * 256 + ((place ^ (row & 15)) << 4));
}

// Vt keeps a block as four groups of 32 keys, each [128 features][32 keys]: a sub-tile is 8 KiB of consecutive bytes
__device__ __forceinline__ uint32_t v_lane_offset(int chunk, int lane)
{
    const int row = chunk * 16 + (lane >> 2), place = lane & 3;
    return (uint32_t)(row * (KS * 2) + ((place ^ ((row >> 2) & 3)) << 4));
}

// half: which of the two rings of a split row (see attn_wide_kernel) this wave reads
__device__ __forceinline__ LaneOffsets lane_offsets(int half, int wave, int lane)
{
    LaneOffsets r;
    const int ln = lane & 31, lh = lane >> 5;
#pragma unroll
    for (int c = 0; c < kLoadsPerWave; ++c) r.dma[c] = wave == 0 ? k_lane_offset(c, lane) : v_lane_offset(c, lane);
    // K' fragment x: logical piece 2 x + h of row n;  V'^T fragment (dt, k2): logical piece 2 k2 + h of row 32 dt + n
#pragma unroll
    for (int x = 0; x < 8; ++x) r.kfr[x] = (uint32_t)(half * sizeof(Stage) + ln * 256 + (((2 * x + lh) ^ (ln & 15)) << 4));
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) r.vfr[k2] = (uint32_t)(half * sizeof(Stage) + ln * 64 + (((2 * k2 + lh) ^ ((ln >> 2) & 3)) << 4));
    return r;
}

// Scalar operands of the loads of part P of block j into stage sg.
struct StageLoad {
    __amdgpu_buffer_rsrc_t rsrc;
    int soff;                          // scalar byte offset of the sub-tile in the tensor
    __attribute__((address_space(3))) unsigned char *dst;    // LDS destination of load 0
};

// Stage P receives the K' part P of block jk and the V'^T part (P + 3) % 4 of block jv.
template <int P>
__device__ __forceinline__ StageLoad stage_load(__attribute__((address_space(3))) unsigned char *dst, const TileBuffers &buf, int jk, int jv, int wave)
{
    StageLoad a;
    static_assert(BLOCK * 256 == D * BLOCK * 2 && KS * 256 == D * KS * 2, "blocks and sub-tiles of K' and Vt are equally large");
    a.rsrc = buf.tile;
    a.soff = scalar_offset((wave == 0 ? jk : jv) * (BLOCK * 256) + (wave == 0 ? P : (P + 3) & 3) * (KS * 256), buf.tile_bytes);
    int own = buf.ring + wave * kStageB;                   // sg.k for wave 0, sg.v behind it for wave 1
    asm volatile("" : "+s"(own));      // formed here: 32 loop-invariant addresses would not fit the scalar registers
    a.dst = dst + own;
    return a;
}

// load c of the eight
template <int C>
__device__ __forceinline__ void issue_load(const StageLoad &a, const LaneOffsets &off)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(a.rsrc, (lptr_t)(a.dst + C * 1024), 16, off.dma[C], a.soff, 0, 0);
}

// Original positions of the 32 keys of part P of block j, next to their K' rows.  Only sub-tiles under the
// token-level mask read them, but the load is issued for every sub-tile, by all lanes of both waves (four bytes per
// lane, the same 256 bytes from each wave): one more instruction in the stream costs less than a branch around it.  The way to the
// part is the instruction's own offset, which counts in memory and in LDS and belongs to what the hardware checks against the
// descriptor's size; the scalar one, to the block, lies within it, since a block has at least one key.
template <int P>
__device__ __forceinline__ void issue_positions(__attribute__((address_space(3))) unsigned char *dst, const TileBuffers &buf,
                                                int j, int lane)
{
    constexpr int part = P * KS * 4;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buf.pos, (lptr_t)(dst + buf.ring - part), 4, lane * 4, j * (BLOCK * 4), part, 0);
}

// K' part P of block j and the V'^T part (P + 3) % 4 of block jv
template <int P>
__device__ __forceinline__ void issue_stage(Stage &sg, const TileBuffers &buf, const LaneOffsets &off, int j, int jv, int wave,
                                            int lane)
{
    const StageLoad a = stage_load<P>((__attribute__((address_space(3))) unsigned char *)sg.k, buf, j, jv, wave);
    issue_load<0>(a, off); issue_load<1>(a, off); issue_load<2>(a, off); issue_load<3>(a, off);
    issue_load<4>(a, off); issue_load<5>(a, off); issue_load<6>(a, off); issue_load<7>(a, off);
    issue_positions<P>((__attribute__((address_space(3))) unsigned char *)sg.pos, buf, j, lane);
}

// Every asynchronous load of this wave has landed, then all waves meet: the stages loaded so far are complete.
__device__ __forceinline__ void sync_stages()
{
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0), gfx9 encoding
    __syncthreads();
}

// The loop's meeting point.  Each wave has waited for all of its loads except the nine it issued in the previous
// iteration, and for its fragment reads; after the barrier the loads of every wave up to two iterations back are
// complete.  That is all an iteration needs: it reads K' fragments loaded two iterations earlier and V'^T fragments
// loaded four iterations earlier, so a load has two full iterations to arrive.  (A plain barrier instruction, not
// __syncthreads(): the fence of the latter would wait for every load.)
__device__ __forceinline__ void sync_older_stages()
{
    __builtin_amdgcn_s_waitcnt(0x0079);                    // vmcnt(9) lgkmcnt(0), gfx9 encoding
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

struct State {
    floatx16 acc_o[4][2];
    float mref[2], l[2];    // reference (log2 units) and sum of exp2(s*c2 - mref), this lane's half of the keys
    bool seen[2];           // the query has met a visible key, i.e. mref is set
    bool all_seen;          // every query of the wave has (the same in all lanes)
};

__device__ __forceinline__ void load_kf(bf16x8 (&kf)[8], const Stage &sg, const LaneOffsets &off)
{
#pragma unroll
    for (int x = 0; x < 8; ++x) kf[x] = *reinterpret_cast<const bf16x8 *>(sg.k + off.kfr[x]);
}

// Score MFMAs are written as assembly statements so that their operands sit where this kernel needs them: the
// result in vector registers (the softmax reads it there), the K' and Q' fragments in accumulation registers
// (AGPRs), which no other instruction of the loop needs (the Q' fragments of query tile 1 stay in vector registers to
// balance the two files).  Everything else is left to the compiler, whose MFMAs keep
// their accumulators -- O^T here -- in AGPRs.  The compiler does not see inside the statements, so the one software
// hazard of a matrix result that can occur is covered by hand: the scores are read by vector instructions, and that
// is always more than a dozen instructions after the last statement (next loop iteration) or behind mfma_fence().
template <int NT>
__device__ __forceinline__ void s_mfma_first(floatx16 &s, const bf16x8 &k, const bf16x8 &q)
{
    if (NT == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=v"(s) : "a"(k), "a"(q));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "a"(k), "v"(q));
}
template <int NT>
__device__ __forceinline__ void s_mfma_next(floatx16 &s, const bf16x8 &k, const bf16x8 &q)
{
    if (NT == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "a"(k), "a"(q));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "a"(k), "v"(q));
}

// More wait states than the longest matrix-result hazard (18 after a 16-pass, 11 after an 8-pass instruction)
__device__ __forceinline__ void mfma_fence()
{
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
}

// S^T of one 32-key sub-tile for both query tiles.  s[nt][x]: key = 16 (x / 8) + 8 h + (x % 8), query = 32 nt + n.
__device__ __forceinline__ void s_mfma(floatx16 (&s)[2], const bf16x8 (&kf)[8], const bf16x8 (&qf)[2][8])
{
    s_mfma_first<0>(s[0], kf[0], qf[0][0]);
    s_mfma_first<1>(s[1], kf[0], qf[1][0]);
#pragma unroll
    for (int x = 1; x < 8; ++x) {
        s_mfma_next<0>(s[0], kf[x], qf[0][x]);
        s_mfma_next<1>(s[1], kf[x], qf[1][x]);
    }
}

// What a sub-tile that is not plain needs before the softmax of one query tile: the token-level mask (masked scores
// become -inf, i.e. probability 0), and for queries that meet their first visible key the reference, set to the row
// maximum of this sub-tile.  A reference, once set, never moves (see the note on kBigRowSum), so O^T is never
// rescaled and the softmax itself is the same code for every sub-tile.
__device__ __forceinline__ void mask_tile(floatx16 (&s)[2], const int *kpos, int room, const int (&qpos)[2], int lh)
{
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int k8 = 16 * u + 8 * lh;                        // 8 consecutive keys of this lane
        // original positions of the keys; slots past the end of the sequence hold 0 and are masked by lim
        const int4 a = *reinterpret_cast<const int4 *>(kpos + k8);
        const int4 b = *reinterpret_cast<const int4 *>(kpos + k8 + 4);
        const int kp[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        if (room >= KS) {                                      // every key of the sub-tile exists (all but a ragged tail)
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                if (kp[x] > qpos[0]) s[0][8 * u + x] = -INFINITY;
                if (kp[x] > qpos[1]) s[1][8 * u + x] = -INFINITY;
            }
        } else {
            const int lim = room - k8;                         // keys x >= lim of this group do not exist
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                if (kp[x] > qpos[0] || x >= lim) s[0][8 * u + x] = -INFINITY;
                if (kp[x] > qpos[1] || x >= lim) s[1][8 * u + x] = -INFINITY;
            }
        }
    }
}

__device__ __forceinline__ void set_reference(State &st, int nt, const floatx16 &s, float c2)
{
    if (!__all(st.seen[nt])) {
        float rmax = -INFINITY;
#pragma unroll
        for (int x = 0; x < 16; ++x) rmax = fmaxf(rmax, s[x]);
        rmax = fmaxf(rmax, __shfl_xor(rmax, 32, 64));
        const bool now = rmax != -INFINITY;
        if (!st.seen[nt]) st.mref[nt] = now ? rmax * c2 : 0.0f;
        st.seen[nt] = st.seen[nt] || now;
    }
}

// O^T MFMA i of a query tile works on V'^T fragment pv_fragment(i): the four O^T tiles with the first 16 keys, then with
// the other 16, so that consecutive MFMAs never share an accumulator
__device__ constexpr int pv_fragment(int i) { return (i & 3) << 1 | i >> 2; }

// What goes out under which of the 32 MFMAs of an iteration (-1: nothing).  The loads and the K' reads take every second
// slot, so that neither the address unit nor LDS, which four waves share, is asked for one a slot.
struct Slots {
    static constexpr int kMeet = 11;                       // the waves meet after this one
    static constexpr int v_read(int m) { return m < 8 ? m : -1; }
    static constexpr int load(int m) { return m > kMeet && m < 31 && m % 2 == 1 ? (m - kMeet - 2) / 2 : -1; }    // 8: positions
    static constexpr int k_read(int m) { return m >= 16 && m % 2 == 0 ? (m - 16) / 2 : -1; }
};

// f(0), f(1), .. with compile-time arguments
template <typename F, int... M>
__device__ __forceinline__ void unrolled(F &f, std::integer_sequence<int, M...>)
{
    (f(std::integral_constant<int, M>{}), ...);
}

// One iteration t (t = P mod 4) of the pipeline described at the top of the file.
// s_cur: scores of sub-tile t (formed by the previous iteration); s_nxt: receives the scores of sub-tile t + 1.
// kf: K' fragments of sub-tile t + 1 on entry, of sub-tile t + 2 on exit.
// pf_prev: probabilities of sub-tile t - 1 (from the previous iteration); pf_new: receives those of sub-tile t.
// sg_v: stage P, whose V'^T part belongs to sub-tile t - 1; after the barrier it receives the K' part P of block jk
// and the V'^T part (P + 3) % 4 of block jv.  sg_k: stage (P + 2) % 4, K' fragments of sub-tile t + 2.
// room / masked describe sub-tile t (its key positions are in sg_v.pos).
template <int P>
__device__ __forceinline__ void step(State &st, floatx16 (&s_cur)[2], floatx16 (&s_nxt)[2], bf16x8 (&kf)[8],
                                     const bf16x8 (&qf)[2][8], const bf16x8 (&pf_prev)[2][2], bf16x8 (&pf_new)[2][2],
                                     Stage &sg_v, const Stage &sg_k, const int (&qpos)[2], int room, bool masked,
                                     float c2, int lh, const TileBuffers &buf, const LaneOffsets &off, int jk, int jv,
                                     int wave, int lane)
{
    bf16x8 vf[8];
    if (__builtin_expect(masked || !st.all_seen, 0)) {
        asm volatile("" ::: "memory");                     // keeps this rare block out of the straight-line code
        if (masked) mask_tile(s_cur, sg_v.pos + buf.ring / 4, room, qpos, lh);
        if (!st.all_seen) {
            set_reference(st, 0, s_cur[0], c2);
            set_reference(st, 1, s_cur[1], c2);
            st.all_seen = __all(st.seen[0] && st.seen[1]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // Softmax of score pair q (query tile q / 8, scores 2 (q % 8) and + 1) in three stages, issued in consecutive
    // MFMA slots so that no instruction waits on the one just before it: multiply-add in slot 2 q, exponentials in
    // slot 2 q + 1, rounding / row sum / pack in slot 2 q + 2.  The row sum adds the unrounded probabilities with two
    // plain additions: on this chip the bf16 dot-product instruction that would sum the rounded pair in one go does
    // not overlap with the matrix instructions the way ordinary vector arithmetic does.
    floatx2 rsum[2] = {{0.0f, 0.0f}, {0.0f, 0.0f}};        // per query tile: sums over even and odd scores
    floatx2 pr = {0.0f, 0.0f}, ar = {0.0f, 0.0f};
    // the vector work of MFMA slot m
    auto softmax_slot = [&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value, q = m >> 1;
        if constexpr ((m & 1) == 0) {
            if constexpr (m > 0) {
                constexpr int z = q - 1, nt = z >> 3;
                bf16x2 t2 = __builtin_convertvector(pr, bf16x2);
                asm volatile("" : "+v"(t2));               // the pack happens here, not where it is consumed
                if constexpr ((z & 7) == 0) rsum[nt] = pr;
                else rsum[nt] += pr;
                asm volatile("" : "+v"(rsum[nt]));
                pf_new[nt][(z & 7) >> 2][2 * (z & 3)] = t2[0];
                pf_new[nt][(z & 7) >> 2][2 * (z & 3) + 1] = t2[1];
            }
            if constexpr (m < 32) {
                ar[0] = __builtin_fmaf(s_cur[q >> 3][2 * (q & 7)], c2, -st.mref[q >> 3]);
                ar[1] = __builtin_fmaf(s_cur[q >> 3][2 * (q & 7) + 1], c2, -st.mref[q >> 3]);
            }
        } else {
            pr[0] = __builtin_amdgcn_exp2f(ar[0]);
            pr[1] = __builtin_amdgcn_exp2f(ar[1]);
        }
        if constexpr (m >= 16) asm volatile("" : "+v"(pr), "+v"(ar));
        __builtin_amdgcn_sched_barrier(0);
    };
    StageLoad ld;
    const auto stage_dst = (__attribute__((address_space(3))) unsigned char *)sg_v.k;
    const auto pos_dst = (__attribute__((address_space(3))) unsigned char *)sg_v.pos;
    auto slot = [&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        if constexpr (m < 16) {
            constexpr int x = m >> 1;
            if constexpr (m == 0) s_mfma_first<0>(s_nxt[0], kf[0], qf[0][0]);
            else if constexpr (m == 1) s_mfma_first<1>(s_nxt[1], kf[0], qf[1][0]);
            else if constexpr ((m & 1) == 0) s_mfma_next<0>(s_nxt[0], kf[x], qf[0][x]);
            else s_mfma_next<1>(s_nxt[1], kf[x], qf[1][x]);
            __builtin_amdgcn_sched_barrier(0);             // the slot's vector work follows its MFMA
        } else {
            constexpr int n = m - 16, f = pv_fragment(n & 7);
            st.acc_o[f >> 1][n >> 3] =
                __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[f], pf_prev[n >> 3][f & 1], st.acc_o[f >> 1][n >> 3], 0, 0, 0);
        }
        constexpr int v = Slots::v_read(m), k = Slots::k_read(m), l = Slots::load(m);
        if constexpr (l >= 0 && l < 8) issue_load<l>(ld, off);
        if constexpr (l == 8) issue_positions<P>(pos_dst, buf, jk, lane);
        if constexpr (v >= 0) vf[v] = *reinterpret_cast<const bf16x8 *>(sg_v.v + off.vfr[v & 1] + (v >> 1) * 2048);
        if constexpr (k >= 0) kf[k] = *reinterpret_cast<const bf16x8 *>(sg_k.k + off.kfr[k]);
        if constexpr (m == Slots::kMeet - 2) {
            ld = stage_load<P>(stage_dst, buf, jk, jv, wave);
            asm volatile("" : "+s"(ld.soff));
        }
        softmax_slot(mc);
        if constexpr (m == Slots::kMeet) sync_older_stages();
    };
    unrolled(slot, std::make_integer_sequence<int, 32>{});
    softmax_slot(std::integral_constant<int, 32>{});
    const float rs0 = rsum[0][0] + rsum[0][1], rs1 = rsum[1][0] + rsum[1][1];
    st.l[0] += rs0;
    st.l[1] += rs1;
    __builtin_amdgcn_sched_barrier(0);
}

// End of a list chunk: the O^T update with its last sub-tile (part 3 of the last block, in stage 0).
__device__ __forceinline__ void drain(State &st, const bf16x8 (&pf)[2][2], const Stage &sg, const LaneOffsets &off)
{
    bf16x8 vf[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) vf[x] = *reinterpret_cast<const bf16x8 *>(sg.v + off.vfr[x & 1] + (x >> 1) * 2048);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            st.acc_o[pv_fragment(i) >> 1][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                vf[pv_fragment(i)], pf[nt][pv_fragment(i) & 1], st.acc_o[pv_fragment(i) >> 1][nt], 0, 0, 0);
}

// A row (query block of one head), in LDS; list entries as (block to load | keys that exist << 20 | mask bit).
struct RowInfo {
    int unit, bhq, i;       // kv head (batch * h_kv + head; -1: there is no such row), query head, query block
    int cnt;                // listed blocks
    int first;              // own segment in token order from this entry on
    int len;                // entries to process (at least one); 0: not known yet
};
constexpr int kEntryBlock = (1 << 18) - 1, kEntryRoomShift = 20, kEntryMask = 1 << 28;
constexpr int kEntryAhead = 1 << 29;                       // behind the last entry: the next row's first block

// Rows are handed out in cohorts of 2^cohort_log2 rows of one kv head with near-equal list lengths, longest lists first;
// XCD x starts with the cohorts x, x + 8, ... (its L2 then holds the tiles its workgroups share).  Ticket t of XCD x ->
// kv head and row of it (0 = the longest list); false past the last cohort, unit = -1 for the unused end of a unit's last
// cohort.
__device__ __forceinline__ bool ticket_row(const Geo &g, int cohort_log2, int x, int t, int &unit, int &mrow)
{
    const int nbk = g.batch * g.h_kv, rows_per_unit = g.r * g.T;
    const int coh = (t >> cohort_log2) * kXcds + x, index = coh / nbk;
    mrow = (index << cohort_log2) + (t & ((1 << cohort_log2) - 1));
    unit = mrow < rows_per_unit ? coh - index * nbk : -1;
    return (index << cohort_log2) < rows_per_unit;
}

// The next row for a workgroup of XCD `home` (one lane) that has drawn `ticket` from its own queue: the row of that
// ticket, else one of the other XCDs' queues (the XCDs run at clocks that differ by up to 8 %).  unit = -1: every queue
// is empty.
__device__ __forceinline__ void claim_row(const Geo &g, int cohort_log2, int32_t *tickets, int home, int ticket, int &unit,
                                          int &mrow)
{
    if (ticket_row(g, cohort_log2, home, ticket, unit, mrow) && unit >= 0) return;
#pragma unroll 1
    for (int k = 0; k < kXcds; ++k) {
        const int x = (home + k) % kXcds;
        while (ticket_row(g, cohort_log2, x, atomicAdd(tickets + x * kTicketStride, 1), unit, mrow))
            if (unit >= 0) return;
    }
    unit = -1;
}

// Queue heads belong to one call: they come from a pool in device memory that is part of the library image (a copy on
// every GPU), never from the caller's workspace, which calls on several streams may share.  The kernel in front of the
// attention kernel takes a set under a key that no other call has (its number; the replays of a graph, which follow
// one another, use theirs again), every workgroup looks its call's set up by the key, and the last one to leave gives it
// back.  More calls than sets at one time: the last ones have none and leave all their rows to the second pass.
constexpr int kQueueSets = 64;                             // one per lane of the wave that looks for its own
constexpr int kLeft = kTicketStride / 2;                   // in a set: workgroups that have left
static __device__ unsigned long long queue_owner[kQueueSets];          // key, 0: free
static __device__ int32_t queue_heads[kQueueSets][kXcds * kTicketStride];

__global__ __launch_bounds__(64) void take_queues_kernel(unsigned long long key)
{
    const int lane = threadIdx.x;
    int set = -1;
    if (lane == 0) {
        for (int k = 0; k < kQueueSets && set < 0; ++k) {
            const int at = (int)((key + k) % kQueueSets);
            if (atomicCAS(&queue_owner[at], 0ull, key) == 0ull) set = at;
        }
    }
    set = __builtin_amdgcn_readfirstlane(set);
    if (set >= 0 && lane < kXcds) queue_heads[set][lane * kTicketStride] = 0;
    if (set >= 0 && lane == kXcds) queue_heads[set][kLeft] = 0;
}

struct Args {
    const bf16_t *Qp, *Kp, *Vt;
    const int32_t *qidx, *kidx, *row_cnt, *col_idx;
    bf16_t *Op;
    float *lse;
    int8_t *redo;
    Geo g;
    int tok_delta;
    unsigned long long key;
    int cohort_log2;
};

// The kernel's arguments, read again where they are used: what only a row's start and end need would otherwise hold scalar
// registers throughout the loop.
__device__ __forceinline__ const Args &args_again()
{
    typedef const __attribute__((address_space(4))) Args *args_t;
    args_t a = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(a));
    return *(const Args *)a;
}

// !QUEUES (key == 0): one workgroup per row, which it finds from its id.  QUEUES: the grid is what the chip holds at a time
// and every workgroup takes rows from the queues of `key` until none is left.  Two kernels, since the loop has no scalar
// registers to spare: as one, with arguments that stayed in registers, 162 of them lay in lanes of vector registers, and a masked
// sub-tile fetched 24 .. 28 back among its 120 instructions.  Without that, and with references that are not looked for
// again once all queries have theirs, attention over 32 / 8 heads x 1152, a twentieth of the blocks, takes 22.1 instead of 25.8 us,
// x 2048 with nothing but masked blocks 81.1 instead of 89.8, x 16384 (queues) over a fiftieth 163.7 instead of 169 .. 174.
//
// Between two rows a wave that has its SIMD to itself has nothing to overlap with, so the next row is prepared under
// the current one: near the end of the current row wave 0 loads its list into LDS (asynchronously) and, a block later,
// brings it into the form the loop reads and draws the ticket of the row after it.  The loads that the last
// block would issue past its end are then those of the next row's first block, and the next Q' fragments travel under
// the epilogue.  (A workgroup per row spent 9-10 us outside its loop and 1-6 us between two workgroups, against 3.3 us per
// block; and the XCDs, which run at clocks up to 8 % apart, waited for the slowest.)
//
// HALVES == 2 (!QUEUES, lists of one chunk): a row has four waves, two to each half of its list, one workgroup to a
// compute unit.  Each half is the pipeline as it stands, on a ring of its own; at the end the halves exchange O^T of
// one query tile each through LDS, bring both to the larger reference and store a tile each.
template <int HALVES, bool QUEUES>
__global__ __launch_bounds__(128 * HALVES) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_wide_kernel(Args args)
{
    __shared__ Stage rg0[HALVES], rg1[HALVES], rg2[HALVES], rg3[HALVES];         // 4 x 16 KiB
    Stage &sg0 = rg0[0], &sg1 = rg1[0], &sg2 = rg2[0], &sg3 = rg3[0];            // buf.ring and off lead to the own ones
    __shared__ floatx4 sums[HALVES == 2 ? 256 : 1];        // row sums and references of a split row's halves
    __shared__ int lists[QUEUES ? 2 : 1][kList];           // block lists (a chunk of each) of this row and the next
    __shared__ int tails[64];                              // the end of a list that is longer than a chunk
    __shared__ int next_cnt[64], sink[64];
    __shared__ RowInfo info[QUEUES ? 2 : 1];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(HALVES == 2 ? threadIdx.x >> 6 & 1 : threadIdx.x >> 6);
    const int half = HALVES == 2 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 7) : 0;
    const bool keeper = wave == 0 && half == 0;            // the wave that keeps the lists
    const int ln = lane & 31, lh = lane >> 5;
    const float c2 = args.g.scale * kLog2eF;
    const LaneOffsets off = lane_offsets(half, wave, lane);
    constexpr int kRawDword = 0x00020000;                  // gfx9 descriptor word 3: raw 32-bit data format

    auto decode = [&](const Args &a, int unit, int mrow, int &bhq, int &i) {
        const Geo &g = a.g;
        const int later = mrow / g.r, kv = unit / g.h_kv;
        i = g.T - 1 - later;
        bhq = kv * g.h_q + (unit - kv * g.h_kv) * g.r + mrow - later * g.r;
    };
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    // the raw list entries [base, base + kList) of a row, up to T (wave 0)
    auto load_list = [&](const Args &a, int bhq, int i, int *list, int base) {
        const Geo &g = a.g;
        const int m = max(0, min(g.T - base, kList));
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<int32_t *>(a.col_idx + ((size_t)bhq * g.T + i) * g.T + base), 0, m * 4, kRawDword);
        for (int k = 0; k < m; k += 64)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)(list + k), 4, lane * 4, k * 4, 0, 0);
    };
    // blocks of a row's own segment that token order may replace, 0: none
    auto own_blocks = [&](const Args &a, int i) {
        return a.tok_delta > 0 && i / a.g.R < a.g.G ? allowed_cols(i, a.g) - first_masked_col(i, a.g) : 0;
    };
    // Raw entries [base, base + kList) -> the form the loop reads (wave 0).  An entry that the causal structure does not
    // admit becomes block 0 with no existing key under the mask: a sub-tile that contributes nothing.
    // Behind the last entry stands a copy of it: the loop reads one entry ahead.
    auto pack_list = [&](const Args &a, int i, int first, int len, int *list, int base) {
        const Geo &g = a.g;
        const int ni = allowed_cols(i, g), jmask = first_masked_col(i, g);
        auto packed = [&](int e, int raw) {
            int j = raw, to = raw;
            if (e >= first) {                              // token order: keys of the diagonal block need the mask
                j = jmask + e - first;
                to = a.tok_delta + j;
            } else if (j < 0 || j >= ni) {
                return (int)kEntryMask;
            }
            const bool masked = e >= first ? j == i : j >= jmask;
            return to | min(BLOCK, g.n - j * BLOCK) << kEntryRoomShift | (masked ? kEntryMask : 0);
        };
        for (int t = lane; t < min(len - base, kList); t += 64) list[t] = packed(base + t, list[t]);
        if (lane == 0 && len - base < kList) list[len - base] = 0;
    };
    // With a list's first chunk (and, where it is longer, its end in tails) in LDS: its length in blocks to process, and
    // the packed entries (wave 0).
    // Own segment in token order: when a list ends with all blocks jmask .. ni - 1 of the query block's own (full)
    // segment, ascending, these entries stand for the blocks jmask .. i of the token-order copies.  Keys of a segment are
    // the same set in either order, so the visible keys are the same; in token order the blocks before the diagonal
    // need no mask and those after it hold no visible key.
    auto close_list = [&](const Args &a, RowInfo &w, int i, int cnt, int *list) {
        const int own = own_blocks(a, i), jmask = first_masked_col(i, a.g);
        int first = INT_MAX, len = cnt;
        if (own > 0 && cnt >= own) {
            const int t = cnt <= kList ? list[min(cnt - own + lane, kList - 1)] : tails[lane];
            if (__all(lane >= own || t == jmask + lane)) {
                first = cnt - own;
                len = first + i - jmask + 1;
            }
        }
        if (len == 0) {                                    // an empty list: one entry that contributes nothing
            len = 1;
            if (lane == 0) list[0] = -1;
        }
        pack_list(a, i, first, len, list, 0);
        if (lane == 0) {
            w.cnt = cnt;
            w.first = first;
            w.len = len;
        }
    };
    auto load_tail = [&](const Args &a, int bhq, int i, int cnt) {
        const Geo &g = a.g;
        const int own = own_blocks(a, i);
        if (own > 0 && cnt > kList) {
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<int32_t *>(a.col_idx + ((size_t)bhq * g.T + i) * g.T + cnt - own), 0, own * 4, kRawDword);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)tails, 4, lane * 4, 0, 0, 0);
        }
    };
    TileBuffers buf;
    buf.ring = half * (int)sizeof(Stage);
    auto open_buffers = [&](const Args &a, int unit) {
        const Geo &g = a.g;
        // tok_delta > 0: a token-order copy of K', Vt and kidx lies tok_delta = batch * h_kv * T blocks behind the
        // permuted one, so block j of this head in token order is block tok_delta + j of the same descriptors
        const size_t bhk = unit;
        const int reach = a.tok_delta * BLOCK + g.n;       // rows within reach of this head's descriptors
        buf.tile_bytes = wave == 0 ? reach * 256 : (a.tok_delta + g.T) * (D * BLOCK * 2);
        buf.tile = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(wave == 0 ? a.Kp + bhk * (size_t)g.n * D
                                                                                    : a.Vt + bhk * (size_t)g.T * D * BLOCK),
                                                     0, buf.tile_bytes, kRawDword);
        buf.pos = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(a.kidx + bhk * (size_t)g.n), 0, reach * 4, kRawDword);
    };
    // jv0: the first iteration of a row multiplies V'^T part 3 of this block by zero probabilities; that is a block of the
    // row's list, the same one for both halves, so that infinite values meet no more zeros than they would in one piece
    auto issue_block = [&](int j, int jv0) {
        issue_stage<0>(sg0, buf, off, j, jv0, wave, lane);
        issue_stage<1>(sg1, buf, off, j, j, wave, lane);
        issue_stage<2>(sg2, buf, off, j, j, wave, lane);
        issue_stage<3>(sg3, buf, off, j, j, wave, lane);
    };
    auto query_buffer = [&](const Args &a, int bhq) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(a.Qp + (size_t)bhq * a.g.n * D), 0, a.g.n * 256, kRawDword);
    };
    // Q' fragments: lane (n, h) holds Q'[q0 + 32 nt + n][16 ks + 8 h .. +8]
    // (buffer loads: the compiler moves plain loads of read-only memory down to their use, behind the waits; rows past
    // the end of the head read as zeros)
    bf16x8 qf[2][8];
    int qpos[2];
    auto load_queries = [&](const Args &a, int bhq, int i) {
        const __amdgpu_buffer_rsrc_t r = query_buffer(a, bhq);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const int qs = i * BLOCK + wave * 64 + 32 * nt + ln;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                qf[nt][k] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, qs * 256 + 16 * lh, 32 * k, 0));
            qpos[nt] = qs < a.g.n ? (a.qidx ? a.qidx[(size_t)bhq * a.g.n + qs] : qs) : -1;
        }
    };

    const int home = blockIdx.x % kXcds;
    int32_t *tickets = nullptr;
    if constexpr (QUEUES) {
        const uint64_t mine = __ballot(__hip_atomic_load(&queue_owner[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == args.key);
        if (!mine) {                                       // no set was free: every row is flagged
            for (long long f = 128LL * blockIdx.x + threadIdx.x; f < 2LL * args.g.batch * args.g.h_q * args.g.T; f += 128LL * gridDim.x)
                args.redo[f] = 1;
            return;
        }
        tickets = queue_heads[__builtin_ctzll(mine)];
    }
    auto leave = [&]() {                                   // no ticket is drawn after this (one lane)
        if (atomicAdd(tickets + kLeft, 1) == (int)gridDim.x - 1)
            atomicExch(&queue_owner[(tickets - queue_heads[0]) / (kXcds * kTicketStride)], 0ull);
    };
    // the row of a ticket as the next one (one lane); ticket < 0: there is none
    auto open_next = [&](const Args &a, RowInfo &w, int ticket) {
        int unit = -1, mrow = 0;
        if (ticket >= 0) claim_row(a.g, a.cohort_log2, tickets, home, ticket, unit, mrow);
        w.unit = unit;
        w.len = 0;
        if (unit >= 0) decode(a, unit, mrow, w.bhq, w.i);
    };
    int unit, bhq, i;                                      // of the current row
    {
        const Args &a = args;
        const Geo &g = a.g;
        int mrow;
        if constexpr (!QUEUES) {
            if (!ticket_row(g, a.cohort_log2, home, blockIdx.x / kXcds, unit, mrow) || unit < 0) return;
        } else {
            // the first row is drawn too, not tied to the workgroup's id: a workgroup that another kernel's work keeps off
            // the chip then holds no row back
            if (threadIdx.x == 0)
                claim_row(g, a.cohort_log2, tickets, home, atomicAdd(tickets + home * kTicketStride, 1), next_cnt[0], next_cnt[1]);
            __syncthreads();
            unit = uniform(next_cnt[0]);
            mrow = uniform(next_cnt[1]);
            if (unit < 0) {
                if (threadIdx.x == 0) leave();
                return;
            }
            __syncthreads();                               // (next_cnt is loaded into later)
        }
        decode(a, unit, mrow, bhq, i);
        const size_t at = (size_t)bhq * g.T + i;
        if (keeper) load_list(a, bhq, i, lists[0], 0);
        load_queries(a, bhq, i);
        open_buffers(a, unit);
        const int raw0 = uniform(a.col_idx[at * g.T]);     // read beside the count
        const int cnt = max(0, min(uniform(a.row_cnt[at]), g.T));
        if (keeper) load_tail(a, bhq, i, cnt);
        const bool early = cnt > own_blocks(a, i);            // the first entry cannot be one that token order replaces
        int j0 = raw0 >= 0 && raw0 < allowed_cols(i, g) ? raw0 : 0;
        if (!early) {
            sync_stages();
            if (keeper) close_list(a, info[0], i, cnt, lists[0]);
            __syncthreads();
            j0 = uniform(lists[0][0]) & kEntryBlock;
        }
        if (half == 0) issue_block(j0, j0);
        if (early && keeper) {
            __builtin_amdgcn_s_waitcnt(0x8F74);            // vmcnt(36): what was issued before the tiles has landed
            asm volatile("" ::: "memory");
            close_list(a, info[0], i, cnt, lists[0]);
        }
        if constexpr (HALVES == 2) {
            __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the list is in LDS; the tiles may still travel
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (half == 1) issue_block(uniform(lists[0][(uniform(info[0].len) + 1) >> 1]) & kEntryBlock, j0);
        } else if (QUEUES && threadIdx.x == 0) {
            open_next(a, info[1], atomicAdd(tickets + home * kTicketStride, 1));
        }
        sync_stages();
    }

    for (int cur = 0;; cur ^= 1) {
        // here: the first block's tiles (its four K' parts and V'^T parts) are in the ring, Q' in registers, the row's
        // info and list (first chunk) in info[cur], lists[cur]
        // a split row: the halves' blocks differ by one at most
        const int whole = uniform(info[cur].len), upper = (whole + 1) >> 1;
        const int len = HALVES == 1 ? whole : half == 0 ? upper : whole - upper;
        const int skip = HALVES == 1 ? 0 : half * upper;   // entries of the list in front of this half's
        const int *list = lists[cur] + skip;
        State st;
        st.all_seen = false;
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            st.mref[nt] = 0.0f;
            st.l[nt] = 0.0f;
            st.seen[nt] = qpos[nt] < 0;                    // padding rows never hold the wave on the careful path
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int x = 0; x < 16; ++x) st.acc_o[dt][nt][x] = 0.0f;
        }
        // first scores, the K' fragments of part 1
        floatx16 sa[2], sb[2];
        bf16x8 kf[8];
        load_kf(kf, sg0, off);
        s_mfma(sa, kf, qf);
        mfma_fence();
        load_kf(kf, sg1, off);
        bf16x8 pa[2][2], pb[2][2];                         // probabilities of the previous / the current sub-tile
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int x = 0; x < 8; ++x) pa[u >> 1][u & 1][x] = (bf16_t)0.0f;
        __builtin_amdgcn_sched_barrier(0);

        // The next row's preparation (wave 0), in steps 0 .. 2 at the ends of blocks; 3: done, info[cur ^ 1] and
        // lists[cur ^ 1] are complete.  The last step also puts the row's first entry behind this row's last one, where
        // the block before the last one picks it up: both waves, so that a block's barriers have to lie in between.
        constexpr int kPrepare = 5;
        int step_no = 0, ticket = -1;
        auto prepare = [&]() {
            asm volatile("" ::: "memory");                 // no read of LDS moves up across the blocks' barriers
            RowInfo &w = info[cur ^ 1];
            if (uniform(w.unit) < 0) {
                step_no = 3;
                return;
            }
            const Args &a = args_again();
            const int nb = uniform(w.bhq), nq = uniform(w.i);
            if (step_no == 0) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(a.row_cnt + (size_t)nb * a.g.T + nq), 0, 4, kRawDword),
                    (lptr_t)next_cnt, 4, lane * 4, 0, 0, 0);
                load_list(a, nb, nq, lists[cur ^ 1], 0);
                // one word of every line of the row's Q' block, so that its fragments come from the cache
                const __amdgpu_buffer_rsrc_t r = query_buffer(a, nb);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)sink, 4, lane * 128,
                                                             scalar_offset(nq * (BLOCK * 256) + k * 8192, a.g.n * 256), 0, 0);
                step_no = 1;
                return;
            }
            const int cnt = max(0, min(uniform(next_cnt[0]), a.g.T));
            if (step_no == 1 && cnt > kList) {
                load_tail(a, nb, nq, cnt);
                step_no = 2;
                return;
            }
            close_list(a, w, nq, cnt, lists[cur ^ 1]);
            if (lane == 0 && w.unit == unit) lists[cur][len & (kList - 1)] = lists[cur ^ 1][0] | kEntryAhead;
            if (lane == 0) ticket = atomicAdd(tickets + home * kTicketStride, 1);        // of the row after that, used in the epilogue
            step_no = 3;
        };
        // rare work at the end of block e: the next chunk of a list of more than kList entries, preparation steps
        const int chunk_end = len >= kList ? kList - 3 : INT_MAX;
        int event = QUEUES && wave == 0 ? min(chunk_end, max(0, len - kPrepare)) : chunk_end;
        auto at_event = [&](int e) {
            asm volatile("" ::: "memory");
            if (((e + 3) & (kList - 1)) == 0 && e + 3 <= len) {
                __syncthreads();
                if (wave == 0) {
                    const Args &a = args_again();
                    load_list(a, bhq, i, lists[cur], e + 3);
                    __builtin_amdgcn_s_waitcnt(0x0F70);
                    asm volatile("" ::: "memory");
                    pack_list(a, i, uniform(info[cur].first), len, lists[cur], e + 3);
                }
                sync_stages();
            }
            if constexpr (QUEUES)
                if (wave == 0 && e >= len - kPrepare && e <= len - 4 && step_no < 3) prepare();
            const int chunk = e + 3 + kList <= len ? ((e + 3) & -kList) + kList - 3 : INT_MAX;
            event = QUEUES && wave == 0 ? min(chunk, e < len - kPrepare ? len - kPrepare : e + 1) : chunk;
        };

        int pk = uniform(list[0]);
        int later = list[1];                               // the entry after the next one, read a block ahead
        int jc = pk & kEntryBlock;
        for (int e = 0; e < len; ++e) {
            const int pn = uniform(later);                 // past the end: the next row's first block or any (unused)
            later = HALVES == 1 ? list[(e + 2) & (kList - 1)] : lists[cur][(skip + e + 2) & (kList - 1)];
            const int jn = pn & kEntryBlock;
            const bool masked = (pk & kEntryMask) != 0;
            const int room0 = (pk >> kEntryRoomShift) & 255;             // keys of the block that exist
            // part p: probabilities of part p; scores of part p + 1; O^T update with part p - 1; K' fragments of
            // part p + 2 (parts outside 0..3 are those of the neighbouring listed blocks).  Stage p is refilled with
            // K' part p of the next block and V'^T part p - 1 of the next block (part 3 of this block when p = 0).
            // The first iteration of a row updates O^T with zero probabilities.
            step<0>(st, sa, sb, kf, qf, pa, pb, sg0, sg2, qpos, room0, masked, c2, lh, buf, off, jn, jc, wave, lane);
            step<1>(st, sb, sa, kf, qf, pb, pa, sg1, sg3, qpos, room0 - KS, masked, c2, lh, buf, off, jn, jn, wave, lane);
            step<2>(st, sa, sb, kf, qf, pa, pb, sg2, sg0, qpos, room0 - 2 * KS, masked, c2, lh, buf, off, jn, jn, wave, lane);
            step<3>(st, sb, sa, kf, qf, pb, pa, sg3, sg1, qpos, room0 - 3 * KS, masked, c2, lh, buf, off, jn, jn, wave, lane);
            jc = jn;
            pk = pn;
            if constexpr (HALVES == 1)
                if (__builtin_expect(e == event, 0)) at_event(e);
        }
        if (HALVES == 2 && len < upper)                    // the other half's last block: its meeting points
            for (int p = 0; p < BLOCK / KS; ++p) __builtin_amdgcn_s_barrier();
        const bool ahead = (pk & kEntryAhead) != 0;        // the ring holds the next row's first block
        drain(st, pa, sg0, off);
        const Args &a = args_again();

        // ---- O' = diag(l)^-1 O; acc_o[dt][nt][x]: d = 32 dt + 8 (x / 4) + 4 h + (x % 4), query = q0 + 32 nt + n.
        // The two lanes of a query exchange pieces so that each stores 8 consecutive features.
        uintx4 out[2][4][2];
        float lt[2];
        auto finish_tile = [&](auto tile) __attribute__((always_inline)) {
            constexpr int nt = decltype(tile)::value;
            lt[nt] = st.l[nt] + __shfl_xor(st.l[nt], 32, 64);
            const float inv = lt[nt] > 0.0f ? 1.0f / lt[nt] : 0.0f;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int half8 = 0; half8 < 2; ++half8) {
                    uint32_t piece[2][2];                  // [features 8 (2 half8 + y)][pair]
#pragma unroll
                    for (int y = 0; y < 2; ++y)
#pragma unroll
                        for (int z = 0; z < 2; ++z) {
                            const int x = 4 * (2 * half8 + y) + 2 * z;
                            const floatx2 o = {st.acc_o[dt][nt][x] * inv, st.acc_o[dt][nt][x + 1] * inv};
                            piece[y][z] = __builtin_bit_cast(uint32_t, __builtin_convertvector(o, bf16x2));
                        }
#pragma unroll
                    for (int z = 0; z < 2; ++z) {
                        // lower half: (own, other's) of piece 0; upper half: (other's, own) of piece 1
                        const auto sw = __builtin_amdgcn_permlane32_swap(piece[0][z], piece[1][z], false, false);
                        out[nt][dt][half8][z] = sw[0];
                        out[nt][dt][half8][2 + z] = sw[1];
                    }
                }
        };
        auto store_tile = [&](auto tile) __attribute__((always_inline)) {
            constexpr int nt = decltype(tile)::value;
            const int qs = i * BLOCK + wave * 64 + 32 * nt + ln;
            if (qs < a.g.n) {
                bf16_t *dst = a.Op + ((size_t)bhq * a.g.n + qs) * D + 8 * lh;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int y = 0; y < 2; ++y) *reinterpret_cast<uintx4 *>(dst + 32 * dt + 16 * y) = out[nt][dt][y];
                if (a.lse && lh == 0)
                    a.lse[(size_t)bhq * a.g.n + qs] = lt[nt] > 0.0f ? (st.mref[nt] + log2f(lt[nt])) * kLn2F : -INFINITY;
            }
        };
        constexpr auto tile0 = std::integral_constant<int, 0>{};
        constexpr auto tile1 = std::integral_constant<int, 1>{};
        auto finish = [&]() {
            finish_tile(tile0);
            finish_tile(tile1);
        };
        // each wave's half of the row's flag: some probability outgrew its fixed reference (the caller redoes the row)
        auto outgrown = [](float l) { return !(l <= kBigRowSum); };
        auto flag_row = [&](bool lane_bad) {
            const bool bad = __any(lane_bad);
            if (lane == 0) {
                const size_t f = ((size_t)bhq * a.g.T + i) * 2 + wave;
                if (QUEUES) a.redo[f] = bad ? 1 : 0;
                else reinterpret_cast<int16_t *>(a.redo)[f] = bad ? 1 : 0;
            }
        };
        auto store = [&]() {
            store_tile(tile0);
            store_tile(tile1);
            flag_row(outgrown(st.l[0]) || outgrown(st.l[1]));
        };
        if constexpr (HALVES == 2) {
            // Half h keeps query tile h: it leaves O^T of the other one in its own ring, where stage dt takes
            // [wave][4 registers][lane] of feature tile dt, and adds what the other half has left.
            sync_stages();                                 // every load has landed, every fragment has been read
            auto ring_tile = [&](int dt, int of) {
                Stage &sg = dt == 0 ? rg0[of] : dt == 1 ? rg1[of] : dt == 2 ? rg2[of] : rg3[of];
                static_assert(sizeof(floatx4) * 2 * 4 * 64 == kStageB, "a feature tile of both waves fits the K' part of a stage");
                return reinterpret_cast<floatx4 *>(sg.k) + wave * 256 + lane;
            };
            auto leave_tile = [&](auto tile) __attribute__((always_inline)) {
                constexpr int nt = decltype(tile)::value;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        ring_tile(dt, half)[64 * x] = floatx4{st.acc_o[dt][nt][4 * x], st.acc_o[dt][nt][4 * x + 1],
                                                              st.acc_o[dt][nt][4 * x + 2], st.acc_o[dt][nt][4 * x + 3]};
            };
            if (half == 0) leave_tile(tile1);
            else leave_tile(tile0);
            // a query that has met no key has no reference: the other half's is taken
            sums[threadIdx.x] = floatx4{st.l[0], st.l[1], st.seen[0] ? st.mref[0] : -INFINITY, st.seen[1] ? st.mref[1] : -INFINITY};
            __syncthreads();
            const floatx4 other = sums[threadIdx.x ^ 128];
            // (first half) the sums of the whole row against its first reference, as an undivided row has them: the same rows
            // are redone
            bool bad = outgrown(other[0]) || outgrown(other[1]);
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                bad = bad || outgrown(st.l[nt] + (st.seen[nt] ? other[nt] * __builtin_amdgcn_exp2f(other[2 + nt] - st.mref[nt]) : 0.0f));
            auto merge_tile = [&](auto tile) __attribute__((always_inline)) {
                constexpr int nt = decltype(tile)::value;
                const float ra = st.seen[nt] ? st.mref[nt] : -INFINITY, rb = other[2 + nt], ref = fmaxf(ra, rb);
                const float wa = ra == ref ? 1.0f : __builtin_amdgcn_exp2f(ra - ref);
                const float wb = rb == ref ? 1.0f : __builtin_amdgcn_exp2f(rb - ref);
                st.mref[nt] = ref;
                st.l[nt] = st.l[nt] * wa + other[nt] * wb;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const floatx4 o = ring_tile(dt, half ^ 1)[64 * x];
#pragma unroll
                        for (int y = 0; y < 4; ++y)
                            st.acc_o[dt][nt][4 * x + y] = st.acc_o[dt][nt][4 * x + y] * wa + o[y] * wb;
                    }
                finish_tile(tile);
                store_tile(tile);
            };
            if (half == 0) {
                merge_tile(tile0);
                flag_row(bad);
            } else {
                merge_tile(tile1);
            }
            return;
        }
        if constexpr (!QUEUES) {
            finish();
            store();
            break;
        }
        if (!ahead) {
            if (wave == 0)
                while (step_no < 3) {                      // a list too short to prepare the next row under it
                    __builtin_amdgcn_s_waitcnt(0x0F70);
                    prepare();
                }
            sync_stages();                                 // info, list; the loads issued past the end have landed
        }
        const int unit1 = uniform(info[cur ^ 1].unit);
        if (unit1 < 0) {                                   // no further row
            finish();
            store();
            if (threadIdx.x == 0) leave();
            break;
        }
        const int bhq1 = uniform(info[cur ^ 1].bhq), i1 = uniform(info[cur ^ 1].i);
        const int j1 = uniform(lists[cur ^ 1][0]) & kEntryBlock;
        load_queries(a, bhq1, i1);
        if (ahead) {                                       // V'^T part 3 of the first block is all that is missing
            __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): this wave has read sg0.v ...
            __builtin_amdgcn_s_barrier();                  // ... and so has the other
            __builtin_amdgcn_sched_barrier(0);
            if (wave == 1) {
                const StageLoad ld = stage_load<0>((__attribute__((address_space(3))) unsigned char *)sg0.k, buf, j1, j1, 1);
                issue_load<0>(ld, off); issue_load<1>(ld, off); issue_load<2>(ld, off); issue_load<3>(ld, off);
                issue_load<4>(ld, off); issue_load<5>(ld, off); issue_load<6>(ld, off); issue_load<7>(ld, off);
            }
        } else {
            open_buffers(a, unit1);
            issue_block(j1, j1);
        }
        __builtin_amdgcn_sched_barrier(0);
        finish();
        __builtin_amdgcn_sched_barrier(0);
        if (threadIdx.x == 0) open_next(a, info[cur], ticket);              // in the place of this row's
        sync_stages();                                     // Q' and the first block are here
        store();
        unit = unit1;
        bhq = bhq1;
        i = i1;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // the loads issued past the end have landed
}

}  // namespace wide

// Whether workgroups take their rows from queues: with a few rows per workgroup a queue's lookahead of one row costs more
// balance than the gaps between workgroups.
bool wide_rows_from_queues(const Geo &g) { return (long long)g.batch * g.h_q * g.T >= wide::kQueueRows; }

// redo: [batch * h_q * T] flags, written for every query block: int32, or int16 where rows come from queues.
pbs_status launch_attn_wide(const Geo &g, const void *Qp, const void *Kp, const void *Vt, const int32_t *qidx,
                            const int32_t *kidx, const int32_t *row_cnt, const int32_t *col_idx, void *Op, float *lse,
                            void *redo, int tok_delta, hipStream_t s)
{
    const long long units = (long long)g.batch * g.h_kv, rows = (long long)g.r * g.T;
    const bool queues = wide_rows_from_queues(g);
    // With one row to a compute unit the longest row is what a call waits for, and half of the chip is idle: its list is cut
    // in two.  One piece against two, whole call on causal lists: 4 / 2 heads x 1024 29.9 -> 22.7 us, 32 / 8 x 1024 (256
    // rows) 32.2 -> 25.7 us, 4 / 2 x 4096 77.7 -> 49.5 us.  A second row after the first pays its start and end again, which
    // the lists have to be long for: 8 / 2 x 8192 (512 rows) 168 -> 136 us, but with a twentieth of the blocks 38.5 ->
    // 43.0 us; the lengths are not known here.  (A list of such a call fits one chunk.)
    const bool split = units * rows <= wide::kSplitRows;
    static_assert(wide::kSplitRows < wide::kList, "a split row's list lies in LDS whole, with an entry behind it");
    // A split row has a compute unit to itself: the XCDs take turns row by row, so that none has more rows than compute units,
    // and no workgroup is there for the unused end of a cohort.  In cohorts of 64 with 8 or more kv heads, of 8 with fewer,
    // against that, lists of a tenth of the blocks, us: 250 heads x 128 79.4 / 17.1, 64 x 512 29.6 / 17.4, 40 x 700 33.0 / 20.1, 12 x
    // 2600 33.8 / 22.2, 7 x 4600 32.6 / 25.4, 32 / 8 x 1024 20.1 / 20.1, 2 / 1 x 16000 35.6 / 35.1.
    const int cohort_log2 = queues ? wide::kCohortLog2 : split ? 0 : __builtin_ctz(cohort_rows(g));
    unsigned wgs = wide::kResident;
    unsigned long long key = 0;
    if (queues) {
        static std::atomic<unsigned long long> calls{0};
        key = calls.fetch_add(1, std::memory_order_relaxed) + 1;
        const pbs_status st = launch(wide::take_queues_kernel, dim3(1), dim3(64), 0, s, key);
        if (st != PBS_OK) return st;
    } else {
        const long long cohorts = units * ((rows + (1 << cohort_log2) - 1) >> cohort_log2);
        wgs = (unsigned)(((cohorts + wide::kXcds - 1) / wide::kXcds * wide::kXcds) << cohort_log2);
    }
    return launch(queues ? wide::attn_wide_kernel<1, true> : split ? wide::attn_wide_kernel<2, false> : wide::attn_wide_kernel<1, false>,
                  dim3(wgs), dim3(split ? 256 : 128), 0, s,
                  wide::Args{(const bf16_t *)Qp, (const bf16_t *)Kp, (const bf16_t *)Vt, qidx, kidx, row_cnt, col_idx, (bf16_t *)Op,
                             lse, (int8_t *)redo, g, tok_delta, key, cohort_log2});
}

}  // namespace pbs

// Chunked prefill over the paged cache for gfx950: causal attention of a chunk of new query rows
// against history + chunk, both already in the cache (each row is Background Eq. 1 over its
// visible prefix, with the grouping of Opt-GQA Eq. 7 and the valid-block rule of Opt-Pa Eq. 9).
//
// Query length > 1 makes this a dense contraction, so the matrix cores are used at full width and
// every cache byte is fetched and converted once per WORKGROUP:
//   * A score tile has 16 query rows of ONE query head as its columns (column n = chunk row
//     i0+n).  A wavefront carries two such tiles as one operand of 32 columns, a workgroup of 8
//     wavefronts 16 of them (256 rows), all of the same (sequence, KV head) pair; or 8 tiles, four
//     waves' worth, where a pair has no more (the other waves then bring three quarters of the stream:
//     8 sequences x 16 rows over 8192 tokens 72 -> 61 us, one 16-column tile a wave before).
//   * The pair's K/V stream, two 16-token blocks (a group) at a time, through a ring of LDS slots
//     in matrix-core operand order, already converted to fp16.  The waves form two
//     producer teams that share a stage's four groups three to one (the first team's waves are the
//     older ones on their SIMDs and get through a stage sooner); in a team wave 0 brings block
//     A's K and all K scales, wave 1 block B's K and the V scales, waves 2 and 3 the V pieces of both
//     blocks (tokens that are not in the cache are zeroed, so stale bytes cannot reach an accumulator).
//     All eight then read their operands back with 16-byte LDS loads and run the online-softmax
//     update of attn_tile.hpp's arithmetic on their columns.  One barrier per stage of four groups;
//     the global loads of the stage after next are in flight while a stage is consumed.
//   * What bounds it: energy.  At d = 128 over E4M3 a stage takes 7 500 cycles against 4 350 of matrix
//     instructions and the chip lowers its clock to 1.9 GHz; the form with 16x16x32 products and without
//     the pipeline below took 9 600 cycles at 2.35 GHz, 4.10 us a stage against 3.99.  (On zeros, which
//     hardly toggle a wire, the clock stays at 2.4 GHz: 731 -> 598 us for 8 x 512 rows over 8192
//     tokens.)  Without the K/V operand reads from LDS a stage is 11 % shorter, without production
//     10 %, without exponentials 6 %.
//   * Workgroup ids are dealt to the 8 XCDs round-robin, so the mapping puts all workgroups of a
//     pair on ONE XCD: the pair's 2 MB of cache are fetched from HBM once and re-read from that
//     XCD's L2 by the pair's other workgroups.
//   * A launch runs in rounds of one workgroup per CU.  The tiles of a last round that would be
//     mostly empty go to a launch of half-size workgroups behind it, or -- when the caller brings a
//     workspace -- to full-size workgroups of the same launch, 2 to 8 per 16 tiles, that each stream
//     one of as many equal runs of the pair's stages and leave (m, l, unnormalised sums) per tile,
//     which a merge launch combines (Opt-Pa Eq. 10 over the parts).
// The only difference from decode in the arithmetic is that the visible-token limit is per column
// (causal).
//
// The launch's order.  A causal stream is as long as its last row needs and one workgroup holds a
// CU, so how long a launch takes is decided by which rows a workgroup takes and in which order the
// workgroups start: tiles by row, the longest streams first, whole and split streams in one launch
// (prefill_deal.hpp).  Three fresh prompts of 301, 1039 and 1777 rows (40 over
// 8 heads, d = 128): 156 us a pass with tiles by head, first rows first and the split streams in a
// launch behind the whole ones, 100 us so; 8 x 512 rows over 8192 tokens 763 -> 744 us.
//
// A workgroup's two ends, where its CU's matrix cores idle, are latency: the rows leave through LDS in
// whole lines (straight from the registers, 16 bytes of 32 rows an instruction, the CU got its next
// workgroup 6-8 us after the stream's end, so 3), the block numbers of three stages are asked for
// before anything else, and nothing is read ahead of the stream (a pass over all v_scales for their
// largest took 3-6 us a workgroup).  Together: the three prompts 102 -> 90 us, 8 x 352 rows 92 -> 80.
#include "attn_tile.hpp"
#include "kv_quant.hpp"
#include "launch_grid.hpp"
#include "prefill_deal.hpp"

namespace coopt {

struct PrefillArgs : PrefillDeal {
    const half_t* q;
    CacheView cv;
    const int32_t* block_tables;
    const int32_t* context_lens;
    const int32_t* query_start;
    half_t* out;
    int32_t H_q, H_k, G;
    Divisor kv_heads;         // H_k
    int32_t max_blocks;
    int32_t pool_tiles;
    float scale_log2e;
    float* part;              // the split workgroups' partial rows, in the workspace
    int32_t rank_bits;        // > 0: workgroups in the order of their streams' lengths, which have so many bits (in stages)
};

constexpr int kPrefillGroupsPerStage = kPrefillStageTokens / (2 * kBlock);      // two-block groups between two barriers
constexpr int kPrefillSlots = 2 * kPrefillGroupsPerStage + 1;      // groups in LDS: two stages and one more (below)
// Groups of a stage produced by the first team (waves 0-3); the second team takes the rest.
constexpr int kPrefillFirstTeamGroups = 3;
constexpr int kPrefillFirstTeamGroupsOf8 = 1;      // of a workgroup of 8 tiles, whose first team alone consumes
constexpr float kNoReference = -1.0e30f;        // a running reference below every score
constexpr long long kPrefillXcdL2 = 4LL << 20;   // bytes of L2 per XCD

// Byte offsets inside one LDS stage (one group = blocks A and B of one KV head, 32 tokens).  Operands
// are in the order in which a 32x32x16 product takes them, lane 32h + r 16 bytes at 16 (32h + r).
template <int HEAD_DIM>
struct PrefillStage {
    static constexpr int kOps = HEAD_DIM / 16;          // operands of K, and of V
    static constexpr int kK = 0;                        // [dim / 16][h][token of the group]: dims 8h .. 8h+7
    static constexpr int kV = kOps * 1024;              // [dim / 32][u][h][dim % 32]: tokens 8u + 4h .. +3 of A, of B
    static constexpr int kS = 2 * kOps * 1024;          // 16 floats each: k_scale*c A, B; log2 v_scale A, B
    static constexpr int kF = kS + 256;                 // the factor that the 1/v_scale entries carry, undone (below)
    static constexpr int kR = kF + 16;                  // [u][h][cut, remainder] of 8 halves: 1/v_scale (below)
    static constexpr int kZero = 128;                   // of kR: 16 bytes of zeros, and again kRStride behind them
    static constexpr int kRStride = 64;
    static constexpr int kBytes = kS + 512;
};

// The weights enter the second product rounded to fp16, w~ = fp16(P * v_scale): one token's weight
// is then off by up to 2^-11 relative, which shows in the output when that token carries the row
// (an fp16 output near |x| = 3 moves by 0.7e-3).  So the row sum is taken from the SAME rounded
// weights, l = sum_j w~_j / v_scale_j: numerator and denominator then describe one softmax with
// weights perturbed by at most 2^-11 relative, whose result differs from the exact one by at most
// that times the weighted mean deviation of the value rows from the result -- nothing for one
// token or a dominant one.  The sum runs on the matrix cores: one more operand (kR) has in row 0
// 2^-8 / v_scale of the group's 32 tokens, times a power of two that the sum is freed of again, cut to
// fp16, in row 1 the remainder (the producers write both).  A 16x16x32 product takes the weight operand of
// a 32x32x16 one as it is, with columns 16..31 as further k-slots, for which the operand has the same in
// rows 2 and 3; two such products per group accumulate both tiles' sums instead of sixteen vector additions.
// Column 16 + n's weights are thus multiplied by zeros for column n, and zero times NaN is NaN: a wave that ends
// with such a sum goes over its keys once more for the sums alone, in additions that keep columns apart.  (To
// keep NaN out of the products, group by group, costs every launch 1.5 % to 4.5 % of 8 x 512 rows over 8192 tokens.)
//
// v_scale reaches the weight through the exponent: the producers leave lv = log2(v_scale) beside
// k_scale, the score of a token is z' = s * ksc + lv in
// one fused multiply-add, and the running reference m follows the maximum of z'.  The weight
// exp2(z' - m) = P * v_scale * 2^(...) then needs no multiplication of its own and is at most
// 2^(kPShift + kRescaleSlack) whatever the scales are.  A token that is not in the cache has
// lv = -inf and so the weight 0.
// ---- The two tiles of a wave as ONE tile of 32 columns (lane 32h + c: column c, tile c / 16), for
// 32x32x16 products.  S^T[token][col]: row = token of the group, so lane (c, h) has the scores of
// tokens 8j + 4h + 0..3 (j = 0, 1 of block A, 2, 3 of B) in registers 4j ..; as k-slots of
// O^T[dim][col] += V^T P^T product u takes registers 4u .. and 8 + 4u ..: tokens 8u + 4h of A and of B.
__device__ __forceinline__ floatx16 mfma_32x32x16(half8_t a, half8_t b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// z = s * ksc + lv of four tokens (registers 4j ..), and their maximum.
template <bool TAIL>
__device__ __forceinline__ float wide_logits(floatx16& z, int j, floatx4 ksc, floatx4 lv, int vis)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float x = __builtin_fmaf(z[4 * j + i], ksc[i], lv[i]);
        z[4 * j + i] = TAIL ? (i < vis ? x : -INFINITY) : x;       // (a select also drops a NaN score)
    }
    return fmaxf(fmaxf(z[4 * j], z[4 * j + 1]), fmaxf(z[4 * j + 2], z[4 * j + 3]));
}

// Two weights, registers k and k + 1 of z, rounded to fp16 (one instruction, as cutting them is: errors
// against 64 bits of 2.5e-4 to 2.9e-4 of the norm instead of 2.9e-4 to 3.2e-4).
__device__ __forceinline__ half2_t wide_weights(const floatx16& z, int k, float mm)
{
    return half2_t{(half_t)__builtin_amdgcn_exp2f(z[k] - mm), (half_t)__builtin_amdgcn_exp2f(z[k + 1] - mm)};
}
// The same from scores that are not scaled yet (an fp16 cache: one factor for all tokens).
__device__ __forceinline__ half2_t wide_weights(const floatx16& s, int k, float scale, float mm)
{
    return half2_t{(half_t)__builtin_amdgcn_exp2f(__builtin_fmaf(s[k], scale, -mm)),
                   (half_t)__builtin_amdgcn_exp2f(__builtin_fmaf(s[k + 1], scale, -mm))};
}

// TILES: of a workgroup, 16 or, where a pair has no more, 8 (whose first four waves alone consume).
template <int HEAD_DIM, int KV, int TILES, bool BIG>
__global__ void __launch_bounds__(64 * kPrefillWaves, 2)
prefill_chunk_kernel(const PrefillArgs a)
{
    using St = PrefillStage<HEAD_DIM>;
    constexpr bool FP8 = kIsFp8<KV>;
    constexpr int NL = BlockRegs<HEAD_DIM, KV>::NL;   // 16-byte pieces per lane of a K (or V) tile
    constexpr int NLH = (NL + 1) / 2;                 // V pieces per V wave
    constexpr int NP = NL > 2 * NLH ? NL : 2 * NLH;   // producer registers per wave
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];     // kPrefillSlots groups

    const int lane = threadIdx.x & 63;
    const int wave_id = wave_uniform((int)(threadIdx.x >> 6));
    const int wave = wave_id & 3;                      // producer role inside its team
    const int team = wave_id >> 2;                     // which groups of a stage it produces: below
    const int n = lane & 15, grp = lane >> 4;
    int pair, turn, qs, C, t;
    if (a.rank_bits > 0) {
        // Lane p: the XCD's p-th pair.  The stream length (in stages) of the workgroup that I am in the
        // order of all pairs' items by length, bit by bit; then which of the items of that length.
        const int my_pair = 8 * lane + (int)(blockIdx.x & 7), rank = blockIdx.x >> 3;
        const bool there = lane < a.xcd_pairs && my_pair < a.num_pairs;
        const int my_seq = there ? a.kv_heads.quotient(my_pair) : 0;
        const int my_qs = a.query_start[my_seq], my_C = there ? a.query_start[my_seq + 1] - my_qs : 0;
        const int my_t = a.context_lens[my_seq];
        const PairItems items(a, my_t, my_C, a.G, TILES);
        const int stages = stages_of_rank(rank, a.rank_bits, [&](int l) { return wave_total(items.at_least(l)); });
        if (stages == 0) return;                                   // fewer items than workgroups
        const int longer = items.at_least(stages + 1), here = items.at_least(stages) - longer;
        const int behind = rank - wave_total(longer);              // among the items of this length
        const int before = wave_inclusive_scan(here) - here;
        const unsigned long long mine = __builtin_amdgcn_ballot_w64(behind >= before && behind < before + here);
        if (mine == 0) return;                                     // (a length beyond what the block table holds)
        const int it = __builtin_ctzll(mine);
        const int my_turn = items.turn(stages, behind - before);
        pair = 8 * it + (int)(blockIdx.x & 7);
        turn = __builtin_amdgcn_readlane(my_turn, it);
        qs = __builtin_amdgcn_readlane(my_qs, it);
        C = __builtin_amdgcn_readlane(my_C, it);
        t = __builtin_amdgcn_readlane(my_t, it);
    } else {
        pair = prefill_pair(a, blockIdx.x, turn);
        if (pair >= a.num_pairs) return;
        const int seq = a.kv_heads.quotient(pair);
        qs = a.query_start[seq];
        C = a.query_start[seq + 1] - qs;
        t = a.context_lens[seq];
        if (C <= 0) return;
    }
    const int seq = a.kv_heads.quotient(pair);
    const int g = pair - seq * a.H_k;
    const int t_ctx = t - C;
    const int tiles_per_head = (C + 15) / 16;
    const int total_tiles = a.G * tiles_per_head;
    const PrefillShare share = prefill_share(a, turn, t, C, total_tiles);
    const bool whole = share.parts == 1 || prefill_runs_whole(a, t);
    if (whole && share.part > 0) return;
    const int block = share.block, parts = whole ? 1 : share.parts, part = share.part;
    if (share.base + block * TILES >= share.end) return;    // the whole workgroup leaves together
    TileOrder order(tiles_per_head, share.base, share.end);
    order.to_scalar();
    constexpr int NR = 2;                              // tiles of a wave: its 32 columns
    const int first = block * TILES + wave_id * NR;    // position of my first tile
    const int count = order.count();
    const bool active = wave_id * NR < TILES && first < count;     // a wave without tiles still produces

    constexpr int NQ = HEAD_DIM / 16;                  // q operands
    // Lane r works out tile r of the wave, lane NR the workgroup's last, which sees furthest.
    int tile_row, tile_head;
    order.at(lane < NR ? min(first + lane, count - 1)             // surplus tiles repeat the last
                       : min((block + 1) * TILES, count) - 1, tile_row, tile_head);
    const int wg_max = t_ctx + min(16 * __builtin_amdgcn_readlane(tile_row, NR) + 15, C - 1) + 1;
    const int nblk = (wg_max + kBlock - 1) / kBlock;
    const int num_groups = (nblk + 1) >> 1;
    const int32_t* bt = a.block_tables + (size_t)seq * a.max_blocks;
    // A stage holds GPS consecutive groups; one barrier per stage.  The workgroup streams stages
    // s_lo .. s_hi-1: all of them, or one of `parts` equal runs in a split launch (an empty run
    // leaves the neutral partial m = kNoReference, l = 0).
    constexpr int GPS = kPrefillGroupsPerStage;
    const int num_stages = (num_groups + GPS - 1) / GPS;
    const int s_lo = parts == 1 ? 0 : wave_uniform(quotient(num_stages * part, parts));
    const int s_hi = parts == 1 ? num_stages : wave_uniform(quotient(num_stages * (part + 1), parts));
    const int g_end = min(num_groups, s_hi * GPS);            // groups below this one are mine

    // (finite, not -inf: a workgroup that streams a later run of a pair's stages meets columns that
    // see none of a group's tokens before any they do see, and the weights exp2(z - m) of such a
    // column must come out as exp2(-inf) = 0, not exp2(-inf + inf))
    float m = kNoReference;
    // the row sums / 2^8, in lanes 0..15: rows 0 and 1 (registers 0 and 1) of column n, 2 and 3 of 16 + n
    floatx4 lacc = {0.f, 0.f, 0.f, 0.f};
    floatx16 acc[HEAD_DIM / 32];
#pragma unroll
    for (int c = 0; c < HEAD_DIM / 32; ++c) acc[c] = floatx16{};

    // ---- which team produces which group of a stage.  The two waves of a SIMD do not get equal
    // shares of it: the older one (a wave of the first team) is through with a stage's groups well
    // before the younger one, so the first team produces more of the next stage.
    constexpr int kFirst = TILES == 8 ? kPrefillFirstTeamGroupsOf8 : kPrefillFirstTeamGroups;           // sub-groups 0 .. kFirst-1: team 0
    constexpr int kOwn = kFirst > GPS - kFirst ? kFirst : GPS - kFirst;   // most groups a wave holds
    static_assert(kFirst >= 1 && kFirst <= GPS, "the first team produces at least one group");
    auto owner = [](int sub) { return sub < kFirst ? 0 : 1; };
    auto own_index = [](int sub) { return sub < kFirst ? sub : sub - kFirst; };
    // ---- block numbers: lane 2i + b fetches the number of block b of the team's i-th group, in ONE
    // vector load per stage that is issued a whole stage before the tile loads it serves and ahead
    // of the tile loads of the stage before (the vector-memory counter is in order: by the time
    // those tiles have been waited for, the numbers are back).  Fetched where they are needed --
    // through the scalar unit or not -- their latency sat between two tile loads and again in
    // front of the barrier, every stage.
    const __amdgpu_buffer_rsrc_t bt_rsrc = TileLoader<HEAD_DIM, KV, BIG>::rsrc(bt, a.max_blocks * 4);
    auto load_ids = [&](int stage) {
        const int p = stage * GPS + (team == 0 ? 0 : kFirst) + (lane >> 1);
        const int b = min(2 * p + (lane & 1), nblk - 1);
        return __builtin_amdgcn_raw_buffer_load_b32(bt_rsrc, lane < 2 * kOwn ? 4 * b : 0, 0, 0);
    };
    auto id_of = [&](uint32_t ids, int i, int b) { return __builtin_amdgcn_readlane((int)ids, 2 * i + b); };
    // (the first three stages' at once, ahead of everything that a wave asks for: the first tiles wait
    // for nothing else)
    uint32_t ids = load_ids(s_lo), ids_second = load_ids(s_lo + 1), ids_next = load_ids(s_lo + 2);

    // ---- the queries
    half8_t qop[NQ];
    int row0_of[NR], head_of[NR];      // of my tiles: first row, head of the group
    int my_max = 0, min_row = 0x7fffffff;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        head_of[r] = __builtin_amdgcn_readlane(tile_head, r);
        row0_of[r] = 16 * __builtin_amdgcn_readlane(tile_row, r);
        my_max = max(my_max, t_ctx + min(row0_of[r] + 15, C - 1) + 1);
        min_row = min(min_row, row0_of[r]);
    }
    // (columns 16r .. are tile r's; surplus rows repeat row C-1)
    const bool second = grp & 1;
    const int h = grp >> 1;                    // lane 32h + c: column c
    const int my_row = min((second ? row0_of[NR - 1] : row0_of[0]) + n, C - 1);
    const int limit = t_ctx + my_row + 1;      // tokens visible to this lane's column
    const half_t* qrow = a.q + ((size_t)(qs + my_row) * a.H_q + g * a.G + (second ? head_of[NR - 1] : head_of[0])) * HEAD_DIM +
                         8 * h;
#pragma unroll
    for (int m = 0; m < NQ; ++m) qop[m] = *reinterpret_cast<const half8_t*>(qrow + 16 * m);
    if (!active) my_max = 0;
    // (a negative softmax scale is the queries' sign: the scores' factor is not negative then)
    const float scale = fabsf(a.scale_log2e);
    if (a.scale_log2e < 0.0f) {
#pragma unroll
        for (int m = 0; m < NQ; ++m) qop[m] = -qop[m];
    }

    // ---- producer side: this wave's pieces of group p
    const TileLoader<HEAD_DIM, KV, BIG> loader(a.cv, lane, a.pool_tiles);
    u32x4 prs[kOwn][NP];
    float pscs[kOwn];
    // The four producer roles of a team -- 0: K of block A, 1: K of block B, 2 and 3: the two halves
    // of the V pieces of both blocks (and the v_scale work of block A, B).  A V role costs twice a
    // K role (890 against 440 cycles per group).  The two teams take the roles crosswise: waves w
    // and w + 4 share a SIMD, so with the second team's roles shifted by two every SIMD carries
    // one K role and one V role (1 % faster than the same roles in both teams; shifts of one or
    // three, and rotating the roles from group to group inside a team, were slower).
    float norm = 0x1p126f;                             // of the v_scales (below): the first one lowers it
    const int my_token = 4 * grp + (n & 3);            // of a block: whose scales this lane takes
    // (v_scale: of block A where n < 8, of B otherwise; 1 / v_scale cut to fp16, or with n & 4 the rest)
    const int r_entry = (grp >> 1) * St::kRStride + 32 * (grp & 1) + 16 * ((n >> 2) & 1) + 8 * (n >> 3) + 2 * (n & 3);
    auto role_of = [&](int) { return (wave + 2 * team) & 3; };
    auto produce_issue = [&](int p, int blockA, int blockB, u32x4 (&pr)[NP], float& psc) {
        const int role = role_of(p);
        const int vj0 = role == 2 ? 0 : NLH;               // first V piece of a V role
        const int vcnt = role == 2 ? NLH : NL - NLH;       // and how many it brings
        const bool okA = 2 * p < nblk, okB = 2 * p + 1 < nblk;
        const int tA = blockA * a.H_k + g;
        const int tB = blockB * a.H_k + g;
        // (one comparison for "is my block there": a choice between the two flags okA and okB
        // would be made in vector registers, the very ones the loads issued a moment ago will
        // fill, and cost a wait for those loads)
        const int mine = role & 1;                         // roles 0, 2: block A; roles 1, 3: block B
        const bool ok_mine = 2 * p + mine < nblk;
        const int t_mine = mine ? tB : tA;
        if (role < 2) {
            // (ahead of the pieces: its address is made in vector registers, and one that a load will fill is
            // waited for; an absent B's scales are A's, which nobody looks at)
            if constexpr (FP8)
                psc = loader.load_scale_of(role == 0 ? a.cv.k_scale : a.cv.v_scale, n >= 8 && okB ? tB : tA, my_token);
#pragma unroll
            for (int j = 0; j < NL; ++j) pr[j] = loader.load_piece(a.cv.k_cache, t_mine, j, ok_mine);
        } else {
#pragma unroll
            for (int jj = 0; jj < NLH; ++jj) {
                if (jj < vcnt) {
                    pr[2 * jj] = loader.load_piece(a.cv.v_cache, tA, vj0 + jj, okA);
                    pr[2 * jj + 1] = loader.load_piece(a.cv.v_cache, tB, vj0 + jj, okB);
                }
            }
        }
    };
    auto produce_store = [&](int p, unsigned char* st, const u32x4 (&pr)[NP], float psc) {
        const int role = role_of(p);
        const int vj0 = role == 2 ? 0 : NLH;
        const int vcnt = role == 2 ? NLH : NL - NLH;
        if (role < 2) {
            // (a one-byte piece: dims 16 (4j + grp) .. +15 of token n, both h; an fp16 one: 8 dims)
            unsigned char* kdst = st + St::kK + 16 * (16 * role + n) +
                                  (FP8 ? 1024 * grp : 1024 * (grp >> 1) + 512 * (grp & 1));
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                if constexpr (FP8) {
                    *reinterpret_cast<half8_t*>(kdst + j * 4096) = fp8x8_to_half8<KV>(pr[j].x, pr[j].y);
                    *reinterpret_cast<half8_t*>(kdst + j * 4096 + 512) = fp8x8_to_half8<KV>(pr[j].z, pr[j].w);
                } else {
                    *reinterpret_cast<u32x4*>(kdst + j * 2048) = pr[j];
                }
            }
            if constexpr (FP8) {
                float* dst = reinterpret_cast<float*>(st + St::kS + 128 * role + 64 * (n >> 3) + 4 * my_token);
                if (role == 0) {
                    if ((n & 4) == 0) *dst = psc * scale;
                } else {
                    // The group's v_scales, one token a lane: the logarithms, and the entries of the row-sum
                    // operands, 2^-8 / v_scale cut to fp16 and the remainder (an entry: four tokens of block A,
                    // the same of B).  Scales may be of any magnitude (an E5M2 cache's are 2^-7 of an E4M3
                    // cache's, small value rows' smaller still) and fp16 holds five bits of exponent, so the
                    // entries are taken times a power of two, 1 over the one just above the largest scale so
                    // far, which the group's row sums are multiplied by again: both are exact.
                    const bool there = my_token + (n >= 8 ? kBlock : 0) < t - 32 * p;      // (else a stale scale)
                    const float vs = there ? psc : 0.0f;
                    if ((n & 4) == 0) *dst = __builtin_amdgcn_logf(vs);                    // log2; -inf: absent
                    // (kept from group to group: one vote in the place of a reduction, but where a scale is
                    // larger than all before it)
                    if (__builtin_amdgcn_ballot_w64(vs * norm > 1.0f) != 0) {
                        // largest = f * 2^e, f in [1, 2): norm = 2^-(e+1)
                        const uint32_t ebits = (__builtin_bit_cast(uint32_t, wave_max(fmaxf(vs, 0.0f))) >> 23) & 0xffu;
                        if (ebits > 0u && ebits < 253u) norm = __builtin_bit_cast(float, (253u - ebits) << 23);
                    }
                    if (lane == 0) *reinterpret_cast<float*>(st + St::kF) = norm;
                    // (the hardware reciprocal, 1 ulp: far inside what the fp16 pair keeps)
                    const float r = fminf(vs > 0.0f ? 0.00390625f * __builtin_amdgcn_rcpf(vs * norm) : 0.0f, 65504.0f);
                    const float hi = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, r) & 0xffffe000u);
                    *reinterpret_cast<half_t*>(st + St::kR + r_entry) = (half_t)((n & 4) ? r - hi : hi);
                }
            }
        } else {
            unsigned char* vdst = st + St::kV + 512 * grp + 16 * n;       // dim n of the first 32, tokens 4 grp ..
            // this lane's 4 tokens of block A start at 32p + 4grp, of block B 16 later
            const int cacheA = t - (32 * p + 4 * grp), cacheB = cacheA - kBlock;
            uint32_t a0 = 0xffffffffu, a1 = 0xffffffffu, b0 = 0xffffffffu, b1 = 0xffffffffu;
            if (32 * p + 2 * kBlock > t) {          // wave-uniform: only the cache's last group
                token_masks<KV>(cacheA, a0, a1);
                token_masks<KV>(cacheB, b0, b1);
            }
#pragma unroll
            for (int jj = 0; jj < NLH; ++jj) {
                if (jj < vcnt) {
                    if constexpr (FP8) {
                        const u32x4 wa = pr[2 * jj] & a0, wb = pr[2 * jj + 1] & b0;
#pragma unroll
                        for (int cc = 0; cc < 4; ++cc) {
                            const half4_t va = fp8x4_to_half4<KV>(wa[cc]), vb = fp8x4_to_half4<KV>(wb[cc]);
                            *reinterpret_cast<half8_t*>(vdst + (2 * (vj0 + jj) + (cc >> 1)) * 2048 + (cc & 1) * 256) =
                                half8_t{va[0], va[1], va[2], va[3], vb[0], vb[1], vb[2], vb[3]};
                        }
                    } else {
                        const u32x4 wa = pr[2 * jj] & u32x4{a0, a1, a0, a1};
                        const u32x4 wb = pr[2 * jj + 1] & u32x4{b0, b1, b0, b1};
                        *reinterpret_cast<u32x4*>(vdst + (vj0 + jj) * 2048) =
                            u32x4{wa.x, wa.y, wb.x, wb.y};
                        *reinterpret_cast<u32x4*>(vdst + (vj0 + jj) * 2048 + 256) =
                            u32x4{wa.z, wa.w, wb.z, wb.w};
                    }
                }
            }
        }
    };

    // ---- consumer side
    const int full_limit = min(t, t_ctx + min_row + 1);   // tokens visible to every column of mine
    auto op = [&](const unsigned char* st, int at) { return *reinterpret_cast<const half8_t*>(st + at + 16 * lane); };
    auto scales = [&](const unsigned char* st, int at) { return *reinterpret_cast<const floatx4*>(st + St::kS + at); };
    // My row-sum operand: the cut reciprocals and the rest of tokens 8u + 4h .. are rows 0 and 1 in the lanes
    // of columns 0..15 (grp even), rows 2 and 3 in those of columns 16..31; zeros elsewhere.
    const int r_of = (n >> 1) == (grp & 1) ? 32 * h + 16 * (n & 1) : St::kZero;
    auto r_op = [&](const unsigned char* st, int u) {
        return *reinterpret_cast<const half8_t*>(st + St::kR + u * St::kRStride + r_of);
    };
    auto norm_of = [&](const unsigned char* st) { return FP8 ? *reinterpret_cast<const float*>(st + St::kF) : 1.0f; };
    // raises the reference of this lane's column where a score of the group exceeds it
    auto raise = [&](float bm) {
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(bm > m + kRescaleSlack) == 0, 1)) return;   // wave-uniform
        float nm = fmaxf(bm, __shfl_xor(bm, 32));
        nm = fmaxf(nm, m);
        const float alpha = __builtin_amdgcn_exp2f(m - nm);   // m = kNoReference at the start gives 0
        const float other = __shfl(alpha, 16 + n);             // (column 16 + n's)
        lacc *= floatx4{alpha, alpha, other, other};
#pragma unroll
        for (int c = 0; c < HEAD_DIM / 32; ++c) acc[c] *= alpha;
        m = nm;
    };
    auto consume = [&](const unsigned char* st, int gi) {
        const int baseA = 2 * gi * kBlock;
        const bool tail = baseA + 2 * kBlock > full_limit;        // (a missing block B is beyond every limit)
        floatx16 z = {};
#pragma unroll
        for (int k = 0; k < NQ; ++k) z = mfma_32x32x16(op(st, St::kK + 1024 * k), qop[k], z);
        float bm = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            floatx4 ksc = {scale, scale, scale, scale}, lv = {0.f, 0.f, 0.f, 0.f};
            if constexpr (FP8) {
                ksc = scales(st, 32 * j + 16 * h);
                lv = scales(st, 128 + 32 * j + 16 * h);
            }
            bm = fmaxf(bm, tail ? wide_logits<true>(z, j, ksc, lv, limit - baseA - 8 * j - 4 * h)
                                : wide_logits<false>(z, j, ksc, lv, 0));
        }
        raise(bm);
        const float mm = m - kPShift;
        floatx4 sum = FP8 ? floatx4{} : lacc;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            half8_t pop;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const half2_t w = wide_weights(z, 4 * u + 2 * (i & 1) + 8 * (i >> 1), mm);
                pop[2 * i] = w.x;
                pop[2 * i + 1] = w.y;
            }
            sum = mfma_16x16x32(r_op(st, u), pop, sum);
#pragma unroll
            for (int c = 0; c < HEAD_DIM / 32; ++c)
                acc[c] = mfma_32x32x16(op(st, St::kV + 2048 * c + 1024 * u), pop, acc[c]);
        }
        lacc = FP8 ? lacc + sum * norm_of(st) : sum;
    };
    // Groups live in a ring of slots; `ring` is that of stage si's first group.
    int ring = 0;
    auto slot = [&](int sub) {                                // of group `sub` counted from there, 0 .. 2 GPS - 1
        const int x = ring + sub;
        return lds + (x >= kPrefillSlots ? x - kPrefillSlots : x) * St::kBytes;
    };
    auto next_stage = [&]() { ring = ring + GPS >= kPrefillSlots ? ring + GPS - kPrefillSlots : ring + GPS; };
    // (a wave keeps registers for the sub-groups of its own team)
    auto issue_first_stage = [&]() {
#pragma unroll
        for (int sub = 0; sub < GPS; ++sub)
            if (owner(sub) == team && s_lo * GPS + sub < g_end)
                produce_issue(s_lo * GPS + sub, id_of(ids, own_index(sub), 0), id_of(ids, own_index(sub), 1),
                              prs[own_index(sub)], pscs[own_index(sub)]);
    };
    // the zeros of every slot's row-sum operands; over an fp16 cache the others as well (every scale is 1)
    if (threadIdx.x < 16 * kPrefillSlots) {
        const int of = threadIdx.x & 15;                                   // 16 bytes of the 256 at kR
        const bool zero = of == St::kZero / 16 || of == (St::kZero + St::kRStride) / 16;
        const uint32_t w = zero || (of & 1) ? 0u : 0x1c001c00u;            // 2^-8, and no remainder
        if (zero || (!FP8 && of < St::kZero / 16))
            *reinterpret_cast<u32x4*>(lds + (threadIdx.x >> 4) * St::kBytes + St::kR + 16 * of) = u32x4{w, w, w, w};
    }
    issue_first_stage();
#pragma unroll
    for (int sub = 0; sub < GPS; ++sub)
        if (owner(sub) == team && s_lo * GPS + sub < g_end)
            produce_store(s_lo * GPS + sub, slot(sub), prs[own_index(sub)], pscs[own_index(sub)]);
#pragma unroll
    for (int sub = 0; sub < GPS; ++sub)
        if (owner(sub) == team && (s_lo + 1) * GPS + sub < g_end)
            produce_issue((s_lo + 1) * GPS + sub, id_of(ids_second, own_index(sub), 0), id_of(ids_second, own_index(sub), 1),
                          prs[own_index(sub)], pscs[own_index(sub)]);
    __syncthreads();
    // The producers' part of stage si's turn, one of the team's groups at a time: the next stage's to LDS,
    // the one after that asked for.
    uint32_t ids_use = 0;
    auto produce = [&](int si, int i) {
        const int sub = team == 0 ? i : kFirst + i;
        if (sub >= GPS || (team == 0 && i >= kFirst)) return;
        const int gn = (si + 1) * GPS + sub;
        if (gn < g_end) produce_store(gn, slot(GPS + sub), prs[i], pscs[i]);
        if (i == 0) {
            // (ahead of the tile loads: by the time those are waited for, the numbers are back)
            ids_use = ids_next;
            ids_next = load_ids(si + 3);
        }
        if (gn + GPS < g_end) {
            const int bA = id_of(ids_use, i, 0), bB = id_of(ids_use, i, 1);
            produce_issue(gn + GPS, bA, bB, prs[i], pscs[i]);
        }
    };
    // Stages of tokens that every column of mine sees run as a pipeline over their groups, so that the
    // vector ALU has work under every product: the score products of a group run beside the
    // exponentials of half the tokens of the group before it, that group's value products over those
    // tokens beside the other half's exponentials, and over the other half beside the new group's
    // multiply-adds and maxima; the order is pinned by scheduling fences.  Operands are asked for half a
    // group's products ahead, in the registers that the ones just used leave.  The pipeline does not
    // drain at a stage's end: the barrier behind which the next stage may be read stands in front of the
    // stage's last group, and that group's slot is the ring's spare one -- until the next barrier nobody
    // writes to it.
    constexpr int W = NQ / 2;                                  // operands in flight
    constexpr int PER = 8 / NQ;                                // d = 64 has half as many products for the same vector work
    const int h16 = 16 * h;
    half8_t ops[W];
    floatx16 z;
    auto k_op = [&](const unsigned char* st, int k) { return op(st, St::kK + 1024 * k); };
    auto v_op = [&](const unsigned char* st, int u, int c) { return op(st, St::kV + 2048 * c + 1024 * u); };
    // The scores of four tokens scaled, and their maximum.  An fp16 cache's are left as they are (the
    // exponentials' multiply-adds scale them), its maximum scaled behind: the factor is not negative.
    auto ksc_of = [&](const unsigned char* st, int j) { return FP8 ? scales(st, 32 * j + h16) : floatx4{}; };
    auto lv_of = [&](const unsigned char* st, int j) { return FP8 ? scales(st, 128 + 32 * j + h16) : floatx4{}; };
    auto logits = [&](floatx16& x, int j, floatx4 ksc, floatx4 lv) {
        if constexpr (FP8) return wide_logits<false>(x, j, ksc, lv, 0);
        else return fmaxf(fmaxf(x[4 * j], x[4 * j + 1]), fmaxf(x[4 * j + 2], x[4 * j + 3]));
    };
    auto top = [&](float bm) { return FP8 ? bm : bm * scale; };
    auto pipeline_start = [&]() {                              // scores of the first group; K operands of the second
        const unsigned char* st = slot(0);
        floatx4 ksc[4], lv[4];
        z = floatx16{};
#pragma unroll
        for (int k = 0; k < W; ++k) ops[k] = k_op(st, k);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            ksc[j] = ksc_of(st, j);
            lv[j] = lv_of(st, j);
        }
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            z = mfma_32x32x16(ops[k % W], qop[k], z);
            ops[k % W] = k < W ? k_op(st, k + W) : k_op(slot(1), k - W);
        }
        float bm = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4; ++j) bm = fmaxf(bm, logits(z, j, ksc[j], lv[j]));
        raise(top(bm));
    };
    auto pipeline_stage = [&](int si, bool more) {            // more: the stage behind this one is such a stage, too
        static_assert(kOwn < GPS, "a stage is in LDS before the last group of the one in front of it");
#pragma unroll
        for (int sub = 0; sub < GPS; ++sub) {
            const unsigned char* st = slot(sub);
            const unsigned char* sn = slot(sub + 1);
            const float mm = m - kPShift;
            half8_t pop[2];
            floatx16 zn = {};
            floatx4 ksc, lv;
            half8_t rop;
            floatx4 sum;
            float norm;
            auto weights = [&](int u, int i) {                 // tokens 8u + 4h .. of block A, then of B
                const int x = 4 * u + 2 * (i & 1) + 8 * (i >> 1);
                const half2_t w = FP8 ? wide_weights(z, x, mm) : wide_weights(z, x, scale, mm);
                pop[u][2 * i] = w.x;
                pop[u][2 * i + 1] = w.y;
            };
            if (sub == GPS - 1) {
                __syncthreads();                               // stage si+1 is complete, and nobody reads stage si but for this group
#pragma unroll
                for (int k = 0; k < W; ++k) ops[k] = k_op(sn, k);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int k = 0; k < NQ; ++k) {
                zn = mfma_32x32x16(ops[k % W], qop[k], zn);
                ops[k % W] = k < W ? k_op(sn, k + W) : v_op(st, 0, k - W);
                if (k == NQ - 1) rop = r_op(st, 0);
#pragma unroll
                for (int e = 0; e < PER; ++e)
                    if ((PER * k + e) & 1) weights(0, (PER * k + e) >> 1);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int c = 0; c < W; ++c) {
                if (c == 0) {
                    sum = mfma_16x16x32(rop, pop[0], FP8 ? floatx4{} : lacc);
                    rop = r_op(st, 1);
                    norm = norm_of(st);
                }
                acc[c] = mfma_32x32x16(ops[c], pop[0], acc[c]);
                ops[c] = v_op(st, 1, c);
                if (c == W - 1) {
                    ksc = ksc_of(sn, 0);
                    lv = lv_of(sn, 0);
                }
#pragma unroll
                for (int e = 0; e < PER; ++e) weights(1, PER * c + e);
                __builtin_amdgcn_sched_barrier(0);
            }
            float bm = -INFINITY;
#pragma unroll
            for (int c = 0; c < W; ++c) {
                if (c == 0) sum = mfma_16x16x32(rop, pop[1], sum);
                acc[c] = mfma_32x32x16(ops[c], pop[1], acc[c]);
                if (sub != GPS - 2) ops[c] = k_op(slot(sub + 2), c);
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                    const int j = PER * c + e;
                    bm = fmaxf(bm, logits(zn, j, ksc, lv));
                    if (j < 3) {
                        ksc = ksc_of(sn, j + 1);
                        lv = lv_of(sn, j + 1);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            lacc = FP8 ? lacc + sum * norm : sum;
            if (sub < kOwn) produce(si, sub);
            if (sub < GPS - 1 || more) raise(top(bm));
            z = zn;
        }
    };

    // Whole stages that all my columns see, then the others group by group.  (Two loops, not a branch
    // in one: the pipeline leaves no registers for what the two forms would share.  Waves may change
    // over at different stages; each passes one barrier per stage.)
    int si = s_lo;
    const int whole_stages = min(active ? min(g_end, full_limit / (2 * kBlock)) / GPS : 0, s_hi);
    if (si < whole_stages) {
        pipeline_start();
        for (; si < whole_stages; ++si) {
            pipeline_stage(si, si + 1 < whole_stages);
            next_stage();
        }
    }
    for (; si < s_hi; ++si) {
#pragma unroll 1
        for (int gi = si * GPS; gi < min((si + 1) * GPS, g_end) && 2 * gi * kBlock < my_max; ++gi)
            consume(slot(gi - si * GPS), gi);
#pragma unroll
        for (int i = 0; i < kOwn; ++i) produce(si, i);
        __syncthreads();                                       // stage si+1 is complete, and nobody reads stage si
        next_stage();
    }

    if (!active) return;
    // the sums of the lane's column: rows 0 and 1 of lacc, rows 2 and 3 for columns 16..31
    const float sum_a = __shfl(lacc[0] + lacc[1], n), sum_b = __shfl(lacc[2] + lacc[3], n);
    // (a NaN weight in either column of a lane is in all four of its registers; asked of those, not of the
    // sums, whose way through LDS the hot path need not wait for here)
    const bool once_more = __builtin_amdgcn_ballot_w64(lacc[0] != lacc[0]) != 0;
    float again = 0.0f;
    if (__builtin_expect(once_more, 0)) {
        // The weights once more, under the last reference, straight from the cache: lane 32h + r brings token r of a
        // group, dims 16k + 8h ..
        // (The launch's arguments, and what follows from them, once more, too: kept through the stream they push its
        // scalars out of their registers, 1.5 % of three fresh prompts.)
        const PrefillArgs* args = (const PrefillArgs*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        const PrefillArgs& a = *args;
        const int* bt = a.block_tables + (size_t)a.kv_heads.quotient(pair) * a.max_blocks;
        const int stages = (((nblk + 1) >> 1) + GPS - 1) / GPS;
        constexpr int ES = FP8 ? 1 : 2;
        const float mm = m - kPShift, scale = fabsf(a.scale_log2e);
#pragma unroll 1
        for (int gi = parts == 1 ? 0 : quotient(stages * part, parts) * GPS; gi < g_end && 2 * gi * kBlock < my_max; ++gi) {
            auto tile_of = [&](int b) {                        // (no read beyond the table or the pool)
                const int tile = bt[min(min(2 * gi + b + 1, nblk), a.max_blocks) - 1] * a.H_k + g;
                return (uint32_t)tile < (uint32_t)a.pool_tiles ? tile : 0;
            };
            const uint8_t* row = a.cv.k_cache + (size_t)tile_of((lane >> 4) & 1) * (kBlock * HEAD_DIM * ES) + 16 * n;
            floatx16 z = {};
#pragma unroll
            for (int k = 0; k < NQ; ++k) {
                half8_t kop;
                if constexpr (FP8) {
                    const uint2 x = *reinterpret_cast<const uint2*>(row + 256 * k + 8 * h);
                    kop = fp8x8_to_half8<KV>(x.x, x.y);
                } else {
                    kop = *reinterpret_cast<const half8_t*>(row + 512 * k + 256 * h);
                }
                z = mfma_32x32x16(kop, qop[k], z);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const size_t at = (size_t)tile_of(j >> 1) * kBlock + 8 * (j & 1) + 4 * h;
                const int vis = limit - 2 * gi * kBlock - 8 * j - 4 * h;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float vs = FP8 ? a.cv.v_scale[at + i] : 1.0f;
                    const float x = FP8 ? __builtin_fmaf(z[4 * j + i], a.cv.k_scale[at + i] * scale, __builtin_amdgcn_logf(vs))
                                        : z[4 * j + i] * scale;
                    const float w = (float)(half_t)__builtin_amdgcn_exp2f(x - mm);
                    again += i < vis ? (vs > 0.0f ? w * __builtin_amdgcn_rcpf(vs) : w * 0.0f) : 0.0f;
                }
            }
        }
        again += __shfl_xor(again, 32);
    }
    const float L = once_more ? again : (second ? sum_b : sum_a) * 256.0f;
    // The rows leave through LDS, so that a store instruction writes whole rows: a lane's registers are
    // 4 dims of 8 each (register 4j + i of acc[c]: dim 32c + 8j + 4h + i),
    // 16 bytes of 32 rows an instruction.  Every wave has a slot of its own: of the last stage only its
    // last group can still be read by others, and that is the ring's ninth.
    const int col = lane & 31;
    unsigned char* mine = slot(wave_id);
    static_assert(2 * GPS >= kPrefillWaves && 32 * (4 * HEAD_DIM + 16) <= St::kBytes, "a wave's rows fit its slot");
    // (the 2^kPShift common to acc and l cancels)
    if (parts > 1) {
        // this run's share of the tiles: reference, row sum and unnormalised sums per column
        constexpr int kRow = 4 * HEAD_DIM + 16;
#pragma unroll
        for (int c = 0; c < HEAD_DIM / 32; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *reinterpret_cast<floatx4*>(mine + col * kRow + 4 * (32 * c + 8 * j + 4 * h)) =
                    floatx4{acc[c][4 * j], acc[c][4 * j + 1], acc[c][4 * j + 2], acc[c][4 * j + 3]};
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            if (first + r >= count) break;
            float* dst = a.part + (((size_t)pair * a.tail_cap + head_of[r] * tiles_per_head + row0_of[r] / 16 - share.base) * parts + part) * (16 * (HEAD_DIM + 2));
            if (h == 0 && col >> 4 == r) {
                dst[n] = m;
                dst[16 + n] = L;
            }
#pragma unroll
            for (int at = 4 * lane; at < 16 * HEAD_DIM; at += 256)
                *reinterpret_cast<floatx4*>(dst + 32 + at) = *reinterpret_cast<const floatx4*>(
                    mine + (16 * r + at / HEAD_DIM) * kRow + 4 * (at % HEAD_DIM));
        }
        return;
    }
    constexpr int kRow = 2 * HEAD_DIM + 16;
    const float inv = 1.0f / L;
#pragma unroll
    for (int c = 0; c < HEAD_DIM / 32; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            half4_t o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (half_t)(acc[c][4 * j + i] * inv);
            *reinterpret_cast<half4_t*>(mine + col * kRow + 2 * (32 * c + 8 * j + 4 * h)) = o;
        }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if (first + r >= count) break;
        half_t* dst = a.out + ((size_t)(qs + row0_of[r]) * a.H_q + g * a.G + head_of[r]) * HEAD_DIM;
#pragma unroll
        for (int at = 8 * lane; at < 16 * HEAD_DIM; at += 512) {
            const int rr = at / HEAD_DIM;
            if (row0_of[r] + rr < C)
                *reinterpret_cast<u32x4*>(dst + (size_t)rr * a.H_q * HEAD_DIM + at % HEAD_DIM) =
                    *reinterpret_cast<const u32x4*>(mine + (16 * r + rr) * kRow + 2 * (at % HEAD_DIM));
        }
    }
}

// Combines the parts a split launch left for every tile: with M = max_p m_p and e_p = 2^(m_p - M),
// row = sum_p A_p e_p / sum_p l_p e_p (the merge rule of the online softmax, Opt-Pa Eq. 10).
// Bound by the latency of its loads: HEAD_DIM/4 lanes take one row, a wavefront 64 / (HEAD_DIM/4)
// rows, and a lane asks for its 16 bytes of every part, all parts' references and sums, before it
// waits for any.  (One wavefront per tile, which walked the parts one after the other, took 11 us
// whatever the size; the prefill of 333 rows x 40 heads over 4096 tokens went from 82.3 to 76.6 us,
// that of three prompts of up to 1777 rows from 160.4 to 153.5 us.)
template <int HEAD_DIM>
__global__ void __launch_bounds__(256)
prefill_split_merge_kernel(const PrefillArgs a)
{
    constexpr int kPart = 16 * (HEAD_DIM + 2);          // floats per tile and part
    constexpr int LPR = HEAD_DIM / 4;                   // lanes per row
    constexpr int RPB = 256 / LPR;                      // rows per workgroup: 8 or 16
    constexpr int BPT = 16 / RPB;                       // workgroups per tile: 2 or 1
    const long long id = blockIdx.x / BPT;              // pair * tail_cap + tile
    const int n = (blockIdx.x % BPT) * RPB + threadIdx.x / LPR;      // row of the tile
    const int piece = threadIdx.x % LPR;
    const int pair = (int)(id / a.tail_cap);
    const int tile = a.tile_limit + (int)(id - (long long)pair * a.tail_cap);
    const int seq = pair / a.H_k;
    const int g = pair - seq * a.H_k;
    const int parts = a.split;
    // (a branch of its own, taken where it can decide something: behind it the loads are one round trip)
    if (a.whole_tokens > 0 && prefill_runs_whole(a, a.context_lens[seq])) return;
    // every load but the two row offsets' own lies inside the workspace whatever those say
    const float* p0 = a.part + (size_t)id * parts * kPart;
    float m[kPrefillMaxParts], l[kPrefillMaxParts];
    floatx4 x[kPrefillMaxParts];
#pragma unroll
    for (int p = 0; p < kPrefillMaxParts; ++p) {
        // (a slot past the last part loads that part again: no branch between the loads)
        const float* pp = p0 + (size_t)min(p, parts - 1) * kPart;
        m[p] = pp[n];
        l[p] = pp[16 + n];
        x[p] = *reinterpret_cast<const floatx4*>(pp + 32 + n * HEAD_DIM + 4 * piece);
    }
    const int qs = a.query_start[seq];
    const int C = a.query_start[seq + 1] - qs;
    if (C <= 0) return;
    const int tiles_per_head = (C + 15) / 16;
    if (tile >= a.G * tiles_per_head) return;           // (nobody wrote this tile's parts)
    const int hh = tile / tiles_per_head;
    const int row = (tile - hh * tiles_per_head) * 16 + n;
    if (row >= C) return;
    float M = kNoReference;                 // (a row sees at least one token: some part has a real m)
#pragma unroll
    for (int p = 0; p < kPrefillMaxParts; ++p) M = fmaxf(M, m[p]);
    float den = 0.0f;
    floatx4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < kPrefillMaxParts; ++p) {
        // (left out, not weighted by zero: a sum may be infinite, and infinity * 0 is no number.  By
        // selects: the compiler moves loads into a branch, behind the others' arrival)
        const float e = __builtin_amdgcn_exp2f(m[p] - M);
        den += p < parts ? l[p] * e : 0.0f;
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] += p < parts ? x[p][c] * e : 0.0f;
    }
    const float inv = 1.0f / den;
    half4_t h;
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = (half_t)(o[i] * inv);
    *reinterpret_cast<half4_t*>(a.out + ((size_t)(qs + row) * a.H_q + g * a.G + hh) * HEAD_DIM + 4 * piece) = h;
}

}  // namespace coopt

using namespace coopt;

extern "C" size_t coopt_prefill_workspace_bytes(const coopt_shape* sh, int32_t max_chunk_len)
{
    if (check_shape(sh) != COOPT_OK || max_chunk_len <= 0 || sh->num_seqs == 0) return 0;
    return PrefillLaunchPlan(sh, max_chunk_len, true).workspace_bytes(sh);
}

static int prefill_chunk(const void* q, const void* k_cache, const void* v_cache, const float* k_scale,
                         const float* v_scale, const int32_t* block_tables, const int32_t* context_lens,
                         const int32_t* query_start, int32_t num_query_rows, int32_t max_chunk_len,
                         void* out, void* workspace, const coopt_shape* sh, void* hip_stream);

extern "C" int coopt_paged_gqa_prefill_chunk(const void* q, const void* k_cache, const void* v_cache,
                                             const float* k_scale, const float* v_scale,
                                             const int32_t* block_tables,
                                             const int32_t* context_lens,
                                             const int32_t* query_start, int32_t num_query_rows,
                                             int32_t max_chunk_len, void* out,
                                             const coopt_shape* sh, void* hip_stream)
{
    return prefill_chunk(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, query_start,
                         num_query_rows, max_chunk_len, out, nullptr, sh, hip_stream);
}

extern "C" int coopt_paged_gqa_prefill_chunk_ws(const void* q, const void* k_cache, const void* v_cache,
                                                const float* k_scale, const float* v_scale,
                                                const int32_t* block_tables,
                                                const int32_t* context_lens,
                                                const int32_t* query_start, int32_t num_query_rows,
                                                int32_t max_chunk_len, void* out, void* workspace,
                                                size_t workspace_bytes, const coopt_shape* sh,
                                                void* hip_stream)
{
    int st = check_shape(sh);
    if (st != COOPT_OK) return st;
    if (max_chunk_len > 0 && sh->num_seqs > 0) {
        const size_t need = PrefillLaunchPlan(sh, max_chunk_len, true).workspace_bytes(sh);
        if (need > 0 && !workspace) return COOPT_ERR_NULL;
        if (workspace_bytes < need) return COOPT_ERR_WORKSPACE;
        if (need == 0) workspace = nullptr;
    }
    return prefill_chunk(q, k_cache, v_cache, k_scale, v_scale, block_tables, context_lens, query_start,
                         num_query_rows, max_chunk_len, out, workspace, sh, hip_stream);
}

// The merge of the tiles behind the cut, of all sequences in one launch where a grid holds them.
template <int HEAD_DIM>
static void launch_split_merge(PrefillArgs a, int num_seqs, hipStream_t stream)
{
    // 256 / (d/4) rows per workgroup: two workgroups per tile at d = 128, one at 64
    const long long seq_wgs = (long long)a.H_k * a.tail_cap * (HEAD_DIM / 64);
    const long long step = seqs_per_launch(num_seqs, seq_wgs);
    for (long long left = num_seqs; left > 0; left -= step) {
        const long long n = step < left ? step : left;
        hipLaunchKernelGGL((prefill_split_merge_kernel<HEAD_DIM>), dim3((unsigned)(n * seq_wgs)), dim3(256), 0,
                           stream, a);
        a.query_start += n;
        a.context_lens += n;
        a.part += (size_t)n * a.H_k * a.tail_cap * a.split * (16 * (HEAD_DIM + 2));
    }
}

static int prefill_chunk(const void* q, const void* k_cache, const void* v_cache, const float* k_scale,
                         const float* v_scale, const int32_t* block_tables, const int32_t* context_lens,
                         const int32_t* query_start, int32_t num_query_rows, int32_t max_chunk_len,
                         void* out, void* workspace, const coopt_shape* sh, void* hip_stream)
{
    int st = check_shape(sh);
    if (st != COOPT_OK) return st;
    if (num_query_rows < 0 || max_chunk_len < 0) return COOPT_ERR_SHAPE;
    if (sh->num_seqs == 0 || num_query_rows == 0 || max_chunk_len == 0) return COOPT_OK;
    if (!q || !k_cache || !v_cache || !block_tables || !context_lens || !query_start || !out)
        return COOPT_ERR_NULL;
    if (sh->kv_dtype != COOPT_KV_FP16 && (!k_scale || !v_scale)) return COOPT_ERR_NULL;

    PrefillArgs a{};
    a.q = (const half_t*)q;
    a.cv = CacheView{(const uint8_t*)k_cache, (const uint8_t*)v_cache, k_scale, v_scale};
    a.block_tables = block_tables;
    a.context_lens = context_lens;
    a.query_start = query_start;
    a.out = (half_t*)out;
    a.H_q = sh->num_q_heads;
    a.H_k = sh->num_kv_heads;
    a.kv_heads = Divisor(sh->num_kv_heads);
    a.G = sh->num_q_heads / sh->num_kv_heads;
    a.max_blocks = sh->max_blocks_per_seq;
    a.pool_tiles = sh->num_blocks * sh->num_kv_heads;
    a.scale_log2e = sh->softmax_scale * kLog2e;

    const PrefillLaunchPlan lp(sh, max_chunk_len, workspace != nullptr);
    const int pairs8 = lp.pairs8, a_per_pair = lp.a_per_pair, b_per_pair = lp.b_per_pair;
    a.set(lp, sh->num_seqs * sh->num_kv_heads, (long long)sh->max_blocks_per_seq * kBlock);
    a.part = (float*)workspace;
    const bool split = a.split >= 2;                  // (the table may hold no sequence long enough)
    const int split_per_pair = a.split * a.split_blocks;
    // Turn by turn, so that the longest streams of all pairs start first and the launch ends evenly,
    // while the streams of all of an XCD's pairs can share its 4 MB L2; else pair after pair, whose
    // workgroups then read their stream together.  (8 pairs of 2.3 MB an XCD: 760 us a pass by
    // pair, 770 turn by turn.)  The host does not see the lengths, only what bounds them, the table's
    // width: three fresh prompts of up to 1777 rows take 94 us with a table as wide as the longest
    // and 102 with one of 2048 columns, 3 x 3.5 MB an XCD (159 by head, first rows first).
    const long long token_bytes = (sh->kv_dtype == COOPT_KV_FP16 ? 4LL : 2LL) * sh->head_dim +
                                  (sh->kv_dtype == COOPT_KV_FP16 ? 0 : 8);
    a.by_pair = a.xcd_pairs * (long long)sh->max_blocks_per_seq * kBlock * token_bytes > kPrefillXcdL2;
    // Ragged batches in the order of their streams' lengths, over up to 64 pairs an XCD (one a lane).  A
    // workgroup goes to the XCD's four shader engines in turn whether they have room or not, so a long
    // stream behind a short one, or a workgroup without tiles, holds up all that come after it.  Finding
    // one's rank takes a workgroup 1.2-2 us, so only where many workgroups follow each other on a CU and
    // rows are missing: 16 prompts of 100 to 800 rows (8 a CU, 56 % of the rows) 139 -> 120 us, 6 of 200 to
    // 1500 (d = 64, 4.7 a CU) 95 -> 89; 3 of 301 to 1777 (3.6 a CU) 90 -> 93, 8 of 352 rows each 80 -> 88.
    const long long wgs = (long long)pairs8 * (a_per_pair + b_per_pair + split_per_pair);
    if (!a.by_pair && a.xcd_pairs <= 64 && wgs >= 4 * kPrefillCUs &&
        4LL * num_query_rows <= 3LL * sh->num_seqs * max_chunk_len)
        while ((1LL << a.rank_bits) <= ((long long)sh->max_blocks_per_seq * kBlock + kPrefillStageTokens - 1) / kPrefillStageTokens)
            ++a.rank_bits;
    if (wgs > 0x7fffffffLL) return COOPT_ERR_SHAPE;
    const dim3 block(64 * kPrefillWaves);
    const size_t lds = kPrefillSlots *
                       (size_t)(sh->head_dim == 128 ? PrefillStage<128>::kBytes : PrefillStage<64>::kBytes);
    hipStream_t stream = (hipStream_t)hip_stream;
    const bool big = !pool_fits_small(sh);
#define COOPT_PREFILL_FULL(D, KV, BIG, TILES)                                                          \
    do {                                                                                            \
        hipLaunchKernelGGL((prefill_chunk_kernel<D, KV, TILES, BIG>),                                  \
                           dim3((unsigned)((long long)pairs8 * (a_per_pair + split_per_pair))), block, lds, \
                           stream, a);                                                              \
        if (split)                                                                                  \
            launch_split_merge<D>(a, sh->num_seqs, stream);                                         \
    } while (0)
#define COOPT_PREFILL(D, KV, BIG)                                                                   \
    do {                                                                                            \
        if (lp.nr == 1) {                                                                           \
            COOPT_PREFILL_FULL(D, KV, BIG, 8);                                                      \
        } else {                                                                                    \
            COOPT_PREFILL_FULL(D, KV, BIG, 16);                                                      \
            if (!split && b_per_pair) {                                                             \
                a.set_rest(lp);                                                                     \
                hipLaunchKernelGGL((prefill_chunk_kernel<D, KV, 8, BIG>),                           \
                                   dim3((unsigned)((long long)pairs8 * b_per_pair)), block, lds, stream, a); \
            }                                                                                       \
        }                                                                                           \
    } while (0)
    if (sh->kv_dtype == COOPT_KV_E4M3) {
        if (sh->head_dim == 128) { if (big) COOPT_PREFILL(128, COOPT_KV_E4M3, true); else COOPT_PREFILL(128, COOPT_KV_E4M3, false); }
        else { if (big) COOPT_PREFILL(64, COOPT_KV_E4M3, true); else COOPT_PREFILL(64, COOPT_KV_E4M3, false); }
    } else if (sh->kv_dtype == COOPT_KV_E5M2) {
        if (sh->head_dim == 128) { if (big) COOPT_PREFILL(128, COOPT_KV_E5M2, true); else COOPT_PREFILL(128, COOPT_KV_E5M2, false); }
        else { if (big) COOPT_PREFILL(64, COOPT_KV_E5M2, true); else COOPT_PREFILL(64, COOPT_KV_E5M2, false); }
    } else {
        if (sh->head_dim == 128) { if (big) COOPT_PREFILL(128, COOPT_KV_FP16, true); else COOPT_PREFILL(128, COOPT_KV_FP16, false); }
        else { if (big) COOPT_PREFILL(64, COOPT_KV_FP16, true); else COOPT_PREFILL(64, COOPT_KV_FP16, false); }
    }
#undef COOPT_PREFILL
#undef COOPT_PREFILL_FULL
    return launch_status();
}

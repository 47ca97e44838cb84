// How a prefill launch deals the query tiles of a batch to its workgroups: the host's plan, the order
// of a pair's tiles, and what the workgroup of a given number takes.  Plain C++ but for wave_uniform (a
// value that is the same in every lane), the two function qualifiers and a reciprocal that only device
// code takes from its builtin, so that a host program which defines the former can walk a launch
// and look at every index that the kernel stores through.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "coopt_attn.h"

namespace coopt {

constexpr int kPrefillWaves = 8;                // two teams of four producer roles
constexpr int kPrefillMaxParts = 8;             // runs a split launch cuts a stream into, at most
constexpr int kPrefillStageTokens = 128;        // between two barriers of the stream
constexpr int kPrefillCUs = 256;                // MI355X: the launch shape is planned for its CU count

// A divisor that the host knows: a quotient of wave-uniform values is then a product on the scalar unit
// (a division goes through the vector ALU, 0.1 us of a workgroup's start each).  0 <= x < 2^31.
struct Divisor {
    uint32_t d, m;             // m = floor((2^32 - 1) / d): the high half of x m is the quotient or one less
    Divisor() = default;
    explicit Divisor(int by) : d((uint32_t)by), m(0xffffffffu / (uint32_t)by) {}
    __device__ __forceinline__ int quotient(int x) const
    {
        const uint32_t q = (uint32_t)(((uint64_t)(uint32_t)x * m) >> 32);
        return (int)(q + ((uint32_t)x - q * d >= d ? 1u : 0u));
    }
};

// x / y for a divisor that only the device knows, 0 <= x, 1 <= y.  Below 2^22 by way of binary32: x and y
// are exact there, the reciprocal is off by an ulp and the product by half of one, so the truncated
// product is the quotient or one off it.
__device__ __forceinline__ int quotient(int x, int y)
{
    if (x >= (1 << 22)) return (int)((uint32_t)x / (uint32_t)y);
#if defined(__HIP_DEVICE_COMPILE__)
    const float r = __builtin_amdgcn_rcpf((float)y);
#else
    const float r = 1.0f / (float)y;
#endif
    const int q = (int)((float)x * r), left = x - q * y;
    return q + (left >= y ? 1 : 0) - (left < 0 ? 1 : 0);
}

// How the tiles of every pair are dealt to launches.  One workgroup (8 waves, 2 tiles each) fills
// a CU, so a launch runs in rounds of one workgroup per CU, and a last round that is mostly empty
// costs a full one.  Where that happens the last tiles of every pair go to a launch of half-size
// workgroups behind it (8 tiles), which takes about 0.65-0.8 of a round -- or, when the
// caller brings a workspace, to full-size workgroups of the same launch, `parts` per 16 tiles, that
// each stream one of `parts` equal runs of the pair's stages, with `parts` (2 to 8) chosen so that
// the round is as short as it gets (a launch of fewer workgroups than CUs is all "last round": a
// single sequence's chunk is spread over the chip this way); the parts are combined by
// prefill_split_merge_kernel.  (The rounds are counted as if a workgroup cost nothing but its stream,
// which is not so for short ones: the device, which sees the lengths, has those run whole after all,
// prefill_runs_whole.)
struct PrefillLaunchPlan {
    int tiles, pairs8, a_per_pair, b_per_pair, rest, parts;
    int nr;          // tiles per 64 lanes of the full-size workgroups: 2, or 1 where a pair has at most 8 tiles
    int wg_tiles;    // = 8 nr
    PrefillLaunchPlan(const coopt_shape* sh, int max_chunk_len, bool with_workspace)
    {
        const int G = sh->num_q_heads / sh->num_kv_heads;
        tiles = G * ((max_chunk_len + 15) / 16);
        pairs8 = (sh->num_seqs * sh->num_kv_heads + 7) / 8 * 8;
        // (a short chunk -- 16 rows of a five-head group, say -- fills half the waves at most: the kernel
        // of 8 tiles then has the other half bring the stream, 0.85 of the time)
        nr = tiles <= kPrefillWaves ? 1 : 2;
        wg_tiles = nr * kPrefillWaves;
        const int full_per_pair = (tiles + wg_tiles - 1) / wg_tiles;
        a_per_pair = full_per_pair;
        b_per_pair = 0;
        rest = 0;
        parts = 0;
        auto rounds = [](long long wgs) { return (double)((wgs + kPrefillCUs - 1) / kPrefillCUs); };
        const long long W = (long long)pairs8 * full_per_pair;
        const int cand = (int)((W / kPrefillCUs) * kPrefillCUs / pairs8);   // full rounds only
        if (cand >= full_per_pair) return;                                   // whole rounds
        const int r = tiles - cand * wg_tiles;                               // tiles of the last round, per pair
        // p parts make p times the workgroups, each 1/p as long; a part costs about 2 % of a
        // round on top (its start, its partial rows, its share of the merge)
        const long long last = (long long)pairs8 * ((r + wg_tiles - 1) / wg_tiles);
        int best = 1;
        double best_cost = rounds(last);
        for (int p = 2; p <= kPrefillMaxParts; ++p) {
            const double cost = rounds(last * p) / p + 0.02 * (p - 1);
            if (cost < best_cost) {
                best_cost = cost;
                best = p;
            }
        }
        if (best >= 2 && with_workspace) {
            a_per_pair = cand;
            rest = r;
            parts = best;
            return;
        }
        if (cand >= 1 && nr == 2) {
            const int small = (r + kPrefillWaves - 1) / kPrefillWaves;
            const double split = rounds((long long)pairs8 * cand) + 0.65 * rounds((long long)pairs8 * small);
            if (split < rounds(W)) {
                a_per_pair = cand;
                b_per_pair = small;
                rest = r;
                return;
            }
        }
        // What a workspace would split runs whole, but behind the same cut: which rows share a wavefront
        // decides when their references are raised, and the tiles in front of the cut are to have the
        // same bits with and without a workspace.
        if (best >= 2) {
            a_per_pair = cand;
            rest = r;
            parts = 1;
        }
    }
    // workgroups per pair over the tiles behind the cut
    int split_per_pair() const { return parts * ((rest + wg_tiles - 1) / wg_tiles); }
    size_t workspace_bytes(const coopt_shape* sh) const
    {
        if (parts < 2) return 0;
        return (size_t)sh->num_seqs * sh->num_kv_heads * rest * parts * 16 * (sh->head_dim + 2) * sizeof(float);
    }
};

// What the kernel is told about the deal.
struct PrefillDeal {
    int32_t num_pairs;        // num_seqs * H_k
    int32_t xcd_pairs;        // pairs per XCD: num_pairs rounded up to a multiple of 8, over 8
    int32_t by_pair;          // order of an XCD's workgroups (prefill_pair)
    int32_t blocks_per_pair;  // workgroups per pair over tiles [tile_base, tile_limit): whole streams
    int32_t tile_base;
    int32_t tile_limit;
    // split workgroups, behind the whole-stream ones in the grid (the tiles from tile_limit on of
    // every pair, `split` workgroups per 16 tiles: workgroup p of them streams the p-th of `split`
    // equal runs of the pair's stages and leaves per tile 16 x (m, l) and the 16 x HEAD_DIM
    // unnormalised sums in the workspace, which a merge launch combines)
    int32_t split;            // parts (0: no such workgroups; 1: whole streams, rows written to out)
    int32_t split_blocks;     // runs of 16 tiles per pair they cover
    int32_t tail_cap;         // tiles per pair they cover (sizes the workspace)
    int32_t whole_tokens;     // sequences up to this length have their split streams run whole after all
    Divisor pairs_of_xcd, whole_of_pair, rest_of_pair, split_parts, blocks_of_part;     // (at least 1 each)

    // The first launch of a plan (its only one but for a plan's half-size workgroups).  most_tokens: no
    // sequence is longer.
    void set(const PrefillLaunchPlan& lp, int pairs, long long most_tokens = 0x7fffffff)
    {
        num_pairs = pairs;
        xcd_pairs = lp.pairs8 / 8;
        blocks_per_pair = lp.a_per_pair;
        tile_base = 0;
        tile_limit = lp.rest > 0 ? lp.a_per_pair * lp.wg_tiles : 0x7fffffff;
        split = lp.parts;
        split_blocks = lp.parts > 0 ? lp.split_per_pair() / lp.parts : 0;
        tail_cap = lp.parts > 0 ? lp.rest : 0;
        // A workgroup costs its n stages and the time of 2.3 on top: its start, its rows, the change to the
        // CU's next (9 us; a stage takes 4).  In R rounds of whole streams, or S rounds of p parts, whole
        // ones are the faster where R (2.3 + n) <= S (2.3 + n / p): 8 fresh prompts of 352 rows, 3 rounds of
        // quarters of 3 stages, take 79 us split and 64 whole, 3 x 777 rows behind 500 tokens, 3 rounds
        // of fifths of 10 stages, 117 and 104.
        // (One figure for all kernels: 2.3 stages are of E4M3 at 128 dims.  At 64 dims a stage takes 3.1 us
        // and the ends are more of them, so the rule is on the side of splitting there, which is what every call
        // did without it: 8 x 352 rows fresh 38 us split and 30 whole, behind 500 tokens 64 and 54.)
        whole_tokens = 0;
        if (split > 1) {
            const long long last = (long long)lp.pairs8 * split_blocks;
            const double R = (double)((last + kPrefillCUs - 1) / kPrefillCUs);
            const double S = (double)((last * split + kPrefillCUs - 1) / kPrefillCUs);
            const double stages = R * split > S ? 2.3 * (S - R) / (R - S / split) : 1e6;
            whole_tokens = kPrefillStageTokens * (int)(stages < 1e6 ? stages : 1e6);
            // (where every sequence would: no workgroups for parts that nobody streams)
            if (most_tokens <= whole_tokens) split = 1;
        }
        set_divisors();
    }
    // ... and the one of half-size workgroups behind it: the tiles that it left.
    void set_rest(const PrefillLaunchPlan& lp)
    {
        tile_base = tile_limit;
        tile_limit = 0x7fffffff;
        blocks_per_pair = lp.b_per_pair;
        set_divisors();
    }
    void set_divisors()
    {
        const int rest = (split - 1) * split_blocks;
        pairs_of_xcd = Divisor(xcd_pairs > 0 ? xcd_pairs : 1);
        whole_of_pair = Divisor(blocks_per_pair > 0 ? blocks_per_pair : 1);
        rest_of_pair = Divisor(rest > 0 ? rest : 1);
        split_parts = Divisor(split > 0 ? split : 1);
        blocks_of_part = Divisor(split_blocks > 0 ? split_blocks : 1);
    }
};

// The pair of workgroup `wg`, and `turn`: which of the pair's workgroups it is, longest stream first.
// All workgroups of a pair sit on one XCD (ids go round-robin over 8 XCDs).  By pair: an XCD's
// whole-stream workgroups pair after pair, then of its split ones as many as there would be of whole streams
// (prefill_share), then the rest of them; otherwise turn after turn of all its pairs.  A pair >= num_pairs is none.
__device__ __forceinline__ int prefill_pair(const PrefillDeal& a, unsigned wg, int& turn)
{
    const int k8 = wg >> 3;
    const int whole = a.xcd_pairs * a.blocks_per_pair;           // whole-stream workgroups per XCD
    int xcd_pair;
    if (a.by_pair) {
        const int first = whole + a.xcd_pairs * a.split_blocks;
        const int k = k8 < whole ? k8 : k8 < first ? k8 - whole : k8 - first;
        Divisor per = a.rest_of_pair;
        if (k8 < first) per = a.blocks_of_part;
        if (k8 < whole) per = a.whole_of_pair;
        xcd_pair = per.quotient(k);
        turn = k - xcd_pair * (int)per.d + (k8 < whole ? 0 : a.blocks_per_pair + (k8 < first ? 0 : a.split_blocks));
    } else {
        turn = a.pairs_of_xcd.quotient(k8);
        xcd_pair = k8 - turn * a.xcd_pairs;
    }
    return xcd_pair * 8 + (wg & 7);
}

// Whether a sequence of t tokens has its split streams run whole (by the workgroup of their first part;
// the others have nothing to do, nor has the merge).
__device__ __forceinline__ bool prefill_runs_whole(const PrefillDeal& a, int t) { return t <= a.whole_tokens; }

// How many whole-stream workgroups of a pair start before those behind the cut: all of them where these are
// runs of about t / split tokens and the history is longer than that, none where they are whole streams;
// and those of longer streams in front of the first rows of a fresh prompt.  (In binary32, the same for
// every workgroup of the pair: it only places them.)
__device__ __forceinline__ int prefill_ahead(const PrefillDeal& a, int t, int C)
{
    if (a.split * a.split_blocks == 0 || a.by_pair) return a.blocks_per_pair;
    const int tokens = prefill_runs_whole(a, t) ? t : a.split_parts.quotient(t);
    const int shorter = (int)((float)(tokens - (t - C)) * (float)a.blocks_per_pair / (float)C);
    return a.blocks_per_pair - min(max(shorter, 0), a.blocks_per_pair);
}

// A workgroup's tiles: positions block * WG .. of the range [base, end) in TileOrder, as one of `parts`
// runs of their stream.
struct PrefillShare {
    bool tail;
    int block, base, end, parts, part;
};

// The pair's workgroups by the length of their streams: whole streams from the last rows down, and the
// split ones where their length has its place (prefill_ahead): all parts of a block's stream one after the
// other, but where whole streams run after all, first the workgroups that have nothing to do, then those of
// the first parts (by pair the other way round, which puts the latter of all pairs together).  Ids go
// round-robin over an XCD's four shader engines, so with work in every second or fourth alone two engines or
// one had all of it: 8 x 352 rows behind 1500 tokens of a table for 7400 took 228 us, so 129; 2 x 777 of 64
// dims behind 4000, 196 and 113.  (Idle ones behind everything instead: 3 fresh prompts of 301 to 1777 rows,
// the short ones whole, 48.7 against 44.6 us, since short streams then start ahead of long ones.)
// t: the sequence's tokens, C of them new rows, total_tiles tiles.  C comes from the device and may be more than the host was told: tiles
// beyond those that the launch and its workspace were sized for are left out.
__device__ __forceinline__ PrefillShare prefill_share(const PrefillDeal& a, int turn, int t, int C, int total_tiles)
{
    const int num_split = a.split * a.split_blocks;
    const int ahead = wave_uniform(prefill_ahead(a, t, C));
    PrefillShare s;
    s.tail = turn >= ahead && turn < ahead + num_split;
    const int nth = s.tail ? turn - ahead : (turn < ahead ? turn : turn - num_split);
    s.parts = s.tail ? a.split : 1;
    const bool whole = s.tail && prefill_runs_whole(a, t);
    Divisor by = a.split_parts;
    if (whole) by = a.blocks_of_part;
    const int q = s.tail ? by.quotient(nth) : nth, rest = s.tail ? nth - q * (int)by.d : 0;
    const int split_block = whole ? rest : q;
    s.part = !whole ? rest : a.by_pair ? q : s.parts - 1 - q;    // which run of the pair's stages is mine
    s.block = (s.tail ? a.split_blocks : a.blocks_per_pair) - 1 - split_block;
    s.base = s.tail ? a.tile_limit : a.tile_base;
    s.end = min(total_tiles, s.tail ? a.tile_limit + a.tail_cap : a.tile_limit);
    return s;
}

// The tiles [base, end) of a pair -- tile h T + i is rows 16i .. of head h, T tiles a head -- in the
// order in which workgroups take them: by row, then by head.  A causal stream is as long as its
// last row needs, so the 16 tiles of a workgroup should lie at neighbouring rows: by head, a
// workgroup of 256 rows streams up to 240 tokens too far for most of them.
struct TileOrder {
    int T, base, end, hb, ib, he, ie;
    __device__ __forceinline__ TileOrder(int tiles_per_head, int b, int e) : T(tiles_per_head), base(b), end(e)
    {
        hb = quotient(b, T);
        ib = b - hb * T;
        he = quotient(e, T);
        ie = e - he * T;
    }
    // (where both ends are known as head and row already)
    __device__ __forceinline__ TileOrder(int tiles_per_head, int b, int b_head, int e, int e_head)
        : T(tiles_per_head), base(b), end(e), hb(b_head), ib(b - b_head * T), he(e_head), ie(e - e_head * T) {}
    // (quotients are made on the vector ALU; where they are the same in every lane this takes them off it)
    __device__ __forceinline__ void to_scalar()
    {
        hb = wave_uniform(hb);
        ib = wave_uniform(ib);
        he = wave_uniform(he);
        ie = wave_uniform(ie);
    }
    __device__ __forceinline__ int count() const { return end - base; }
    // Position p (0 .. count-1) -> first row / 16 and head.  Row i has he - hb tiles of this range,
    // one more from ib .. or up to ie (whichever of the two partial heads reaches it).
    __device__ __forceinline__ void at(int p, int& i, int& h) const
    {
        const int N = he - hb, b1 = min(ib, ie), b2 = max(ib, ie);
        const int c2 = ie > ib ? N + 1 : N - 1;                  // tiles per row between b1 and b2
        const int n1 = b1 * N, n2 = n1 + (b2 - b1) * c2;
        // (one division whatever the lane's third of the rows; max: a divisor even where nothing divides)
        const bool mid = p >= n1 && p < n2;
        i = (p < n1 ? 0 : mid ? b1 : b2) + quotient(p - (p < n1 ? 0 : mid ? n1 : n2), max(mid ? c2 : N, 1));
        h = p - below(i) + hb + (i < ib ? 1 : 0);
    }
    // Tiles of the range in the rows in front of row i.
    __device__ __forceinline__ int below(int i) const { return i * (he - hb) + min(i, ie) - min(i, ib); }
};

// What a pair gives a launch to do, for an order of the workgroups over several pairs (whose sequences
// differ in length): its workgroups that have tiles at all, whole-stream ones and those behind the cut,
// each kind longest stream first.
struct PairItems {
    int whole, split;          // of either kind
    int ahead, num_split, empty_whole, t, t_ctx, rows, tail_tokens, wg_tiles;
    bool runs;                 // behind the cut: runs of a stream, all about tail_tokens long (else whole streams)
    TileOrder order, tail;
    __device__ __forceinline__ PairItems(const PrefillDeal& a, int tokens, int C, int G, int wg_tiles_)
        : whole(0), split(0), ahead(0), num_split(a.split * a.split_blocks), empty_whole(0), t(tokens), t_ctx(tokens - C),
          rows((max(C, 1) + 15) / 16), tail_tokens(0), wg_tiles(wg_tiles_), runs(a.split > 1 && !prefill_runs_whole(a, tokens)),
          order(range(a.tile_base, min(G * rows, a.tile_limit), G)),
          tail(range(a.tile_limit, G * rows, G))
    {
        // (a sequence longer than announced: tiles that nobody takes)
        if (a.tail_cap < tail.count()) tail = TileOrder(rows, tail.base, tail.base + a.tail_cap);
        if (C <= 0) return;
        whole = min(blocks(order.count()), a.blocks_per_pair);
        split = (runs ? a.split : 1) * blocks(tail.count());
        ahead = prefill_ahead(a, t, C);
        empty_whole = a.blocks_per_pair - whole;
        tail_tokens = a.split_parts.quotient(t);
    }
    // Tiles [b, e) of G heads, none if e <= b.  (Most ends are the last head's: no quotient.)
    __device__ __forceinline__ TileOrder range(int b, int e, int G) const
    {
        if (e <= b) return TileOrder(rows, 0, 0, 0, 0);
        const int b_head = b == 0 ? 0 : quotient(b, rows);
        return TileOrder(rows, b, b_head, e, e == G * rows ? G : quotient(e, rows));
    }
    __device__ __forceinline__ int blocks(int tiles) const { return wg_tiles == 16 ? (tiles + 15) >> 4 : (tiles + 7) >> 3; }
    // Of `have` workgroups over a range those whose stream is longer than `tokens`.
    __device__ __forceinline__ int longer(const TileOrder& o, int have, int tokens) const
    {
        const int row = max(tokens - t_ctx, 0) >> 4;                         // tiles from this row on
        const int pos = row < rows && tokens < t ? o.below(row) : o.count();
        return pos < o.count() ? max(have - (wg_tiles == 16 ? pos >> 4 : pos >> 3), 0) : 0;
    }
    // Those of at least so many stages, as far as it decides an order: all at 1, never more with more stages.
    __device__ __forceinline__ int whole_at_least(int stages) const
    {
        return stages <= 1 ? whole : longer(order, whole, (stages - 1) * kPrefillStageTokens);
    }
    __device__ __forceinline__ int split_at_least(int stages) const
    {
        if (stages <= 1 || split == 0) return split;
        const int tokens = (stages - 1) * kPrefillStageTokens;
        return !runs ? longer(tail, split, tokens) : tail_tokens >= tokens ? split : 0;
    }
    __device__ __forceinline__ int at_least(int stages) const { return whole_at_least(stages) + split_at_least(stages); }
    // The turn (prefill_share) of the k-th item of exactly so many stages.
    __device__ __forceinline__ int turn(int stages, int k) const
    {
        const int w = whole_at_least(stages + 1), of_whole = whole_at_least(stages) - w;
        if (k >= of_whole) return ahead + num_split - (split - split_at_least(stages + 1) - k + of_whole);
        const int nth = empty_whole + w + k;
        return nth < ahead ? nth : nth + num_split;
    }
};

// The most stages that more than `rank` items have, 0 if there are not so many items: the length of the
// item at that rank.  total(stages): PairItems::at_least over the pairs; lengths are below 2^bits.
template <class Total>
__device__ __forceinline__ int stages_of_rank(int rank, int bits, Total total)
{
    int stages = 0;
    for (int bit = 1 << (bits - 1); bit > 0; bit >>= 1)
        if (total(stages + bit) > rank) stages += bit;
    return stages;
}

}  // namespace coopt

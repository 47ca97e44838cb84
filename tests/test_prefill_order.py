"""The order of a prefill launch's workgroups over sequences of different lengths (csrc/prefill_deal.hpp,
compiled here for the CPU): the workgroup of every rank, found as the kernel finds it, takes a turn of its
own; every turn that has tiles is taken and none that has not; lengths never grow by more than the one
stage that the split streams' rounded length may be off.  Where split streams run whole after all,
the workgroups without work lie together in front of those, and where every sequence's do there are none.  And the quotients that the
deal is made of."""
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent

SOURCE = r"""
#include <algorithm>
#include <cstdio>
#include <set>
#include <vector>
#define __device__
#define __forceinline__ inline
using std::max;
using std::min;
template <class T> T wave_uniform(T v) { return v; }
#include "prefill_deal.hpp"
using namespace coopt;

static int bad = 0;
static char what[200];
#define CHECK(c) do { if (!(c) && ++bad < 10) printf("line %d: %s: %s\n", __LINE__, what, #c); } while (0)

// Stages of the workgroup of a turn, 0: it has no tiles.
static int stages_of(const PrefillDeal& a, int turn, int t, int C, int G, int wg_tiles)
{
    if (C <= 0) return 0;
    const int T = (C + 15) / 16;
    const PrefillShare s = prefill_share(a, turn, t, C, G * T);
    if (s.block < 0 || s.base + s.block * wg_tiles >= s.end) return 0;
    const bool whole = s.parts == 1 || prefill_runs_whole(a, t);
    if (whole && s.part > 0) return 0;
    const TileOrder order(T, s.base, s.end);
    int i, h;
    order.at(min((s.block + 1) * wg_tiles, order.count()) - 1, i, h);
    const int stages = (t - C + min(16 * i + 15, C - 1) + kPrefillStageTokens) / kPrefillStageTokens;
    return max(1, whole ? stages : (t / s.parts + kPrefillStageTokens) / kPrefillStageTokens);
}

static long long launches = 0;

static void launch(const PrefillDeal& a, int G, int H_k, int nr, int per_pair, int bits, const std::vector<int>& C,
                   const std::vector<int>& t)
{
    ++launches;
    const int wg_tiles = kPrefillWaves * nr;
    for (int xcd = 0; xcd < 8; ++xcd) {
        std::vector<PairItems> items;
        std::vector<int> seq;
        int expected = 0;
        for (int p = 0; p < a.xcd_pairs; ++p) {
            const int pair = 8 * p + xcd, s = pair < a.num_pairs ? pair / H_k : 0, c = pair < a.num_pairs ? C[s] : 0;
            seq.push_back(s);
            items.push_back(PairItems(a, t[s], c, G, wg_tiles));
            for (int turn = 0; turn < per_pair; ++turn) expected += stages_of(a, turn, t[s], c, G, wg_tiles) > 0;
        }
        auto total = [&](int l) { int n = 0; for (auto& i : items) n += i.at_least(l); return n; };
        // (a workgroup with work in every second or fourth place is one or two shader engines' work)
        for (int p = 0; p < a.xcd_pairs; ++p) {
            const int pair = 8 * p + xcd;
            if (pair >= a.num_pairs || a.split < 2 || C[seq[p]] <= 0 || !prefill_runs_whole(a, t[seq[p]])) continue;
            int first = -1;
            for (int turn = 0; turn < per_pair; ++turn) {
                const PrefillShare s = prefill_share(a, turn, t[seq[p]], C[seq[p]], G * ((C[seq[p]] + 15) / 16));
                if (s.tail && first < 0) first = turn;
                if (s.tail) CHECK((s.part > 0) == (turn - first < (a.split - 1) * a.split_blocks));
            }
        }
        std::set<std::pair<int, int>> taken;
        int previous = 1 << 30;
        for (int rank = 0; rank < a.xcd_pairs * per_pair; ++rank) {
            const int stages = stages_of_rank(rank, bits, total);
            CHECK((stages > 0) == (rank < expected));
            if (stages == 0) continue;
            int behind = rank - total(stages + 1), p = 0;
            while (p < a.xcd_pairs && behind >= items[p].at_least(stages) - items[p].at_least(stages + 1)) {
                behind -= items[p].at_least(stages) - items[p].at_least(stages + 1);
                ++p;
            }
            CHECK(p < a.xcd_pairs);
            if (p >= a.xcd_pairs) continue;
            const int turn = items[p].turn(stages, behind);
            CHECK(turn >= 0 && turn < per_pair);
            CHECK(taken.insert({p, turn}).second);
            const int length = stages_of(a, turn, t[seq[p]], C[seq[p]], G, wg_tiles);
            CHECK(length > 0);
            CHECK(length <= previous + 1);
            previous = min(previous, length);
        }
    }
}

int main()
{
    for (int d : {1, 2, 3, 5, 7, 40, 255, 1000003, 0x7fffffff}) {
        sprintf(what, "divisor %d", d);
        const Divisor by(d);
        for (long long q = 0; q * d <= 0x7fffffffLL; q += 1 + q / 5)
            for (int off = -1; off <= 1; ++off) {
                const long long x = q * d + off;
                if (x < 0 || x > 0x7fffffffLL) continue;
                CHECK(by.quotient((int)x) == (int)(x / d));
                CHECK(quotient((int)x, d) == (int)(x / d));
            }
    }
    const int heads[][2] = {{40, 8}, {32, 8}, {8, 8}, {40, 40}, {4, 2}, {16, 1}};
    for (auto& hh : heads)
        for (int S : {1, 2, 3, 6, 13, 40})
            for (int announced : {1, 16, 17, 130, 333, 352, 777, 1777})
                for (int ragged = 0; ragged < 4; ++ragged)
                    for (int history : {0, 50, 900}) {
                        std::vector<int> C, t;
                        int longest = 1;
                        for (int s = 0; s < S; ++s) {
                            int c = ragged == 0 ? announced : ragged == 1 ? announced - announced * s / S
                                    : ragged == 2 ? (s % 3 == 1 ? 0 : announced * (s + 1) / S) : announced + 16 * (s % 4);
                            C.push_back(c);
                            t.push_back(c + history * (s % 2 + 1));
                            longest = max(longest, t.back());
                        }
                        for (int ws = 0; ws < 2; ++ws) {
                            coopt_shape sh{};
                            sh.num_seqs = S;
                            sh.num_q_heads = hh[0];
                            sh.num_kv_heads = hh[1];
                            sh.head_dim = 128;
                            const PrefillLaunchPlan lp(&sh, announced, ws);
                            PrefillDeal a{};
                            a.set(lp, S * hh[1]);
                            if (a.xcd_pairs > 64) continue;
                            sprintf(what, "%d/%d heads, %d x %d rows, ragged %d, history %d, workspace %d", hh[0], hh[1], S,
                                    announced, ragged, history, ws);
                            int bits = 0;
                            while ((1 << bits) <= (longest + kPrefillStageTokens - 1) / kPrefillStageTokens) ++bits;
                            launch(a, hh[0] / hh[1], hh[1], lp.nr, lp.a_per_pair + lp.split_per_pair(), bits, C, t);
                            if (lp.parts > 1) {
                                const int line = a.whole_tokens;
                                a.set(lp, S * hh[1], line);
                                CHECK(line == 0 || (a.split == 1 && a.split_blocks == lp.split_per_pair() / lp.parts));
                                launch(a, hh[0] / hh[1], hh[1], lp.nr, lp.a_per_pair + a.split * a.split_blocks, bits, C, t);
                                a.set(lp, S * hh[1], line + 1LL);
                                CHECK(a.split == lp.parts);
                            }
                            if (lp.parts < 2 && lp.b_per_pair) {
                                a.set_rest(lp);
                                launch(a, hh[0] / hh[1], hh[1], 1, lp.b_per_pair, bits, C, t);
                            }
                        }
                    }
    printf("%lld launches, %d bad\n", launches, bad);
    return 0;
}
"""


def test_every_workgroup_with_tiles_once_longest_first(tmp_path):
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", f"-I{ROOT / 'paper_2602_09323_amd' / 'csrc'}", f"-I{ROOT / 'include'}",
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    words = out.splitlines()[-1].split()
    assert int(words[0]) > 1000 and int(words[2]) == 0, out

"""The deal of a prefill launch (csrc/prefill_deal.hpp, compiled here for the CPU): every workgroup of
every launch is walked with the kernel's own mapping.  Every tile of every pair is taken exactly once, or
once per part; a tile that the entry point with a workspace does not split is taken whole by a
workgroup of the same rows with and without one, so that its bits are the same; where a sequence is longer than the `max_chunk_len` the host was told, nothing is stored
beyond the workspace that the host asked for, nor into another pair's share of it."""
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent

SOURCE = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
#define __device__
#define __forceinline__ inline
using std::max;
using std::min;
template <class T> T wave_uniform(T v) { return v; }
#include "prefill_deal.hpp"
using namespace coopt;

static int bad = 0;
#define CHECK(c) do { if (!(c) && ++bad < 10) printf("line %d: %s: %s\n", __LINE__, what, #c); } while (0)
static char what[200];

typedef std::vector<std::vector<int>> Tiles;      // [pair][tile]

struct Walk {
    Tiles taken, of_part;          // times a tile was taken whole; times its parts were
    Tiles group;                   // last row / 16 of the workgroup that took it whole, -1 else
    int parts, limit, cap;
    std::vector<int> slots;        // times a part's slot of the workspace was written
};

static void walk_launch(const PrefillDeal& a, int G, int nr, long long grid, const std::vector<int>& C,
                        const std::vector<int>& t, Walk& w)
{
    const int wg_tiles = kPrefillWaves * nr, H_k = a.num_pairs / (int)C.size();
    for (long long wg = 0; wg < grid; ++wg) {
        int turn;
        const int pair = prefill_pair(a, (unsigned)wg, turn);
        CHECK(pair >= 0 && turn >= 0);
        if (pair >= a.num_pairs) continue;
        const int seq = pair / H_k;
        if (C[seq] <= 0) continue;
        const int T = (C[seq] + 15) / 16, total = G * T;
        const PrefillShare s = prefill_share(a, turn, t[seq], C[seq], total);
        if (s.base + s.block * wg_tiles >= s.end) continue;
        CHECK(s.block >= 0 && s.part >= 0 && s.part < s.parts);
        const TileOrder order(T, s.base, s.end);
        std::vector<int> mine;
        int last_row = -1, last, unused;
        order.at(min((s.block + 1) * wg_tiles, order.count()) - 1, last, unused);
        for (int p = s.block * wg_tiles; p < min((s.block + 1) * wg_tiles, order.count()); ++p) {
            int i, h;
            order.at(p, i, h);
            CHECK(i >= 0 && i < T && h >= 0 && h < G);
            const int tile = h * T + i;
            CHECK(tile >= s.base && tile < s.end);
            last_row = max(last_row, i);
            mine.push_back(tile);
            if (s.parts > 1) {
                CHECK(tile - s.base < a.tail_cap);
                const long long slot = ((long long)pair * a.tail_cap + tile - s.base) * s.parts + s.part;
                CHECK(slot >= 0 && slot < (long long)w.slots.size());
                if (slot >= 0 && slot < (long long)w.slots.size()) ++w.slots[slot];
                ++w.of_part[pair][tile];
            } else {
                ++w.taken[pair][tile];
            }
        }
        CHECK(last == last_row);                     // the stream goes as far as the last position needs
        if (s.parts == 1)
            for (int tile : mine) w.group[pair][tile] = last_row;
    }
}

static Walk walk(int H_q, int H_k, int announced, bool with_workspace, bool by_pair, const std::vector<int>& C,
                 const std::vector<int>& t)
{
    coopt_shape sh{};
    sh.num_seqs = (int)C.size();
    sh.num_q_heads = H_q;
    sh.num_kv_heads = H_k;
    sh.head_dim = 128;
    const PrefillLaunchPlan lp(&sh, announced, with_workspace);
    const int G = H_q / H_k, pairs = sh.num_seqs * H_k;
    Walk w;
    for (int pair = 0; pair < pairs; ++pair) {
        const int total = G * ((C[pair / H_k] + 15) / 16);
        w.taken.push_back(std::vector<int>(total, 0));
        w.of_part.push_back(std::vector<int>(total, 0));
        w.group.push_back(std::vector<int>(total, -1));
    }
    PrefillDeal a{};
    a.by_pair = by_pair;
    a.set(lp, pairs);
    w.parts = lp.parts;
    w.limit = a.tile_limit;
    w.cap = a.tail_cap;
    w.slots.assign(lp.workspace_bytes(&sh) / (16 * (sh.head_dim + 2) * sizeof(float)), 0);
    walk_launch(a, G, lp.nr, (long long)lp.pairs8 * (lp.a_per_pair + lp.split_per_pair()), C, t, w);
    if (lp.parts < 2 && lp.b_per_pair) {
        a.set_rest(lp);
        walk_launch(a, G, 1, (long long)lp.pairs8 * lp.b_per_pair, C, t, w);
    }
    return w;
}

int main(int argc, char** argv)
{
    const int heads[][2] = {{40, 8}, {32, 8}, {8, 8}, {40, 40}, {4, 2}, {16, 1}};
    const int over = atoi(argv[1]);                  // sequences longer than announced, 0: none
    long long calls = 0, split = 0;
    for (auto& hh : heads)
        for (int S : {1, 2, 3, 6, 8, 13})
            for (int announced : {1, 16, 17, 130, 300, 333, 352, 512, 777, 1777})
                for (int ragged = 0; ragged < 3; ++ragged)
                    for (int history : {0, 50, 900}) {
                        std::vector<int> C, t;
                        for (int s = 0; s < S; ++s) {
                            int c = ragged == 0 ? announced : ragged == 1 ? announced - announced * s / S
                                                                          : (s % 3 == 1 ? 0 : announced * (s + 1) / S);
                            if (over && s % 2 == 0) c = announced + announced / 2 + 16 * over;
                            C.push_back(c);
                            t.push_back(c + history * (s % 2 + 1));
                        }
                        // mode 0 comes first: what the entry point without a workspace does
                        Walk plain;
                        for (int mode = 0; mode < 4; ++mode) {
                            const bool ws = mode & 1, by_pair = mode & 2;
                            sprintf(what, "%d/%d heads, %d x %d rows, ragged %d, history %d, workspace %d, by pair %d",
                                    hh[0], hh[1], S, announced, ragged, history, ws, by_pair);
                            const Walk w = walk(hh[0], hh[1], announced, ws, by_pair, C, t);
                            if (mode == 0) plain = w;
                            ++calls;
                            split += w.parts > 1;
                            for (int n : w.slots) CHECK(n <= 1);
                            for (size_t p = 0; p < w.taken.size(); ++p)
                                for (size_t i = 0; i < w.taken[p].size(); ++i) {
                                    const int whole = w.taken[p][i], parts = w.of_part[p][i];
                                    const bool tail = w.parts > 1 && (int)i >= w.limit;
                                    // what the merge combines is what the parts' workgroups left
                                    if (tail) CHECK(whole == 0 && parts == ((int)i < w.limit + w.cap ? w.parts : 0));
                                    else if (C[p / hh[1]] <= announced) CHECK(whole == 1 && parts == 0);
                                    else CHECK(whole <= 1 && parts == 0);
                                    // (the same neighbours: when their references are raised, and so the rounding, depends on them)
                                    if (!tail && whole) CHECK(w.group[p][i] == plain.group[p][i]);
                                }
                        }
                    }
    printf("%lld calls, %lld split, %d bad\n", calls, split, bad);
    return 0;
}
"""


@pytest.fixture(scope="module")
def walker(tmp_path_factory):
    d = tmp_path_factory.mktemp("deal")
    src, exe = d / "deal.cpp", d / "deal"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", f"-I{ROOT / 'paper_2602_09323_amd' / 'csrc'}", f"-I{ROOT / 'include'}",
                    str(src), "-o", str(exe)], check=True)
    return exe


@pytest.mark.parametrize("over", [0, 1, 40], ids=["as announced", "longer than announced", "much longer"])
def test_every_tile_once_and_nothing_beyond_the_workspace(walker, over):
    out = subprocess.run([str(walker), str(over)], check=True, capture_output=True, text=True).stdout
    words = out.splitlines()[-1].split()
    assert int(words[0]) > 4000 and int(words[2]) > 1000, out      # many calls, and many that split
    assert int(words[4]) == 0, out

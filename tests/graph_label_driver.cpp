// Host-side test driver (no GPU): the labels that the lanes of a wave read for the chunks of a graph.  Prints OK, or what
// lies outside (exit status 1).
#include "../paper_2201_12023_amd/csrc/graph_label.hpp"

#include <cstdio>
#include <random>
#include <vector>

using namespace alpa;

int main()
{
    std::mt19937 rng(7);
    int bad = 0;
    for (int n_cells : {2, 3, 65, GRAPH_CELLS})
        for (int n_stages : {1, 63, 64, 65, 200}) {
            // the graph, and behind it what memory may hold: anything
            std::vector<int32_t> words(n_stages + 64);
            for (int e = 0; e < n_stages; ++e) {
                const int cell = 1 + (int)(rng() % (n_cells - 1)), behind = (int)(rng() % n_cells);
                words[e] = graph_label_bytes(cell, behind);
                if (graph_label_behind(words[e], true) != 8u * behind || (words[e] & 0xffff) != 8 * cell) ++bad;
            }
            for (size_t e = n_stages; e < words.size(); ++e) words[e] = e % 3 == 0 ? -1 : (int32_t)rng();
            for (int from = 0; from < n_stages; from += 64)
                for (int lane = 0; lane < 64; ++lane) {
                    const uint32_t at = graph_label_behind(words[from + lane], lane < n_stages - from);
                    if (at % 8 != 0 || at + 8 > 8u * n_cells) {
                        if (bad++ < 5) printf("%d cells, %d stages: lane %d of %d reads byte %u\n", n_cells, n_stages, lane, from, at);
                    }
                }
        }
    printf(bad ? "%d outside\n" : "OK\n", bad);
    return bad != 0;
}

// The table of where the front end's groups begin, as the packing kernel's threads write it, against counting units one by one.
// Built by test_frame_shares.py with the host compiler.
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_1912_11040_amd/csrc/pack_device.h"

int main() {
    std::mt19937 rng(5);
    int faults = 0, cases = 0;
    for (int n_utt : {1, 2, 3, 31, 32, 33, 500})
        for (int most : {1, 2, 7, 300})
            for (int slots : {1, 2, 5, 768, 1024, 4096}) {
                std::vector<int> first(n_utt + 1, 0);
                for (int u = 0; u < n_utt; ++u) first[u + 1] = first[u] + (int)(rng() % (most + 1));       // (some have none)
                const int units = first[n_utt];
                if (!units) continue;
                ++cases;
                aug::PackArgs a{};
                a.n_utt = n_utt;
                a.shares.n_groups = units < slots ? units : slots;
                a.shares.per_group = units / a.shares.n_groups;
                a.shares.longer = units % a.shares.n_groups;
                a.frame_first = first.data();
                std::vector<int2> items(a.shares.n_groups, int2{-1, -1});
                a.frame_items = items.data();
                for (int64_t t = 0; t < aug::pack_threads(a); ++t) aug::pack_utterances(a, (int)t);
                int g = 0, next = 0;
                for (int u = 0, unit = 0; u < n_utt; ++u)
                    for (int i = 0; i < first[u + 1] - first[u]; ++i, ++unit)
                        if (unit == next) {
                            if (items[g].x != u || items[g].y != i) ++faults;
                            next += a.shares.per_group + (g < a.shares.longer ? 1 : 0);
                            ++g;
                        }
                if (g != a.shares.n_groups || next != units) ++faults;
            }
    printf("%d cases, %d faults\n", cases, faults);
    return faults != 0;
}

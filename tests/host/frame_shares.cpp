// The table of where the front end's groups begin, as the packing kernel's threads write it, against counting units one by one, and
// how the host shares the units out.
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

    // The sharing itself, from utterance lengths: every unit is one group's, groups differ by one unit at most, none has a long share, and
    // rows without frames are shared too.  With few units allowed they become larger ones.
    for (int n_utt : {1, 3, 40, 700})
        for (int longest : {0, 300, 5000, 3000000})
            for (int spare : {0, 3, 20000})
                for (int slots : {1, 2, 768})
                    for (int width : {1, 13, 40, 128}) for (int64_t limit : {(int64_t)1 << 30, (int64_t)40000, (int64_t)2000}) {
                        const aug::Framing f{400, 160, width, slots};
                        const int64_t unit_rows = 8192 / (width < 2 ? 1 : width < 16 ? 8 : width < 64 ? 32 : 128);
                        std::vector<int64_t> off(1, 0), foff(1, 0);
                        for (int u = 0; u < n_utt; ++u) {
                            const int64_t len = longest ? (int64_t)(rng() % (unsigned)longest) : 0, frames = len < 400 ? 0 : 1 + (len - 400) / 160;
                            off.push_back(off.back() + len);
                            foff.push_back(foff.back() + frames + (spare ? rng() % (unsigned)spare : 0));
                        }
                        ++cases;
                        const aug::FrameShares s = aug::share_frames(n_utt, off.data(), foff.data(), f, limit);
                        std::vector<int> first(n_utt + 1, 0);
                        for (int u = 0; u < n_utt; ++u) {
                            const int64_t len = off[u + 1] - off[u], frames = len < 400 ? 0 : 1 + (len - 400) / 160, rows = foff[u + 1] - foff[u];
                            const int64_t units = aug::frame_units(len, rows, f, s.shift);
                            first[u + 1] = first[u] + (int)units;
                            if ((units > 0) != (rows > 0)) ++faults;
                            // a unit holds 16 << shift frames at most, and rows without frames make one for every unit_rows << shift
                            if (((units - (rows - frames) / (unit_rows << s.shift)) << (4 + s.shift)) < frames) ++faults;
                            if (rows - frames > (units + 1) * (unit_rows << s.shift)) ++faults;
                        }
                        const int units = first[n_utt];
                        if (units >= limit || (s.shift > 0) != (aug::share_frames(n_utt, off.data(), foff.data(), f).shift != s.shift)) ++faults;
                        if ((int64_t)s.n_groups * s.per_group + s.longer != units || (s.n_groups ? s.longer >= s.n_groups : units != 0)) ++faults;
                        if (units > 0 && (s.n_groups < (units < slots ? units : slots) || s.per_group >= 2 * aug::kUnitsPerGroup)) ++faults;
                        aug::PackArgs a{};
                        a.n_utt = n_utt;
                        a.shares = s;
                        a.frame_first = first.data();
                        std::vector<int2> items(s.n_groups, int2{-1, -1});
                        a.frame_items = items.data();
                        for (int64_t t = 0; t < aug::pack_threads(a); ++t) aug::pack_utterances(a, (int)t);
                        for (int g = 0, u = 0; g < s.n_groups; ++g) {
                            const int begin = g * s.per_group + (g < s.longer ? g : s.longer);
                            while (first[u + 1] <= begin) ++u;
                            if (items[g].x != u || items[g].y != begin - first[u]) { ++faults; break; }
                        }
                    }
    printf("%d cases, %d faults\n", cases, faults);
    return faults != 0;
}

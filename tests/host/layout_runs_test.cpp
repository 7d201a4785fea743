// layout_runs_test.cpp -- which wave of the layout's rank kernel ranks which entries, on the
// host, from the functions that the launch and the kernel use.  Arguments: groups of
// "entries experts".  For each, with 4- and (up to 512 experts) 16-wave workgroups: every
// entry belongs to exactly one wave, and to the tile that counted it.
#include "ep_internal.h"

#include <cstdio>
#include <cstdlib>
#include <vector>

int main(int argc, char **argv) {
    int bad = 0;
    for (int i = 1; i + 1 < argc; i += 2) {
        const uint32_t n = (uint32_t)std::atoll(argv[i]);
        const int32_t E = std::atoi(argv[i + 1]);
        const ep::LayoutGeom g = ep::layout_geometry(n, E);
        const uint32_t tile_entries = (uint32_t)(g.waves * ep::kWave * g.rounds);
        for (int waves : {4, 16}) {
            if (waves == 16 && E > 512)
                continue;
            const int threads = waves * ep::kWave;
            const ep::LayoutRuns r = ep::layout_runs(tile_entries, g.tiles, threads);
            std::vector<uint8_t> owners(n, 0);
            uint64_t strangers = 0, twice = 0, none = 0;
            for (uint32_t tile = 0; tile < g.tiles; ++tile)
                for (uint32_t run = 0; run < r.runs; ++run)
                    for (int w = 0; w < waves; ++w) {
                        const ep::EntryRange e =
                            ep::layout_wave_run(tile, tile_entries, run, r.rounds, threads, w, n);
                        for (uint32_t j = e.begin; j < e.end && j < n; ++j) {
                            strangers += j / tile_entries != tile;
                            twice += owners[j]++ != 0;
                        }
                        strangers += e.end > n && e.begin < e.end;
                    }
            for (uint8_t o : owners)
                none += o == 0;
            std::printf("%u entries, %d experts, %d waves: %lld tiles, %u runs of %d rounds: %llu of another tile, "
                        "%llu twice, %llu nowhere\n", n, E, waves, (long long)g.tiles, r.runs, r.rounds,
                        (unsigned long long)strangers, (unsigned long long)twice, (unsigned long long)none);
            bad += strangers || twice || none;
        }
    }
    return bad ? 1 : 0;
}

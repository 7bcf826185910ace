// Host check of the Z-type sums of a level launch: workgroups of a circuit's
// first step, which is also its last, that do not hold index 0 store zeros and
// leave zero sums, whatever an earlier workgroup left in LDS and in whatever
// order the waves run.  Exit status 0 = all passed.
#include "sweep_replay.h"

#include "../paper_2308_01999_amd/csrc/sv_sweep.hip"

namespace sv {
void pack_matrix(sv_dtype_t, int, int, int, const double*, int, void*) {}
void set_error(const std::string&) {}
}  // namespace sv

using namespace sv;

int main()
{
    int fails = 0, groups = 0;
    for (int n : {13, 15})
        for (uint64_t per : {1, 2, 4}) {
            // three blocks on the lowest qubits: one step of several tiles
            std::vector<double> m(2 * 1024, 0.0);
            for (int i = 0; i < 32; ++i) m[2 * (i * 32 + i)] = 1.0;
            std::vector<FusedBlock> blocks(3);
            for (int b = 0; b < 3; ++b) {
                blocks[b].k = 5;
                for (int a = 0; a < 5; ++a) blocks[b].targets[a] = 2 * b + a;
                blocks[b].m = m.data();
            }
            SweepRules rules;
            rules.keep_order = rules.pad_all = true;
            const auto steps = plan_sweeps(SV_C64, n, 256, blocks.data(), 0, 3, rules);
            if (steps.size() != 1) return 3;
            SweepArgs a = steps[0].args;
            a.warm_lines = 0;
            a.tiles_per_wg = std::min(per, a.n_tiles);
            while ((uint64_t(1) << a.trot) < a.tiles_per_wg) ++a.trot;
            std::vector<char> buf(sweep_bytes(SV_C64, steps[0]) + 256);
            char* desc = buf.data() + (-reinterpret_cast<uintptr_t>(buf.data()) & 255);
            pack_sweep(SV_C64, steps[0], blocks.data(), desc);
            const uint64_t masks[3] = {1, uint64_t(1) << (n - 1), 3};
            for (uint64_t wg = 1; wg * a.tiles_per_wg < a.n_tiles; ++wg, ++groups) {
                std::vector<float> state(size_t(2) << n, 7.f);
                alignas(16) static char lds[8 << 12];
                alignas(16) static double acc[4 * (kZSumsMax + 1)];
                std::fill(acc, acc + 4 * (kZSumsMax + 1), 1e3);  // an earlier workgroup's sums
                double out[4] = {-1, -1, -1, -1};
                const ZSums zs{masks, 3, out, acc};
                run_workgroup(256, [&] {
                    sweep_tiles<float, 12, 256, false, false, false, true, true>(
                        reinterpret_cast<char*>(state.data()), reinterpret_cast<const SweepBlock*>(desc),
                        desc + ((sizeof(SweepBlock) * 3 + 255) & ~size_t(255)), a, wg, lds, zs, nullptr);
                });
                for (double v : out) fails += v != 0.0;
                const auto zeros = std::count(state.begin(), state.end(), 0.f);
                fails += zeros != int64_t(a.tiles_per_wg) * 2 << 12;
            }
        }
    std::printf("workgroups %d fails %d\n", groups, fails);
    return fails ? 1 : 0;
}

// Host check, built with -fsanitize=alignment: a sweep of several blocks reads
// their descriptors, 80 bytes apart, with the alignment they have.  Exit
// status 0 = all passed.
#include "sweep_replay.h"

#include "../paper_2308_01999_amd/csrc/sv_sweep.hip"

namespace sv {
void pack_matrix(sv_dtype_t, int, int, int, const double*, int, void*) {}
void set_error(const std::string&) {}
}  // namespace sv

using namespace sv;

int main()
{
    const int n = 14;
    std::vector<double> m(2 * 1024, 0.0);
    std::vector<FusedBlock> blocks(4);
    for (int b = 0; b < 4; ++b) {
        blocks[b].k = 5;
        for (int a = 0; a < 5; ++a) blocks[b].targets[a] = b + a;
        blocks[b].m = m.data();
    }
    const auto steps = plan_sweeps(SV_C64, n, 256, blocks.data(), 0, 4);
    if (steps.size() != 1) return 3;
    SweepArgs a = steps[0].args;
    a.warm_lines = 0;
    std::vector<char> buf(sweep_bytes(SV_C64, steps[0]) + 256);
    char* desc = buf.data() + (-reinterpret_cast<uintptr_t>(buf.data()) & 255);
    pack_sweep(SV_C64, steps[0], blocks.data(), desc);
    std::vector<float> state(size_t(2) << n, 1.f);
    alignas(16) static char lds[8 << 12];
    run_workgroup(256, [&] {
        sweep_tiles<float, 12, 256, false>(reinterpret_cast<char*>(state.data()),
                                           reinterpret_cast<const SweepBlock*>(desc),
                                           desc + ((sizeof(SweepBlock) * 4 + 255) & ~size_t(255)), a, 1, lds,
                                           ZSums{nullptr, -1, nullptr, nullptr}, nullptr);
    });
    std::puts("passed");
    return 0;
}

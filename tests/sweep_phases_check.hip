// Host check of the phases that pack_sweep leaves for a coupled block: a
// coupled qubit that the state does not have is always 0, so the packed block
// is the one without it.  Exit status 0 = all passed.
#include "../paper_2308_01999_amd/csrc/sv_sweep.hip"

#include <cstdio>
#include <vector>

namespace sv {
void pack_matrix(sv_dtype_t, int, int, int, const double*, int, void*) {}
}  // namespace sv

using namespace sv;

// The buffer of a sweep of one block on qubits 0-4 of 22 with these couplings.
static std::vector<char> packed(const std::vector<int>& qubits)
{
    std::vector<double> m(2 * 1024, 0.25), phases(5 * qubits.size());
    FusedBlock b;
    b.k = 5;
    for (int a = 0; a < 5; ++a) b.targets[a] = a;
    b.m = m.data();
    b.n_couple = int(qubits.size());
    for (size_t c = 0; c < qubits.size(); ++c) {
        b.couple_q[c] = qubits[c];
        for (int a = 0; a < 5; ++a) phases[a * qubits.size() + c] = 0.3 + 0.1 * a + 0.01 * qubits[c];
    }
    b.couple = phases.data();
    const auto steps = plan_sweeps(SV_C64, 22, 256, &b, 0, 1);
    if (steps.size() != 1 || !steps[0].multi || !steps[0].coupled) return {};
    std::vector<char> buf(sweep_bytes(SV_C64, steps[0]));
    pack_sweep(SV_C64, steps[0], &b, buf.data());
    return buf;
}

int main()
{
    int fails = 0;
    const auto want = packed({5, 9, 21});
    fails += want.empty();
    for (int q : {22, 35, 36, 40, 56, 63}) fails += packed({5, 9, 21, q}) != want;
    std::printf("fails %d\n", fails);
    return fails ? 1 : 0;
}

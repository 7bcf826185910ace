// Host check of the phases that pack_sweep leaves for a coupled block: a
// coupled qubit that the state does not have is always 0, so the packed block
// is the one without it; and the sums that the kernel takes (outside the tile, the
// wave's part, the lane's) are the phases to 2^-63 turns a term, as far as a double
// holds them.  Exit status 0 = all passed.
#include "../paper_2308_01999_amd/csrc/sv_sweep.hip"

#include <cstdio>
#include <random>
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

// A sweep of two coupled blocks on n qubits: every target's phase of every group of a tile.
static int wrong_sums(int n, int tile_seed)
{
    std::mt19937_64 rng(tile_seed);
    std::vector<double> m(2 * 1024, 0.25), phases(2 * 5 * 7);
    for (double& p : phases) p = std::ldexp(double(rng() >> 11), -50) - 4.0;
    std::vector<FusedBlock> b(2);
    for (int i = 0; i < 2; ++i) {
        std::vector<int> q(n);
        for (int j = 0; j < n; ++j) q[j] = j;
        std::shuffle(q.begin() + 5, q.end(), rng);
        b[i].k = 5;
        for (int a = 0; a < 5; ++a) b[i].targets[a] = i + a;
        b[i].m = m.data();
        b[i].n_couple = 7;
        for (int c = 0; c < 7; ++c) b[i].couple_q[c] = c == 0 ? 5 * (1 - i) : q[6 + c];
        b[i].couple = phases.data() + i * 35;
    }
    std::swap(b[1].couple_q[0], b[1].couple_q[3]);
    const auto steps = plan_sweeps(SV_C64, n, 256, b.data(), 0, 2);
    if (steps.size() != 1 || !steps[0].coupled) return 1000;
    const SweepStep& st = steps[0];
    std::vector<char> buf(sweep_bytes(SV_C64, st));
    pack_sweep(SV_C64, st, b.data(), buf.data());
    const auto* d = reinterpret_cast<const SweepBlock*>(buf.data());
    const char* mats = buf.data() + ((sizeof(SweepBlock) * 2 + 255) & ~size_t(255));
    // the tile-local index of each slot
    std::vector<uint32_t> local(size_t(1) << st.tile_bits);
    for (uint32_t i = 0; i < local.size(); ++i) local[slot_bytes(SV_C64, i) / 8] = i;
    uint64_t t = rng() % st.args.n_tiles, origin = t << st.args.L;
    for (int j = 0; j < st.args.n_hi; ++j) origin += origin & st.args.hi_mask[j];
    int wrong = 0;
    for (int i = 0; i < 2; ++i) {
        const auto& cp = *(reinterpret_cast<const SweepCouple*>(mats + (i + 1) * matrix_stride(SV_C64, st)) - 1);
        for (uint32_t g = 0; g < 1u << (st.tile_bits - 5); ++g) {
            uint32_t at = 0;
            for (int j = 0; j < st.tile_bits - 5; ++j) at ^= (g >> j) & 1 ? d[i].grp[j] : 0;
            uint64_t index = origin;
            for (int p = 0; p < st.tile_bits; ++p)
                if ((local[at / 8] >> p) & 1) index += st.args.bit_off[p] / 8;
            for (int a = 0; a < 5; ++a) {
                uint64_t u = cp.wave[a][g >> 5] + cp.lane[a][g & 31];
                for (int q = 0; q < n; ++q) u += (origin >> q) & 1 ? cp.out[a][q] : 0;
                long double want = 0;
                for (int c = 0; c < 7; ++c)
                    if ((index >> b[i].couple_q[c]) & 1) {
                        const double turn = b[i].couple[a * 7 + c] / 6.283185307179586476925286766559;
                        want += turn - std::floor(turn);
                    }
                want = std::ldexp(want, 64);
                const auto error = int64_t(u - uint64_t(std::fmod(want, 0x1p64L)));
                // a term: 2^-63 turns of the format, 2^-54 of the double
                wrong += std::llabs(error) > 7 * (2 + 1024);
            }
        }
    }
    return wrong;
}

int main()
{
    int fails = 0;
    for (int seed = 0; seed < 20; ++seed) fails += wrong_sums(22 + seed % 4, seed) != 0;
    const auto want = packed({5, 9, 21});
    fails += want.empty();
    for (int q : {22, 35, 36, 40, 56, 63}) fails += packed({5, 9, 21, q}) != want;
    std::printf("fails %d\n", fails);
    return fails ? 1 : 0;
}

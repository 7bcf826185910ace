// Host-side check of the multi-block sweeps: plans random programs with the
// library's own plan_sweeps and replays, on the CPU, the index arithmetic that
// k_sweep performs with the descriptors of pack_sweep.  Checks that a plan
// holds every block once and keeps the order of blocks that share a qubit
// (and the whole order on states below the reorder size), that a sweep's
// tiles cover every amplitude once, and that each group's members differ from
// its base exactly by the block's target bits; the same for the steps of a
// batch's level path.  Exit status 0 = all passed.
#include "../paper_2308_01999_amd/csrc/sv_sweep.hip"

#include <cstdio>
#include <random>
#include <vector>

namespace sv {
void pack_matrix(sv_dtype_t, int, int, int, const double*, int, void*) {}  // matrices are not checked here
}  // namespace sv

using namespace sv;

static int fails = 0, sweeps = 0, reordered = 0;

static void fail(const char* what, int n, sv_dtype_t dt, int step)
{
    if (++fails <= 10) printf("FAIL %s: n=%d dtype=%d step=%d\n", what, n, int(dt), step);
}

static uint64_t h_origin(uint64_t t, const SweepArgs& a)
{
    if (a.trot > 0) t = ((t & ((uint64_t(1) << a.trot) - 1)) << (a.lg_tiles - a.trot)) | (t >> a.trot);
    uint64_t v = t << a.L;
    for (int j = 0; j < a.n_hi; ++j) {
        v += v & a.hi_mask[j];
    }
    return v;
}

static uint32_t h_group(uint32_t v, const uint32_t* grp)
{
    uint32_t o = 0;
    for (int j = 0; v >> j; ++j)
        if ((v >> j) & 1) o ^= grp[j];
    return o;
}

static void check_sweep(sv_dtype_t dt, int n, const SweepStep& st, const FusedBlock* blocks, int step)
{
    ++sweeps;
    const SweepArgs& a = st.args;
    const int T = st.tile_bits, apv = dt == SV_C64 ? 2 : 1;
    const uint32_t bytes = dt == SV_C64 ? 8 : 16;
    const int nt = (1 << T) / apv / 8;
    const bool one = n <= T;
    if (!one && (a.L + a.n_hi != T || a.n_tiles != uint64_t(1) << (n - T))) return fail("tile shape", n, dt, step);
    // the tile's global offsets, through the kernel's lane and vector parts
    std::vector<uint64_t> glob(size_t(1) << T, ~uint64_t(0));
    for (int u = 0; u < 8; ++u)
        for (int tid = 0; tid < nt; ++tid) {
            const uint32_t local = uint32_t(u * nt + tid) * apv, lane_mask = uint32_t(64 * apv - 1);
            uint64_t loff = 0, roff = 0;
            for (int p = 0; p < T; ++p)
                if ((local >> p) & 1) ((lane_mask >> p) & 1 ? loff : roff) += a.bit_off[p];
            if (loff >> 32 || loff % bytes || roff % bytes) fail("lane offset", n, dt, step);
            loff /= bytes;
            roff /= bytes;
            const uint32_t s = slot_bytes(dt, uint32_t(u * nt + tid) * apv) / bytes;
            for (int e = 0; e < apv; ++e) {
                if (s + e >= glob.size() || glob[s + e] != ~uint64_t(0)) return fail("tile slot taken twice", n, dt, step);
                glob[s + e] = roff + loff + e;
            }
        }
    // every amplitude of the state once (states of up to 16 qubits)
    if (!one && n <= 16) {
        std::vector<char> seen(size_t(1) << n, 0);
        for (uint64_t t = 0; t < a.n_tiles; ++t)
            for (uint64_t g : glob) {
                const uint64_t i = h_origin(t, a) + g;
                if (i >= seen.size() || seen[i]++) return fail("amplitude covered twice", n, dt, step);
            }
    } else if (!one) {
        uint64_t top = h_origin(a.n_tiles - 1, a), most = 0;
        for (uint64_t g : glob) most = std::max(most, g);
        if (top + most != (uint64_t(1) << n) - 1) fail("last amplitude", n, dt, step);
    }
    std::vector<char> buf(sweep_bytes(dt, st));
    pack_sweep(dt, st, blocks, buf.data());
    const auto* d = reinterpret_cast<const SweepBlock*>(buf.data());
    for (size_t j = 0; j < st.blocks.size(); ++j) {
        const FusedBlock& b = blocks[st.blocks[j]];
        const int k = std::min(d[j].kind, 5);
        std::vector<char> used(size_t(1) << T, 0);
        for (uint32_t g = 0; g < (1u << (T - k)); ++g) {
            const uint32_t base = h_group(g, d[j].grp) / bytes;
            for (int r = 0; r < (1 << k); ++r) {
                const uint32_t s = base ^ (d[j].off(r) / bytes);
                if (s >= used.size() || used[s]++) return fail("group member taken twice", n, dt, step);
                uint64_t want = glob[base];
                for (int q = 0; q < b.k; ++q)
                    if ((r >> q) & 1) want += uint64_t(1) << b.targets[q];
                // the padding qubits' part of the index is free
                if (r < (1 << b.k) && glob[s] != want) return fail("group member misplaced", n, dt, step);
            }
        }
    }
}

int main()
{
    std::mt19937 rng(7);
    std::vector<double> m(2 * 1024, 0.0);
    for (sv_dtype_t dt : {SV_C64, SV_C128})
        for (int n = 1; n <= 36; ++n)
            for (int rep = 0; rep < 6; ++rep) {
                std::vector<FusedBlock> blocks(rep == 5 ? 130 : 24);
                for (auto& b : blocks) {
                    const bool local = rep % 2 == 0;  // neighbouring or scattered targets
                    b.k = std::min(n, rep < 2 ? 5 : 1 + int(rng() % 6));
                    std::vector<int> q(n);
                    for (int i = 0; i < n; ++i) q[i] = i;
                    std::shuffle(q.begin(), q.end(), rng);
                    const int lo = int(rng() % uint32_t(n - b.k + 1));
                    for (int a = 0; a < b.k; ++a) b.targets[a] = local ? lo + a : q[a];
                    std::sort(b.targets, b.targets + b.k);
                    b.m = m.data();
                    b.diagonal = rep == 4 && rng() % 4 == 0;
                    // phase couplings to qubits outside the targets
                    if (rep == 1 && n > b.k && rng() % 2) {
                        b.n_couple = 1;
                        b.couple_q[0] = q[b.k + int(rng() % uint32_t(n - b.k))];
                        b.couple = m.data();
                    }
                }
                const int first = rep == 3 ? 3 : 0, end = int(blocks.size()) - (rep == 3 ? 2 : 0);
                // the rules of a batch's level path (complex64, blocks of up
                // to five qubits): every block in order in tiles of 2^12
                for (int spread : {0, 12}) {
                    if (dt != SV_C64 || n < 13 || n > 34 || rep >= 4) continue;
                    std::vector<FusedBlock> five = blocks;
                    for (auto& b : five) b.k = std::min(b.k, 5), b.n_couple = 0;
                    SweepRules rules;
                    rules.keep_order = rules.pad_all = true;
                    rules.spread_lo = spread;
                    int next = first, step = 0;
                    for (const SweepStep& st : plan_sweeps(dt, n, 256, five.data(), first, end, rules)) {
                        if (!st.multi || !st.padded || st.tile_bits != 12) fail("batch step", n, dt, step);
                        for (int i : st.blocks)
                            if (i != next++) fail("batch order", n, dt, step);
                        check_sweep(dt, n, st, five.data(), step++);
                    }
                    if (next != end) fail("batch block lost", n, dt, step);
                }
                const auto plan = plan_sweeps(dt, n, 256, blocks.data(), first, end);
                std::vector<int> order;
                int step = 0;
                for (const SweepStep& st : plan) {
                    for (int i : st.blocks) order.push_back(i);
                    if (!st.multi && st.blocks.size() > 1) fail("step kind", n, dt, step);
                    if (st.multi) check_sweep(dt, n, st, blocks.data(), step);
                    ++step;
                }
                std::vector<int> at(blocks.size(), -1);
                for (size_t i = 0; i < order.size(); ++i) {
                    if (order[i] < first || order[i] >= end || at[order[i]] >= 0) fail("block repeated", n, dt, int(i));
                    at[order[i]] = int(i);
                }
                if (int(order.size()) != end - first) fail("block lost", n, dt, 0);
                for (int i = first; i < end; ++i)
                    for (int j = i + 1; j < end; ++j) {
                        if (at[i] < at[j]) continue;
                        ++reordered;
                        if (n < 22) fail("order changed on a small state", n, dt, i);
                        auto touched = [&](const FusedBlock& b) {
                            uint64_t t = qubit_mask(b);
                            for (int c = 0; c < b.n_couple; ++c) t |= uint64_t(1) << b.couple_q[c];
                            return t;
                        };
                        if ((qubit_mask(blocks[i]) & touched(blocks[j])) | (touched(blocks[i]) & qubit_mask(blocks[j])))
                            fail("blocks that do not commute swapped", n, dt, i);
                    }
            }
    printf("sweeps %d reordered pairs %d fails %d\n", sweeps, reordered, fails);
    return fails ? 1 : 0;
}

// Sweeps that apply several fused blocks to each tile of a state (sv_sweep.hip):
// their device descriptors, and the host's plan of which blocks share a sweep.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "sv_internal.h"

namespace sv {

// One block of a sweep (device).  Tile-local positions: index bit q of the
// state below L is q, the others L plus their rank in hi_pos.
struct SweepBlock {
    uint32_t ins[5];   // group index -> tile-local base: the bits at and above each target, ascending
    int32_t k;         // matrix qubits as swept (5: matrix cores)
    uint32_t off[32];  // byte offset of matrix index r in the swizzled tile
    uint32_t mat;      // byte offset of the packed matrix in the sweep's buffer
    int32_t rows;      // five qubits on the vector units (block5_rows)
};

// Geometry of a sweep (kernel argument).
constexpr int kSweepMaxHigh = 12;
struct SweepArgs {
    uint64_t n_tiles;
    uint64_t tiles_per_wg;
    uint64_t amps;              // amplitudes of the state if it is a single tile
    int32_t L;                  // run bits
    int32_t n_hi;               // T - L
    int32_t hi_pos[kSweepMaxHigh];
    int32_t trot, lg_tiles;     // tile order, as TileArgs
    int32_t n_blocks;
};

// A step of a program: one block on its own kernel (blocks.size() == 1,
// multi false) or a sweep of the listed blocks in this order.
struct SweepStep {
    bool multi = false;
    std::vector<int> blocks;
    SweepArgs args{};
    int tile_bits = 0;
};

// The steps of blocks [first, end) of f on an n-qubit state.
std::vector<SweepStep> plan_sweeps(sv_dtype_t dt, int n, int cu_count, const FusedBlock* blocks, int first, int end);

// Device buffer of a multi step: its descriptors, then its packed matrices.
size_t sweep_bytes(sv_dtype_t dt, const SweepStep& st, const FusedBlock* blocks);
void pack_sweep(sv_dtype_t dt, const SweepStep& st, const FusedBlock* blocks, void* dst);
void launch_sweep(sv_handle_s* h, sv_dtype_t dt, void* psi, const SweepStep& st, const void* buffer);

}  // namespace sv

// Sweeps that apply several fused blocks to each tile of a state (sv_sweep.hip):
// their device descriptors, and the host's plan of which blocks share a sweep.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "sv_internal.h"

namespace sv {

// How a block is swept: 1-4 qubits as they are (states of one tile), five on
// the matrix cores or on the vector units (block_rows); added to kSweepMfma5
// of a split sweep: the block is coupled, and its products are FP32.
constexpr int32_t kSweepMfma5 = 5, kSweepRows5 = 6;
constexpr int32_t kSweepCoupled = 16, kSweepFp32 = 32;

// One block of a sweep (device).  Tile-local positions: index bit q of the
// state below L is q, the others L plus their rank among the tile's high bits.
struct alignas(16) SweepBlock {
    uint32_t bit[5];   // byte offset in the swizzled tile of each bit of the matrix index
    int32_t kind;
    uint32_t grp[12];  // and of each bit of the group index
    uint32_t pad[2];
    // byte offset of matrix index r
    __host__ __device__ __forceinline__ constexpr uint32_t off(int r) const
    {
        uint32_t o = 0;
        for (int a = 0; a < 5; ++a) o ^= ((r >> a) & 1) ? bit[a] : 0u;
        return o;
    }
};
constexpr int kSweepBlockWords = int(sizeof(SweepBlock) / 4);
static_assert(kSweepBlockWords <= 64, "a wave holds a descriptor, one word a lane");
static_assert(sizeof(SweepBlock) == 80, "descriptors lie one behind the other, 16-byte aligned");

// Bytes from one block's packed matrix to the next's.
constexpr uint32_t sweep_matrix_stride(bool c64) { return c64 ? 12u << 10 : 16u << 10; }

// The phases of a block of coupled fusion, behind each matrix of a coupled sweep.
// Target a's phase is the sum of the terms of the coupled qubits that are set,
// as fixed-point turns of 2^-64, whose sum wraps by itself.
struct SweepCouple {
    uint64_t out[5][36];   // the term of qubit q outside the tile
    uint64_t wave[5][8];   // the terms of the qubits that a wave's groups share
    uint64_t lane[5][32];  // and of those that a lane's group adds, lane % 32
    uint32_t pad[8];
};
static_assert(sizeof(SweepCouple) == 3072, "a matrix behind it stays aligned");

// Geometry of a sweep (kernel argument).
constexpr int kSweepMaxHigh = 12;
struct SweepArgs {
    uint64_t n_tiles;
    uint64_t tiles_per_wg;
    uint64_t amps;                     // amplitudes of the state
    uint64_t bit_off[13];              // byte offset of tile-local bit p
    uint64_t hi_mask[kSweepMaxHigh];   // the bits at and above each high bit of the tile
    int32_t L;                         // run bits
    int32_t n_hi;                      // T - L
    int32_t trot, lg_tiles;            // tile order, as TileArgs
    int32_t n_blocks;
    int32_t warm_lines;                // 128-byte lines of descriptors and matrices to bring to the L2 first
};

// A step of a program: one block on its own kernel (multi false) or a sweep
// of the listed blocks in this order.
struct SweepStep {
    bool multi = false;
    std::vector<int> blocks;
    SweepArgs args{};
    bool padded = false;  // blocks of fewer than five qubits are swept as five-qubit ones
    bool split = false;   // products of bf16 pieces (block5_split)
    bool coupled = false; // some of the blocks are coupled
    int tile_bits = 0;
    int hi_pos[kSweepMaxHigh] = {};
};

struct SweepRules {
    bool few_alone = false;   // calls of few blocks on small states launch each on its own
    bool keep_order = false;  // blocks in program order on states of any size
    bool pad_all = false;     // every block is swept as a five-qubit one
    int spread_lo = 0;        // > 0: tiles with runs of at most 1 KiB, filled up with free bits from here up
};

// The steps of blocks [first, end) of f on an n-qubit state.
std::vector<SweepStep> plan_sweeps(sv_dtype_t dt, int n, int cu_count, const FusedBlock* blocks, int first, int end,
                                   const SweepRules& rules = SweepRules());

// Device buffer of a multi step: its descriptors, then its packed matrices.
size_t sweep_bytes(sv_dtype_t dt, const SweepStep& st);
void pack_sweep(sv_dtype_t dt, const SweepStep& st, const FusedBlock* blocks, void* dst);
// The same into separate arrays: the blocks' descriptors, and their matrices
// sweep_matrix_stride apart.
void pack_sweep(sv_dtype_t dt, const SweepStep& st, const FusedBlock* blocks, SweepBlock* desc, char* mats);
void launch_sweep(sv_handle_s* h, sv_dtype_t dt, void* psi, const SweepStep& st, const void* buffer);

}  // namespace sv

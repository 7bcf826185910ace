// Sweeps of several fused blocks (Sec. II-B: fused gates; the state is read
// and written once per sweep instead of once per block).
//
// A tile holds 2^T amplitudes: the low L index bits and T - L chosen higher
// ones.  A run of blocks whose targets all lie among a tile's bits can be
// applied to the tile while it sits in LDS, one after the other, so the state
// crosses HBM once for the whole run.  A state of at most 2^T amplitudes is
// one tile: its whole program runs in one launch of one workgroup.
//
// Per block, each wave gathers whole groups (the 2^k amplitudes a matrix
// mixes).  Below 22 qubits it multiplies them in the same order of operations
// as the single-block sweeps (sv_tile.h, sv_apply.hip), so a state has the same
// bits whichever sweep ran.
//
// What bounds it: HBM for a block alone (30 qubits complex64: 2.9 ms), the matrix
// cores for several.  A block costs a wave 48 MFMAs: of v_mfma_f32_32x32x2_f32
// 3072 cycles (1.7 ms a block at 30 qubits), of v_mfma_f64_16x16x4_f64 the same,
// of v_mfma_f32_32x32x16_bf16 1536 (block5_split, states of 22 qubits and
// more).  A tile is 32 KiB (64 KiB and 512 threads where plan_sweeps says) and a
// workgroup 256 threads and one tile: the runs of 128 bytes that this leaves for
// eight free bits stream at 4.6-5.4 TB/s, and four workgroups a CU, at most 128
// vector registers a thread (the coupled forms spill 11 around a tile's blocks,
// none inside them), hide each other's loads, stores and barriers.  They do it
// better than three that load their next tile during a tile's blocks: loads
// return in order, so a matrix behind a tile waits for HBM (28 qubits, sweeps of
// 4 blocks: complex64 1.38 -> 1.18 ms, complex128 on 27 qubits 1.91 -> 1.83).
// Measured, before (a sweep per block) and after: 30-qubit brickwork circuit
// of depth 20, complex64, 52 blocks in 20 sweeps, 156 -> 92 ms; 28-qubit
// random CNOT/CP circuit, complex128, 71 -> 48 ms; 19-qubit circuit on random
// pairs, complex128, 660 -> 310 us; 14 qubits complex64 as a recorded graph,
// 155 -> 91 us; 12 qubits complex128 194 -> 117 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "sv_batch.h"
#include "sv_tile.h"

namespace sv {
namespace {

using namespace tile;

// Most blocks of one sweep: its descriptors and matrices fit a segment of the
// handle's matrix ring (16 KiB a block at most, 1 MiB).
constexpr size_t kMaxSweepBlocks = 48;

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// LDS slot of tile-local amplitude a: its low bits (5 of complex64's 8-byte
// amplitudes, 4 of complex128's: the 64 banks) XORed with a vector for each
// higher bit that is set.  It is linear over bits: the slot of a group's
// amplitude r is slot(base) ^ slot(off(r)), one XOR per access with the
// host's swizzled offset as the scalar operand.  complex64's vectors leave
// bit 0 alone, so a pair (i, i + 1) keeps its order and stages as one 16-byte
// slot.  An LDS access is as fast as the bank bits that its lanes reach: with
// the vectors below a wave finds, for any five targets, lane bits among the
// other tile bits (choose_lanes) for which a ds_read_b64 and a ds_write_b64
// take 10.2 cycles in the mean and 12.3 at most (8.7 without any conflict), as
// measured for each rank of the lanes' bits in the banks; the XOR of bits 1-4
// with bits 6-9 and lanes on the lowest free bits took 13.7 and up to 48.
constexpr uint32_t kSlot64[8] = {28, 26, 10, 18, 6, 14, 22, 30};      // of bits 5-12
constexpr uint32_t kSlot128[9] = {11, 13, 7, 9, 3, 14, 12, 6, 10};    // of bits 4-12
template <typename R>
__host__ __device__ __forceinline__ constexpr uint32_t slot(uint32_t a)
{
    uint32_t r = a;
    if constexpr (sizeof(R) == 4)
        for (int p = 5; p < 13; ++p) r ^= (0u - ((a >> p) & 1u)) & kSlot64[p - 5];
    else
        for (int p = 4; p < 13; ++p) r ^= (0u - ((a >> p) & 1u)) & kSlot128[p - 4];
    return r;
}

template <typename R>
struct Amp;
template <>
struct Amp<float> {
    using V = f32x2;       // one amplitude
    using W = f32x4;       // one 16-byte access
    static constexpr int kPerVec = 2;
    static constexpr uint32_t kBytes = 8;
};
template <>
struct Amp<double> {
    using V = f64x2;
    using W = f64x2;
    static constexpr int kPerVec = 1;
    static constexpr uint32_t kBytes = 16;
};

// Global index of tile t's first amplitude (tile order as tile_base).
__device__ __forceinline__ uint64_t tile_origin(uint64_t t, const SweepArgs& a)
{
    if (a.trot > 0) t = ((t & ((uint64_t(1) << a.trot) - 1)) << (a.lg_tiles - a.trot)) | (t >> a.trot);
    t <<= a.L;
    for (int j = 0; j < a.n_hi; ++j) t += t & a.hi_mask[j];
    return t;
}

// An address of a uniform and a lane's 32-bit part, kept in that form: left
// to itself the compiler adds the two in vector registers, two a load, and
// holds them across the blocks.
template <typename T>
using Global = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ Global<T>* lane_address(const void* uniform, uint32_t lane_bytes)
{
    auto u = reinterpret_cast<uint64_t>(uniform);
    asm volatile("" : "+s"(u), "+v"(lane_bytes));
    return reinterpret_cast<Global<T>*>(reinterpret_cast<Global<char>*>(u) + lane_bytes);
}

// Masks of a lane's index bits (all ones where the bit is set).
struct LaneBits {
    uint32_t m[6];
    __device__ __forceinline__ explicit LaneBits(int lane)
    {
#pragma unroll
        for (int b = 0; b < 6; ++b) m[b] = 0u - ((uint32_t(lane) >> b) & 1u);
    }
};

// Byte offset of a group in the swizzled tile: the lane's part (N bits of the
// group index) and the part of the bits above, the same for the whole wave.
template <int N>
__device__ __forceinline__ uint32_t lane_part(const LaneBits& l, const uint32_t* grp)
{
    uint32_t o = 0;
#pragma unroll
    for (int b = 0; b < N; ++b) o ^= l.m[b] & grp[b];
    return o;
}
template <int N>
__device__ __forceinline__ uint32_t wave_part(uint32_t v, const uint32_t* grp)
{
    uint32_t o = 0;
#pragma unroll
    for (int b = 0; b < N; ++b) o ^= ((v >> b) & 1u) ? grp[b] : 0u;
    return o;
}

// A lane's share of a five-qubit matrix, as pack5 lays it out.
template <typename R>
struct Ops;
template <>
struct Ops<float> {
    f32x4 re[4], im[4], sum[4];
    template <bool SUM>
    __device__ __forceinline__ void load(const f32x4* __restrict__ m, int lane)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            re[q] = *lane_address<const f32x4>(m + q * 64, uint32_t(lane) * 16);
            im[q] = *lane_address<const f32x4>(m + 256 + q * 64, uint32_t(lane) * 16);
            if (SUM) sum[q] = *lane_address<const f32x4>(m + 512 + q * 64, uint32_t(lane) * 16);
        }
    }
};
template <>
struct Ops<double> {
    f64x2 re[4], im[4];  // the rows 16 rt + i of one row tile
    __device__ __forceinline__ void load_rows(const f64x2* __restrict__ m, int lane, int rt)
    {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            re[h] = *lane_address<const f64x2>(m + (rt * 4 + h) * 64, uint32_t(lane) * 16);
            im[h] = *lane_address<const f64x2>(m + (8 + rt * 4 + h) * 64, uint32_t(lane) * 16);
        }
    }
    template <bool SUM>
    __device__ __forceinline__ void load(const f64x2* __restrict__ m, int lane)
    {
        load_rows(m, lane, 0);  // block5 loads row tile 1 while it multiplies row tile 0
    }
};

// complex64, five qubits, on v_mfma_f32_32x32x2_f32: one column tile of 32
// groups per wave (the chain of tile_c64_k5_sweep).  in / out: LDS byte address of the
// lane's inputs (matrix columns 2j + half) and outputs (rows 8(r/4) + 4 half +
// r%4) before the XOR with the uniform part of the index.  SUM: Re M + Im M is
// read too (states of fewer than 12 qubits take it as the host rounded it, as
// k_apply_mfma_c64_k5 does), otherwise formed here.
// READY: the lane's matrix entries (complex128: of the first row tile) are in
// `o` already.
template <bool SUM, bool READY>
__device__ __forceinline__ void block5(char* lds, const SweepBlock& b, const f32x4* __restrict__ m, Ops<float>& o,
                                       const LaneBits& lb, uint32_t wave, int lane)
{
    const int half = lane >> 5;
    if (!READY) o.load<SUM>(m, lane);
    const uint32_t base = lane_part<5>(lb, b.grp) ^ wave_part<3>(wave, b.grp + 5);
    uint32_t in = base ^ (half ? b.off(1) : 0u), out = base ^ (half ? b.off(4) : 0u);
    asm volatile("" : "+v"(in), "+v"(out));  // keep (base ^ half part) ^ uniform part: one XOR per access
    f32x2 x[2][4];
    auto fetch = [&](int q) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) x[q & 1][jj] = *reinterpret_cast<const f32x2*>(lds + (in ^ b.off(2 * (4 * q + jj))));
    };
    fetch(0);
    f32x16 p1 = {0}, p2 = {0}, p3 = {0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q < 3) fetch(q + 1);
        const f32x4 vs = SUM ? o.sum[q] : o.re[q] + o.im[q];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const f32x2 xv = x[q & 1][jj];
            p1 = __builtin_amdgcn_mfma_f32_32x32x2f32(o.re[q][jj], xv.x, p1, 0, 0, 0);
            p2 = __builtin_amdgcn_mfma_f32_32x32x2f32(o.im[q][jj], xv.y, p2, 0, 0, 0);
            p3 = __builtin_amdgcn_mfma_f32_32x32x2f32(vs[jj], xv.x + xv.y, p3, 0, 0, 0);
        }
        if (!READY) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
        *reinterpret_cast<f32x2*>(lds + (out ^ b.off(8 * (r / 4) + (r % 4)))) =
            f32x2{p1[r] - p2[r], p3[r] - p1[r] - p2[r]};
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pack_bf16(float x, float y)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x, y}), bf16x2));
}

// x and y as three bf16 each: x = x0 + x1 + x2, x0 = bf16(x), x1 = bf16(x - x0),
// x2 the rest (24 bits in 8 + 8 + 8, both differences exact).  lost: bits 0-15
// take those of the rests, which are zero as long as the parts are exact (they
// are from 2^-110 up: a bf16 holds no bit below 2^-133).
__device__ __forceinline__ void split_bf16(float x, float y, uint32_t& w0, uint32_t& w1, uint32_t& w2, uint32_t& lost)
{
    w0 = pack_bf16(x, y);
    x -= __builtin_bit_cast(float, w0 << 16);
    y -= __builtin_bit_cast(float, w0 & 0xffff0000u);
    w1 = pack_bf16(x, y);
    x -= __builtin_bit_cast(float, w1 << 16);
    y -= __builtin_bit_cast(float, w1 & 0xffff0000u);
    w2 = pack_bf16(x, y);
    lost |= __builtin_bit_cast(uint32_t, x) | __builtin_bit_cast(uint32_t, y);
}

__device__ __forceinline__ f32x2 cmul(f32x2 a, f32x2 b)
{
    return f32x2{fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x)};
}

// exp(2 pi i u / 2^64) by the Taylor polynomials of sine and cosine on the
// quadrant's [-pi/4, pi/4] (the terms left out are below 2e-9).
__device__ __forceinline__ f32x2 unit(uint64_t u)
{
    const uint32_t hi = uint32_t(u >> 32), q = (hi + 0x20000000u) >> 30;
    const float turn = fmaf(float(uint32_t(u)), 0x1p-32f, float(int32_t(hi - (q << 30))));
    const float y = turn * 1.46291807926715969e-9f;  // 2 pi / 2^32
    const float z = y * y;
    const float sn = fmaf(y * z, fmaf(z, fmaf(z, fmaf(z, 2.75573192e-6f, -1.98412698e-4f), 8.33333333e-3f), -1.66666667e-1f), y);
    const float cs = fmaf(z, fmaf(z, fmaf(z, fmaf(z, fmaf(z, -2.75573192e-7f, 2.48015873e-5f), -1.38888889e-3f), 4.16666667e-2f), -0.5f), 1.f);
    const float a = (q & 1u) ? -sn : cs, b = (q & 1u) ? cs : sn;
    return (q & 2u) ? f32x2{-a, -b} : f32x2{a, b};
}

// One half (columns 16 s ...) of a lane's share of a matrix in pieces: three of
// Re M, three of Im M.
struct SplitOps {
    u32x4 re[3], im[3];
    __device__ __forceinline__ void load(const u32x4* __restrict__ m, int s, int lane)
    {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            re[q] = *lane_address<const u32x4>(m + (q * 2 + s) * 64, uint32_t(lane) * 16);
            im[q] = *lane_address<const u32x4>(m + (6 + q * 2 + s) * 64, uint32_t(lane) * 16);
        }
    }
};

// complex64, five qubits, on v_mfma_f32_32x32x16_bf16: matrix and amplitudes as
// three bf16 each (together all 24 bits), and of their nine products the six down
// to 2^-16 of the first, summed in FP32: the five small ones of all 32 columns
// first, then the largest, so that a sum is rounded at its full size only as
// often as largest products are added (two to eight times; the FP32 kernels
// round each of 32 products).  The three products left out are at most 2^-24 of
// the whole one and 2^-27.5 in the mean square, the rounding of an FP32 product
// 2^-24 and 2^-25.2.  Four real products instead of the three of the FP32
// kernels (Re M, Im M, Re M + Im M), whose differences cancel.  Of a dense block
// on random amplitudes the error against 64 bits is 0.52e-7 of the 2-norm (FP32
// kernels 1.49e-7), of a 30-qubit circuit's state 3.8e-7 (9.9e-7).
// The wave takes FP32 products of the same matrix where the parts do not hold an
// amplitude (below 2^-110, and next to the largest float), and for a matrix for
// which the host chose them (kSweepFp32).
// A block costs 1536 cycles of the matrix cores instead of 3072, and about 290
// vector instructions of which 176 split the amplitudes (a difference as
// v_dot2_f32_bf16, one instruction for two, was no gain: it takes the matrix
// cores' time).  In a sweep a block takes 0.18 ms on 28 qubits, 0.41 on FP32.
// The order of the products and the check for lost bits cost 0.9% of a 30-qubit
// circuit (sums of one half of the columns after the other, unchecked: 92.6 against
// 93.4 ms, error 6.1e-7).  A lane's outputs are its inputs' slots.
// COUPLED: a block with kSweepCoupled first multiplies each amplitude by its
// phase, exp of the sum of the phases of the targets set in it; turns: their
// parts from outside the tile and from the wave's part of the group index, cp: from
// the lane's.
template <bool COUPLED>
__device__ __forceinline__ void block5_split(char* lds, const SweepBlock& b, const u32x4* __restrict__ m,
                                             const u32x4* __restrict__ next, SplitOps& o, const LaneBits& lb,
                                             uint32_t wave, int lane, const SweepCouple* __restrict__ cp,
                                             const uint64_t* turns)
{
    uint32_t at = lane_part<5>(lb, b.grp) ^ wave_part<3>(wave, b.grp + 5) ^ (lb.m[5] & b.off(4));
    asm volatile("" : "+v"(at));
    const bool coupled = COUPLED && (b.kind & kSweepCoupled);
    // the phase factor of each target
    auto phases = [&](f32x2* w) {
        uint64_t u[5];
#pragma unroll
        for (int a = 0; a < 5; ++a) u[a] = *lane_address<const uint64_t>(cp->lane[a], uint32_t(lane & 31) * 8);
#pragma unroll
        for (int a = 0; a < 5; ++a) w[a] = unit(u[a] + turns[a]);
    };
    f32x16 re = {0}, im = {0};
    uint32_t lost = 0;
#define SV_MFMA(A, X, C) \
    C = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, A), __builtin_bit_cast(bf16x8, X), C, 0, 0, 0)
    auto product = [&](u32x4 ar, u32x4 ai, u32x4 xr, u32x4 xi) {
        SV_MFMA(ar, xr, re);
        SV_MFMA(ar, xi, im);
        SV_MFMA(ai, xi ^ 0x80008000u, re);
        SV_MFMA(ai, xr, im);
    };
#undef SV_MFMA
    // the lane's inputs: half s of the columns, 8 (2 s + e / 4) + 4 (lane / 32) + e % 4
    f32x2 x[2][8];
    auto fetch = [&](int s) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            x[s][e] = *reinterpret_cast<const f32x2*>(lds + (at ^ b.off(16 * s + 8 * (e / 4) + (e % 4))));
    };
    if (coupled) {
        // all of them at once, so that the factors need no registers behind this
        f32x2 w[5], f[4];
        phases(w);
        fetch(0);
        fetch(1);
        f[0] = lane >= 32 ? w[2] : f32x2{1.f, 0.f};
        f[1] = cmul(f[0], w[0]), f[2] = cmul(f[0], w[1]), f[3] = cmul(f[1], w[1]);
        const f32x2 high[4] = {f32x2{1.f, 0.f}, w[3], w[4], cmul(w[3], w[4])};
#pragma unroll
        for (int r = 0; r < 16; ++r)
            x[r / 8][r % 8] = cmul(x[r / 8][r % 8], r < 4 ? f[r] : cmul(f[r % 4], high[r / 4]));
    }
    // the products of half s but the largest, whose parts of the inputs go to x0
    auto small_products = [&](int s, u32x4* x0) {
        if (!coupled) fetch(s);
        u32x4 xr[3], xi[3];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const f32x2 u = x[s][2 * p], v = x[s][2 * p + 1];
            uint32_t w0, w1, w2;
            split_bf16(u.x, v.x, w0, w1, w2, lost);
            xr[0][p] = w0, xr[1][p] = w1, xr[2][p] = w2;
            split_bf16(u.y, v.y, w0, w1, w2, lost);
            xi[0][p] = w0, xi[1][p] = w1, xi[2][p] = w2;
            asm volatile("" : "+v"(lost));  // summed here, not kept for later
        }
        constexpr int pa[5] = {2, 0, 1, 1, 0}, px[5] = {0, 2, 1, 0, 1};
#pragma unroll
        for (int i = 0; i < 5; ++i) product(o.re[pa[i]], o.im[pa[i]], xr[px[i]], xi[px[i]]);
        x0[0] = xr[0], x0[1] = xi[0];
        __builtin_amdgcn_sched_barrier(0);  // one half's operands at a time
    };
    u32x4 x0[2], x1[2];
    small_products(0, x0);
    const u32x4 re0 = o.re[0], im0 = o.im[0];
    o.load(m, 1, lane);
    small_products(1, x1);
    product(re0, im0, x0[0], x0[1]);
    product(o.re[0], o.im[0], x1[0], x1[1]);
    o.load(next, 0, lane);
    // (an amplitude that rounds to no bf16, or is no number: its column holds no number)
    const bool again = ((lost & 0xffffu) != 0) | (re[0] != re[0]);
    if (__builtin_expect((b.kind & kSweepFp32) || __ballot(again) != 0, 0)) {
        // the same sums of FP32 products, the matrix put together from its parts
        re = f32x16{0}, im = f32x16{0};
        f32x2 w[5];
        if (coupled) phases(w);
#pragma nounroll
        for (int r = 0; r < 16; ++r) {
            const int c = (r & 3) | (r & 12) << 1;  // the column of the lanes 0-31, that of the others is c + 4
            f32x2 x = *reinterpret_cast<const f32x2*>(lds + (at ^ b.off(c)));
            if (coupled) {
                if (c & 1) x = cmul(x, w[0]);
                if (c & 2) x = cmul(x, w[1]);
                if (lane >= 32) x = cmul(x, w[2]);
                if (c & 8) x = cmul(x, w[3]);
                if (c & 16) x = cmul(x, w[4]);
            }
            float entry[2];
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                if (b.kind & kSweepFp32) {
                    entry[part] = *lane_address<const float>(m + (part * 16 + r) * 16, uint32_t(lane) * 4);
                    continue;
                }
                entry[part] = 0.f;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const uint32_t v = *lane_address<const uint32_t>(m + ((part * 3 + q) * 2 + (r >> 3)) * 64,
                                                                     uint32_t(lane) * 16 + ((r & 6) << 1));
                    entry[part] += __builtin_bit_cast(float, r & 1 ? v & 0xffff0000u : v << 16);
                }
            }
            re = __builtin_amdgcn_mfma_f32_32x32x2f32(entry[0], x.x, re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f32_32x32x2f32(entry[0], x.y, im, 0, 0, 0);
            re = __builtin_amdgcn_mfma_f32_32x32x2f32(entry[1], -x.y, re, 0, 0, 0);
            im = __builtin_amdgcn_mfma_f32_32x32x2f32(entry[1], x.x, im, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
        *reinterpret_cast<f32x2*>(lds + (at ^ b.off(8 * (r / 4) + (r % 4)))) = f32x2{re[r], im[r]};
}

// complex64, four qubits, on v_mfma_f32_16x16x4_f32 (the chain of
// k_tile_c64_k4), four column tiles of 16 groups per wave of NT / 64, as far as
// the state of `amps` amplitudes has groups.
template <int NT>
__device__ __forceinline__ void block4(char* lds, const SweepBlock& b, const f32x4* __restrict__ m, const LaneBits& lb,
                                       uint32_t wave, int lane, uint64_t amps)
{
    const uint32_t tiles = amps >> 8 ? uint32_t(amps >> 8) : 1u;
    const int q = lane >> 4;
    const f32x4 ar = m[lane], ai = m[64 + lane], as = m[128 + lane];
    const uint32_t lin = ((q & 1) ? b.off(1) : 0u) ^ ((q & 2) ? b.off(2) : 0u);
    const uint32_t lout = ((q & 1) ? b.off(4) : 0u) ^ ((q & 2) ? b.off(8) : 0u);
    for (int i = 0; i < 4; ++i) {
        const uint32_t c = wave + uint32_t(i) * (NT / 64);
        if (c >= tiles) break;
        const uint32_t base = lane_part<4>(lb, b.grp) ^ wave_part<5>(c, b.grp + 4);
        f32x2 x[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) x[s] = *reinterpret_cast<const f32x2*>(lds + (base ^ lin ^ b.off(4 * s)));
        f32x4 p1 = {0}, p2 = {0}, p3 = {0};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            p1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[s], x[s].x, p1, 0, 0, 0);
            p2 = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[s], x[s].y, p2, 0, 0, 0);
            p3 = __builtin_amdgcn_mfma_f32_16x16x4f32(as[s], x[s].x + x[s].y, p3, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<f32x2*>(lds + (base ^ lout ^ b.off(r))) = f32x2{p1[r] - p2[r], p3[r] - p1[r] - p2[r]};
    }
}

// complex128, five qubits, on v_mfma_f64_16x16x4_f64: one column tile of 16
// groups per wave, two row tiles (the chain of k_tile_c128_k5).  The lane's
// inputs are matrix columns 4s + q, its outputs rows 16 rt + 4v + q.
template <bool SUM, bool READY>
__device__ __forceinline__ void block5(char* lds, const SweepBlock& b, const f64x2* __restrict__ m, Ops<double>& o,
                                       const LaneBits& lb, uint32_t wave, int lane)
{
    uint32_t at = lane_part<4>(lb, b.grp) ^ wave_part<3>(wave, b.grp + 4) ^ (lb.m[4] & b.off(1)) ^ (lb.m[5] & b.off(2));
    asm volatile("" : "+v"(at));
    f64x2 x[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) x[s] = *reinterpret_cast<const f64x2*>(lds + (at ^ b.off(4 * s)));
    Ops<double> second;
    if (READY) second.load_rows(m, lane, 1);
    auto rows = [&](int rt, const Ops<double>& w) {
        f64x4 p1 = {0}, p2 = {0}, p3 = {0};
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const double a0 = w.re[s >> 1][s & 1], a1 = w.im[s >> 1][s & 1];
            p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, x[s].x, p1, 0, 0, 0);
            p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, x[s].y, p2, 0, 0, 0);
            p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0 + a1, x[s].x + x[s].y, p3, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
            *reinterpret_cast<f64x2*>(lds + (at ^ b.off(16 * rt + 4 * v))) =
                f64x2{p1[v] - p2[v], p3[v] - p1[v] - p2[v]};
    };
    if (!READY) o.load_rows(m, lane, 0);
    rows(0, o);
    if (!READY) {
        __builtin_amdgcn_sched_barrier(0);
        second.load_rows(m, lane, 1);
    }
    rows(1, second);
}

// k <= 3 on the vector units, in the order of k_apply_dense.  A thread takes all
// its groups (16 amplitudes of complex64, 8 of complex128) at once, so that the
// matrix is read once, as far as the state of `amps` amplitudes has groups (16
// blocks of three qubits on 10 qubits complex64: 79 -> 61 us).
template <typename R, int K, int T, int NT>
__device__ __forceinline__ void block_small(char* lds, const SweepBlock& b, const typename Amp<R>::V* __restrict__ m,
                                            const LaneBits& lb, uint32_t wave, uint64_t amps)
{
    using V = typename Amp<R>::V;
    constexpr int D = 1 << K, kWaves = NT / 64, kAll = 1 << (T - K - 6), G = kAll > kWaves ? kAll / kWaves : 1;
    const uint32_t groups = amps >> (K + 6) ? uint32_t(amps >> (K + 6)) : 1u;  // in units of a wave's 64
    if (wave >= groups || wave >= kAll) return;
    asm volatile("" ::: "memory");  // the matrix stays out of the registers
    const uint32_t lane = lane_part<6>(lb, b.grp);
    uint32_t base[G];
    V v[G][D];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        base[g] = lane ^ wave_part<T - K - 6>(wave + uint32_t(g) * kWaves, b.grp + 6);
        if (g > 0 && wave + uint32_t(g) * kWaves >= groups) break;
#pragma unroll
        for (int c = 0; c < D; ++c) v[g][c] = *reinterpret_cast<const V*>(lds + (base[g] ^ b.off(c)));
    }
#pragma unroll
    for (int r = 0; r < D; ++r) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g > 0 && wave + uint32_t(g) * kWaves >= groups) break;
            R re = 0, im = 0;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const V e = m[r * D + c];
                re = fma(e.x, v[g][c].x, re);
                re = fma(-e.y, v[g][c].y, re);
                im = fma(e.x, v[g][c].y, im);
                im = fma(e.y, v[g][c].x, im);
            }
            *reinterpret_cast<V*>(lds + (base[g] ^ b.off(r))) = V{re, im};
        }
    }
}

// complex128, five qubits (states of fewer than 11 qubits) and four: on the vector
// units in the order of k_apply_dense, one group per lane.  A tile has fewer
// groups than the workgroup lanes, so each wave takes 8 of its groups' rows (16
// blocks of four qubits on 10 qubits, all rows by half of the waves: 148 us, now
// 102).  Every wave reads its groups' inputs before any writes.
template <int K, int T, int NT>
__device__ __forceinline__ void block_rows(char* lds, const SweepBlock& b, const f64x2* __restrict__ m,
                                           const LaneBits& lb, int wave)
{
    constexpr int D = 1 << K, kAll = 1 << (T - K - 6), kRows = D * kAll / (NT / 64);
    static_assert(kRows == 8, "rows of a thread");
    const int first = wave / kAll * kRows;
    const uint32_t base = lane_part<6>(lb, b.grp) ^ wave_part<T - K - 6>(uint32_t(wave % kAll), b.grp + 6);
    f64x2 v[D], y[kRows];
#pragma unroll
    for (int c = 0; c < D; ++c) v[c] = *reinterpret_cast<const f64x2*>(lds + (base ^ b.off(c)));
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const f64x2* row = m + (first + r) * D;
        double re = 0, im = 0;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            re = fma(row[c].x, v[c].x, re);
            re = fma(-row[c].y, v[c].y, re);
            im = fma(row[c].x, v[c].y, im);
            im = fma(row[c].y, v[c].x, im);
        }
        y[r] = f64x2{re, im};
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRows; ++r) *reinterpret_cast<f64x2*>(lds + (base ^ b.off(first + r))) = y[r];
}

// The first 16 words of a block's descriptor (all that a five-qubit block
// needs) in scalar registers, by one load: left to itself the compiler loads
// words one by one where they are used.
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ u32x16 load_words(const SweepBlock* p)
{
    typedef u32x16 Words __attribute__((aligned(alignof(SweepBlock))));
    return *reinterpret_cast<const Words*>(p);
}
__device__ __forceinline__ SweepBlock block_of(const u32x16& w)
{
    SweepBlock b{};
#pragma unroll
    for (int j = 0; j < 5; ++j) b.bit[j] = w[j];
    b.kind = int32_t(w[5]);
#pragma unroll
    for (int j = 0; j < 10; ++j) b.grp[j] = w[6 + j];
    return b;
}

// A block's descriptor from the wave's copy of it (lane l holds word l).
__device__ __forceinline__ SweepBlock unpack_block(uint32_t words)
{
    auto word = [&](int i) { return uint32_t(__builtin_amdgcn_readlane(int(words), i)); };
    SweepBlock b{};
#pragma unroll
    for (int j = 0; j < 5; ++j) b.bit[j] = word(j);
    b.kind = int32_t(word(5));
#pragma unroll
    for (int j = 0; j < 12; ++j) b.grp[j] = word(6 + j);
    return b;
}

// Z-type expectation sums of the state a sweep leaves behind, taken from its
// tiles in LDS (no extra read of the state): for a workgroup, out[t] =
// sum over its amplitudes i of |psi_i|^2 (-1)^popcount(i & zm[t]) for
// t < n_terms, and out[n_terms] = sum |psi_i|^2, all FP64 in a fixed order
// (per thread by a Walsh-Hadamard transform, per wave by a butterfly, waves
// and tiles in order).  acc: LDS of 4 x (kZSumsMax + 1) doubles, zeroed.
// n_terms < 0: no sums.
constexpr int kZSumsMax = 32;
struct ZSums {
    const uint64_t* zm;
    int n_terms;
    double* out;
    double* acc;
};

// Adds a complex64 tile's sums (256 threads, 8 pairs a thread).  i0: global
// index of the thread's first amplitude.  The thread's 16 amplitudes differ in
// the tile-local bits 0 and 9-11 (amplitude j = e + 2u is element e of vector u)
// and share all others, so a term's sum over them is s * c[k]: c the
// Walsh-Hadamard transform of their probabilities over j, c[k] = sum_j p_j
// (-1)^popcount(j & k), k the term mask's bits at those four index bits, s its
// parity over the bits the 16 share.  The norm is the term of mask 0.
__device__ __forceinline__ void add_z_sums(char* lds, const SweepArgs& a, const ZSums& zs, uint64_t i0, int tid)
{
    constexpr int NT = 256;
    const int lane = tid & 63, wave = tid >> 6;
    const uint32_t at = 8u * slot<float>(uint32_t(tid) * 2);
    double c[16];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(lds + (at ^ 8u * slot<float>(uint32_t(u * NT) * 2)));
        c[2 * u] = fma(double(v.x), double(v.x), __dmul_rn(double(v.y), double(v.y)));
        c[2 * u + 1] = fma(double(v.z), double(v.z), __dmul_rn(double(v.w), double(v.w)));
    }
#pragma unroll
    for (int h = 1; h < 16; h <<= 1) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if (j & h) continue;
            const double x = c[j], y = c[j | h];
            c[j] = __dadd_rn(x, y);
            c[j | h] = __dsub_rn(x, y);
        }
    }
    // the coefficients take the thread's own slots (its amplitudes are read;
    // no other thread reads these slots before the next barrier)
#pragma unroll
    for (int u = 0; u < 8; ++u)
        *reinterpret_cast<f64x2*>(lds + (at ^ 8u * slot<float>(uint32_t(u * NT) * 2))) = f64x2{c[2 * u], c[2 * u + 1]};
    int jpos[4];  // index bits of the tile-local bits 0 and 9-11
#pragma unroll
    for (int q = 0; q < 4; ++q) jpos[q] = __builtin_ctzll(a.bit_off[q == 0 ? 0 : 8 + q]) - 3;
    // terms (the norm last, as term n_terms) in passes of eight; a pass's wave
    // sums by a reduce-scatter butterfly: after the exchanges over lane bits
    // 5, 4, 3 a lane holds one term, term (lane >> 3) & 7 of the pass, summed
    // over 8 lanes, and three more exchanges sum the rest
    double* row = zs.acc + wave * (kZSumsMax + 1);
    const bool b5 = (lane & 32) != 0, b4 = (lane & 16) != 0, b3 = (lane & 8) != 0;
    for (int p0 = 0; p0 <= zs.n_terms; p0 += 8) {
        double v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int tt = p0 + t;
            const uint64_t m = tt < zs.n_terms ? zs.zm[tt] : 0;
            const int k = int((m >> jpos[0]) & 1) | int(((m >> jpos[1]) & 1) << 1) | int(((m >> jpos[2]) & 1) << 2) |
                          int(((m >> jpos[3]) & 1) << 3);
            const double x =
                *reinterpret_cast<const double*>(lds + (at ^ 8u * slot<float>(uint32_t((k >> 1) * NT) * 2)) + 8 * (k & 1));
            v[t] = tt > zs.n_terms ? 0.0 : ((__popcll(i0 & m) & 1) ? -x : x);
        }
        double w4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            w4[j] = __dadd_rn(b5 ? v[j + 4] : v[j], __shfl_xor(b5 ? v[j] : v[j + 4], 32, 64));
        double w2[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
            w2[j] = __dadd_rn(b4 ? w4[j + 2] : w4[j], __shfl_xor(b4 ? w4[j] : w4[j + 2], 16, 64));
        double w = __dadd_rn(b3 ? w2[1] : w2[0], __shfl_xor(b3 ? w2[0] : w2[1], 8, 64));
        w = __dadd_rn(w, __shfl_xor(w, 4, 64));
        w = __dadd_rn(w, __shfl_xor(w, 2, 64));
        w = __dadd_rn(w, __shfl_xor(w, 1, 64));
        const int tt = p0 + ((lane >> 3) & 7);
        if ((lane & 7) == 0 && tt <= zs.n_terms) {
            const int r = tt == zs.n_terms ? kZSumsMax : tt;
            row[r] = __dadd_rn(row[r], w);
        }
    }
}

// The sweep of workgroup wg, NT threads on tiles of 2^T amplitudes.  SMALL
// (states of fewer than kPadQubits qubits): one tile a workgroup, blocks of
// fewer than five qubits on the vector units; a state of less than a tile
// leaves the rest of it zeros that no one stores.  FIRST: the state is |0..0>
// and is not read.  zs: complex64 sweeps of 256 threads only.
template <typename R, int T, int NT, bool SMALL, bool SPLIT = false, bool COUPLED = false, bool FIRST = false,
          bool SUMS = false>
__device__ __forceinline__ void sweep_tiles(char* __restrict__ psi, const SweepBlock* __restrict__ blocks,
                                            const char* __restrict__ mats, const SweepArgs& a, uint64_t wg,
                                            char* lds, const ZSums& zs, [[maybe_unused]] uint64_t* turns)
{
    using A = Amp<R>;
    using W = typename A::W;
    constexpr int NV = (1 << T) / A::kPerVec / NT;       // 16-byte vectors per thread
    constexpr int kCols = sizeof(R) == 4 ? 32 : 16;      // groups per wave
    constexpr uint32_t kStride = sweep_matrix_stride(sizeof(R) == 4) + (COUPLED ? sizeof(SweepCouple) : 0);
    auto phases = [&](int i) { return reinterpret_cast<const SweepCouple*>(mats + uint64_t(i + 1) * kStride) - 1; };
    static_assert((1 << (T - 5)) == kCols * (NT / 64), "one column tile per wave");
    static_assert(NV == 8, "three tile-local bits of a vector's index");
    const uint64_t t0 = wg * a.tiles_per_wg;
    if (t0 >= a.n_tiles) return;
    const uint64_t t1 = (a.n_tiles - t0 < a.tiles_per_wg) ? a.n_tiles : t0 + a.tiles_per_wg;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (SUMS && zs.n_terms >= 0 && lane <= kZSumsMax) zs.acc[wave * (kZSumsMax + 1) + lane] = 0.0;
    // the thread's vector u is tile-local amplitude (u NT + tid) amplitudes
    // per vector: the lane's bits give a 32-bit offset (they sit at the lowest
    // of the tile's high bits), the wave's and u's a uniform one
    constexpr int kLane0 = A::kPerVec - 1, kWave0 = kLane0 + 6, kU0 = kWave0 + __builtin_ctz(NT / 64);
    uint32_t loff = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b) loff += ((lane >> b) & 1) ? uint32_t(a.bit_off[kLane0 + b]) : 0u;
    uint64_t woff = 0;
#pragma unroll
    for (int b = 0; b < kU0 - kWave0; ++b) woff += ((wave >> b) & 1) ? a.bit_off[kWave0 + b] : 0u;
    uint64_t roff[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        roff[u] = woff;
#pragma unroll
        for (int b = 0; b < 3; ++b)
            if ((u >> b) & 1) roff[u] += a.bit_off[kU0 + b];
    }
    const uint32_t staged = A::kBytes * slot<R>(uint32_t(tid) * A::kPerVec);
    const LaneBits lb(lane);
    // few workgroups: the descriptors and matrices of all blocks are brought
    // to the L2 at once (one word of each 128-byte line), not block by block
    // (14 qubits complex64 as a graph: 104 -> 92 us, with the offsets of a
    // tile's bits from the host)
    constexpr int kWarm = 4;
    uint32_t warm[kWarm] = {};
    if (!SMALL && a.warm_lines > 0) {
#pragma unroll
        for (int w = 0; w < kWarm; ++w) {
            const int l = w * NT + tid;
            if (l < a.warm_lines) warm[w] = reinterpret_cast<const uint32_t*>(blocks)[l * 32];
        }
    }
    auto matrix = [&](int i) { return reinterpret_cast<const W*>(mats + uint64_t(i) * kStride); };
    for (uint64_t t = t0; t < t1; ++t) {  // (SMALL: once)
        char* base = psi + A::kBytes * tile_origin(t, a);
        if (FIRST && base != psi) {
            // |0..0> is zero on every tile but the first, and so is its image:
            // such a tile is only written
#pragma unroll
            for (int u = 0; u < NV; ++u) __builtin_nontemporal_store(W{}, lane_address<W>(base + roff[u], loff));
            continue;
        }
        W buf[NV];
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            if (FIRST || (SMALL && uint64_t(u * NT + tid) * A::kPerVec >= a.amps))
                buf[u] = W{};
            else
                buf[u] = __builtin_nontemporal_load(lane_address<const W>(base + roff[u], loff));
        }
        if (FIRST && tid == 0) buf[0][0] = 1;
        if constexpr (COUPLED) {
            // the phases of every block, wave and target but the lanes' parts,
            // while the tile is on its way
            const uint64_t origin = uint64_t(base - psi) / A::kBytes;
            for (int j = tid; j < 5 * (NT / 64) * a.n_blocks; j += NT) {
                const SweepCouple* c = phases(j / (5 * (NT / 64)));
                const uint64_t* p = c->out[j % 5];
                uint64_t u = c->wave[j % 5][j / 5 % (NT / 64)];
#pragma nounroll
                for (int q0 = 0; q0 < 36; q0 += 12) {
                    uint64_t v[12];
#pragma unroll
                    for (int q = 0; q < 12; ++q) v[q] = p[q0 + q];
#pragma unroll
                    for (int q = 0; q < 12; ++q) u += ((origin >> (q0 + q)) & 1) ? v[q] : 0;
                }
                turns[j] = u;
            }
        }
#pragma unroll
        for (int u = 0; u < NV; ++u)
            *reinterpret_cast<W*>(lds + (staged ^ A::kBytes * slot<R>(uint32_t(u * NT) * A::kPerVec))) = buf[u];
        __syncthreads();
        if constexpr (!SMALL) {
            // the next block's descriptor is on its way during a block
            u32x16 w = load_words(blocks);
            [[maybe_unused]] SplitOps split;
            if constexpr (SPLIT) split.load(reinterpret_cast<const u32x4*>(mats), 0, lane);
            for (int i = 0; i < a.n_blocks; ++i) {
                const int next = i + 1 < a.n_blocks ? i + 1 : i;
                asm volatile("" : "+s"(w));
                const SweepBlock b = block_of(w);
                w = load_words(blocks + next);
                if constexpr (SPLIT) {
                    block5_split<COUPLED>(lds, b, reinterpret_cast<const u32x4*>(matrix(i)),
                                          reinterpret_cast<const u32x4*>(matrix(next)), split, lb, uint32_t(wave), lane,
                                          phases(i), turns + 5 * (i * (NT / 64) + wave));
                } else {
                    Ops<R> o;
                    block5<false, false>(lds, b, matrix(i), o, lb, uint32_t(wave), lane);
                }
                __syncthreads();
            }
        } else {
            // a workgroup whose one or two waves a SIMD cannot hide the way of
            // a matrix from memory: block i + 1's matrix and block i + 2's
            // descriptor are loaded during block i (12 qubits complex128, 22
            // blocks: 118 -> 93 us)
            auto words = [&](int i) {
                return reinterpret_cast<const uint32_t*>(blocks + (i < a.n_blocks ? i : a.n_blocks - 1))[lane < kSweepBlockWords ? lane : 0];
            };
            Ops<R> o[2];
            uint32_t d[2] = {words(0), words(1)};
            o[0].template load<true>(matrix(0), lane);
            auto one = [&](int i, Ops<R>& now, Ops<R>& next, uint32_t& dw) {
                const SweepBlock b = unpack_block(dw);
                dw = words(i + 2);
                if (i + 1 < a.n_blocks) next.template load<true>(matrix(i + 1), lane);
                if (b.kind == kSweepMfma5) {
                    block5<true, true>(lds, b, matrix(i), now, lb, uint32_t(wave), lane);
                    return;
                }
                const auto* mv = reinterpret_cast<const typename A::V*>(matrix(i));
                if constexpr (sizeof(R) == 8 && NT == 256)
                    if (b.kind == kSweepRows5) block_rows<5, T, NT>(lds, b, mv, lb, wave);
                if (b.kind == 1) block_small<R, 1, T, NT>(lds, b, mv, lb, uint32_t(wave), a.amps);
                if (b.kind == 2) block_small<R, 2, T, NT>(lds, b, mv, lb, uint32_t(wave), a.amps);
                if (b.kind == 3) block_small<R, 3, T, NT>(lds, b, mv, lb, uint32_t(wave), a.amps);
                if (b.kind == 4) {
                    if constexpr (sizeof(R) == 8)
                        block_rows<4, T, NT>(lds, b, mv, lb, wave);
                    else
                        block4<NT>(lds, b, matrix(i), lb, uint32_t(wave), lane, a.amps);
                }
            };
            for (int i = 0; i < a.n_blocks; i += 2) {
                one(i, o[0], o[1], d[0]);
                __syncthreads();
                if (i + 1 == a.n_blocks) break;
                one(i + 1, o[1], o[0], d[1]);
                __syncthreads();
            }
        }
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            if (SMALL && uint64_t(u * NT + tid) * A::kPerVec >= a.amps) continue;
            __builtin_nontemporal_store(
                *reinterpret_cast<const W*>(lds + (staged ^ A::kBytes * slot<R>(uint32_t(u * NT) * A::kPerVec))),
                lane_address<W>(base + roff[u], loff));
        }
        if constexpr (SUMS)
            if (zs.n_terms >= 0) add_z_sums(lds, a, zs, uint64_t(base - psi + int64_t(roff[0]) + loff) / A::kBytes, tid);
        __syncthreads();
    }
    // a workgroup of written tiles only (FIRST) has met no barrier since the
    // waves zeroed their rows
    if constexpr (SUMS && FIRST) __syncthreads();
    if (SUMS && zs.n_terms >= 0 && tid <= zs.n_terms) {
        // the waves' rows in order; the norm last
        const int c = tid == zs.n_terms ? kZSumsMax : tid;
        double v = 0.0;
        for (int w = 0; w < NT / 64; ++w) v = __dadd_rn(v, zs.acc[w * (kZSumsMax + 1) + c]);
        zs.out[tid] = v;
    }
#pragma unroll
    for (int w = 0; w < kWarm; ++w) asm volatile("" ::"v"(warm[w]));
}

template <typename R, int T, int NT, bool SMALL, bool SPLIT = false, bool COUPLED = false>
__global__ __launch_bounds__(NT, SMALL ? 1 : 4) void k_sweep(char* __restrict__ psi, const SweepBlock* __restrict__ blocks,
                                                            const char* __restrict__ mats, SweepArgs a)
{
    __shared__ __align__(16) char lds[Amp<R>::kBytes << T];
    // (7.5 KiB: still four workgroups on the CU's 160 KiB, two of the larger tile)
    __shared__ uint64_t turns[COUPLED ? 5 * (NT / 64) * kMaxSweepBlocks : 1];
    sweep_tiles<R, T, NT, SMALL, SPLIT, COUPLED>(psi, blocks, mats, a, blockIdx.x, lds,
                                                 ZSums{nullptr, -1, nullptr, nullptr}, turns);
}

// Level path of a batch: workgroup w sweeps its tiles of one step of one
// circuit; on a circuit's last step it also leaves the Z-type sums of its
// tiles.  FIRST: the states are |0..0>.  Bound by HBM and the matrix pipe
// about equally: a step holds two blocks in the mean (in program order, since
// a swap would change the states' bits), so that a batch of 512 circuits of 8-20
// qubits moves half the bytes of one sweep per block: 13.5 -> 10.0 ms.
template <bool FIRST>
__global__ __launch_bounds__(256, 4) void k_batch_level(char* __restrict__ states, const BatchSweep* __restrict__ sweeps,
                                                       const BatchLevelEntry* __restrict__ entries,
                                                       const SweepBlock* __restrict__ blocks,
                                                       const char* __restrict__ mats,
                                                       const uint64_t* __restrict__ z_masks,
                                                       double* __restrict__ partials)
{
    __shared__ __align__(16) char lds[8 << 12];
    __shared__ double zacc[4 * (kZSumsMax + 1)];
    const BatchLevelEntry e = entries[blockIdx.x];
    const BatchSweep& d = sweeps[e.sweep];
    const ZSums zs{z_masks + d.term0, d.n_terms, partials + d.red_off + uint64_t(e.wg) * uint64_t(d.n_terms + 1), zacc};
    sweep_tiles<float, 12, 256, false, false, false, FIRST, true>(states + 8 * d.state_off, blocks + d.block0,
                                                    mats + uint64_t(d.block0) * sweep_matrix_stride(true), d.a, e.wg,
                                                    lds, zs, nullptr);
}

constexpr int tile_bits(sv_dtype_t dt) { return dt == SV_C64 ? 12 : 11; }  // 32 KiB

// States of fewer qubits sweep blocks of 1-4 qubits as they are (k_sweep's
// SMALL form), larger ones as five-qubit blocks, as their own sweeps do
// (pad_to_five).  A state of up to tile_bits qubits is one tile and its
// program one launch, and so does one qubit more, with twice the threads on
// a tile twice as large.
constexpr int kPadQubits = 14;

// Smallest state whose blocks may pass blocks on other qubits on their way
// into a sweep (below, a program's blocks keep their order and its amplitudes
// their bits), and whose complex64 sweeps multiply bf16 parts (block5_split): a
// state of 22 qubits is the first that keeps every CU's matrix cores busy.
constexpr int kReorderQubits = 22;

// Largest state whose five-qubit blocks are swept by k_sweep also one at a time
// (512 MiB).  Mean over neighbouring and random targets, the tuned tile kernels
// of one block and this one: complex64 22, 24, 25, 26 qubits 21.7, 63.5, 115 and 201
// us against 20.6, 57.6, 103 and 193; complex128 24 and 25 qubits 138 and 216
// against 117 and 213; on 28 qubits complex64, where HBM alone counts, 686 and 730.
constexpr int lone_qubits(sv_dtype_t dt) { return dt == SV_C64 ? 26 : 25; }
constexpr int kReorderWindow = 96;

// Shortest runs of a tile: 128 bytes, the line of the L2.  (Runs of 64 bytes
// below 22 qubits, for 7% fewer sweeps, measured no faster: 339 us against 324
// on 19 qubits complex128.)
constexpr int min_run_bits(sv_dtype_t dt) { return dt == SV_C64 ? 4 : 3; }

// Largest state of multi-block sweeps: the lanes' part of an address (three
// index bits below the fifth highest one) fits 32 bits.
constexpr int kMaxSweepQubitsC64 = 34, kMaxSweepQubitsC128 = 33;

// States of one tile and little more: a block's own kernel in launches of the
// fastest ones (14 us for the first of a call, 2 for each more; the first block of a
// sweep takes 17-22 us, a second 24).  Calls of up to kFewLaunches take every
// block on its own: 1, 2, 4 and 6 blocks of two qubits on 10 qubits complex64 14, 17, 22 and 27 us
// against 17, 24, 27 and 31 as a sweep; from seven launches on a call waits
// for the device, 65 us against 34.  (A recorded graph has no such cost.)
constexpr int kFewLaunches = 6;
int lone_launches(sv_dtype_t dt, int n, const FusedBlock& b)
{
    if (b.k <= 3 || b.diagonal) return 1;
    if (dt == SV_C64) return b.k == 4 ? (n < 12 ? 1 : 2) : (n < 12 ? 2 : 4);
    return b.k == 4 ? 4 : kFewLaunches + 1;
}

uint64_t qubit_mask(const FusedBlock& b)
{
    uint64_t m = 0;
    for (int a = 0; a < b.k; ++a) m |= uint64_t(1) << b.targets[a];
    return m;
}

// Whether FP32 products leave less error than block5_split's on some amplitudes: a
// real matrix (or i times one) of at most two entries a row, not all of a bf16's
// 8 bits.  One rotation among CNOTs on real amplitudes: FP32 3.2e-8 to 4.0e-8 of the
// state's 2-norm, the parts up to 10% more, since FP32 rounds no more often there
// and leaves nothing out (on complex amplitudes 5.5e-8 and 3.2e-8 to 4.1e-8).  With
// two rotations the parts leave 0.84-0.89 of FP32's error, with five 0.41.
bool few_products(const FusedBlock& b)
{
    const int d = 1 << b.k;
    bool re = false, im = false, wide = false;
    for (int i = 0; i < d; ++i) {
        int row = 0;
        for (int c = 0; c < d; ++c) {
            const float v[2] = {float(b.m[2 * (size_t(i) * d + c)]), float(b.m[2 * (size_t(i) * d + c) + 1])};
            re |= v[0] != 0.f;
            im |= v[1] != 0.f;
            row += v[0] != 0.f || v[1] != 0.f;
            if (row > 2 || (re && im)) return false;
            for (float f : v) {
                uint32_t w;
                std::memcpy(&w, &f, 4);
                wide |= (w & 0xffffu) != 0;
            }
        }
    }
    return wide;
}

// The qubits that decide which blocks commute with b: its targets and the
// qubits its phases depend on.
uint64_t touched_mask(const FusedBlock& b)
{
    uint64_t m = qubit_mask(b);
    for (int c = 0; c < b.n_couple; ++c) m |= uint64_t(1) << b.couple_q[c];
    return m;
}

// Fills st's tile for the qubit set `on`: the runs as long as the set allows
// (bits L.. join the low bits while the tile has room).
void fill_geometry(sv_dtype_t dt, int n, int cu_count, uint64_t on, int spread_lo, SweepStep& st)
{
    const int T = st.tile_bits;
    SweepArgs& a = st.args;
    a = SweepArgs{};
    a.n_blocks = int(st.blocks.size());
    a.amps = uint64_t(1) << n;
    const uint64_t bytes = dt == SV_C64 ? 8 : 16;
    for (int p = 0; p < T; ++p) a.bit_off[p] = bytes << p;
    // states of up to a few tiles a CU: every workgroup meets its blocks'
    // matrices for the first time
    if (n > T && uint64_t(1) << (n - T) <= uint64_t(4 * cu_count)) a.warm_lines = int32_t(sweep_bytes(dt, st) / 128);
    if (n <= T) {
        a.n_tiles = a.tiles_per_wg = 1;
        a.L = T;
        return;
    }
    int L = min_run_bits(dt);
    if (spread_lo > 0) {
        // runs of 1 KiB at most, then free bits from spread_lo up
        const int run = dt == SV_C64 ? 7 : 6;
        while (L < run && __builtin_popcountll(on >> L) + L < T) ++L;
        for (int q = std::max(L, spread_lo); q < n && __builtin_popcountll(on >> L) + L < T; ++q) on |= uint64_t(1) << q;
    }
    while (L < T && __builtin_popcountll(on >> L) + L < T) ++L;
    a.L = L;
    for (int q = L; q < n; ++q)
        if ((on >> q) & 1) {
            a.bit_off[L + a.n_hi] = bytes << q;
            a.hi_mask[a.n_hi] = ~((uint64_t(1) << q) - 1);
            st.hi_pos[a.n_hi++] = q;
        }
    a.lg_tiles = n - T;
    a.n_tiles = uint64_t(1) << a.lg_tiles;
    // one tile a workgroup: four fit a CU and hide each other's loads and stores
    a.tiles_per_wg = 1;
}

}  // namespace

std::vector<SweepStep> plan_sweeps(sv_dtype_t dt, int n, int cu_count, const FusedBlock* blocks, int first, int end,
                                   const SweepRules& rules)
{
    std::vector<SweepStep> steps;
    // one qubit more is one tile where most blocks have five qubits: smaller ones are
    // bound by the vector units of the tile's one CU (32 of three qubits, 12 qubits
    // complex128, as a recorded graph: 148 us as one tile, 107 as two, 111 a launch each)
    int fives = 0, launches = 0;
    for (int i = first; i < end; ++i) {
        fives += blocks[i].k == 5;
        launches += lone_launches(dt, n, blocks[i]);
    }
    const bool one_tile = n <= tile_bits(dt) + (!rules.pad_all && 2 * fives >= end - first);
    const bool small = n < kPadQubits && !rules.pad_all;
    const bool few = small && rules.few_alone && launches <= kFewLaunches;
    // From 22 qubits on a sweep may take a tile of one bit more, if its blocks
    // need it: 24 sweeps become 20 for a 28-qubit CNOT/CP circuit (complex128,
    // 51.3 -> 48.2 ms), 37 become 30 for a 23-qubit coupled program (1.71 -> 1.58
    // ms); 25-qubit circuits complex64 3.47 -> 3.11 and 5.69 -> 5.42 ms.  Not with
    // coupled blocks on the largest states, where lone ones have kernels bound
    // by HBM alone: the 28-qubit QFT took 7.69 ms without and 7.88 with.
    const int T = std::max(tile_bits(dt) + (n >= kReorderQubits && !rules.keep_order), one_tile ? n : 0);
    const bool coupled_large = n <= lone_qubits(dt);
    const int lo = min_run_bits(dt);
    const bool split = dt == SV_C64 && n >= kReorderQubits && !rules.keep_order;
    auto eligible = [&](const FusedBlock& b) {
        if (b.diagonal || b.k > 5) return false;
        // coupled blocks: where the phases have a kernel (block5_split), and no
        // padding qubit could be a coupled one
        if (b.n_couple > 0 && !(split && b.k == 5)) return false;
        if (n > (dt == SV_C64 ? kMaxSweepQubitsC64 : kMaxSweepQubitsC128)) return false;
        if (rules.pad_all) return true;
        // larger states: blocks on 2-4 qubits are swept as five-qubit ones
        // where their own sweep is (with enough qubits below or above
        // theirs), single-qubit ones on their own
        if (n < kPadQubits || b.k == 5) return true;
        const uint64_t on = qubit_mask(b);
        const int outside = __builtin_ctzll(on) + n - 1 - (63 - __builtin_clzll(on));
        return b.k >= 2 && outside >= 5 - b.k;
    };
    auto fits = [&](uint64_t on, bool coupled = false) {
        return one_tile || __builtin_popcountll(on >> lo) <= (coupled && !coupled_large ? tile_bits(dt) : T) - lo;
    };
    auto add = [&](std::vector<int>&& take, uint64_t on) {
        if (few)
            for (; take.size() > 1; take.erase(take.begin())) {
                steps.emplace_back();
                steps.back().blocks = {take[0]};
            }
        SweepStep st;
        const FusedBlock& b0 = blocks[take[0]];
        const bool own = few || (small && lone_launches(dt, n, b0) < kFewLaunches);
        const bool lone = !own && (n < kReorderQubits || rules.pad_all || (n <= lone_qubits(dt) && b0.k == 5));
        st.multi = take.size() > 1 || (lone && eligible(b0));
        st.blocks = std::move(take);
        st.padded = rules.pad_all || n >= kPadQubits;
        for (int i : st.blocks) st.coupled = st.coupled || (st.multi && blocks[i].n_couple > 0);
        st.split = split;
        if (st.multi) {
            st.tile_bits = T;
            if (T > tile_bits(dt) && !one_tile && __builtin_popcountll(on >> lo) <= tile_bits(dt) - lo) --st.tile_bits;
            fill_geometry(dt, n, cu_count, on, rules.spread_lo, st);
        }
        steps.push_back(std::move(st));
    };
    std::vector<int> rest;
    for (int i = first; i < end; ++i) rest.push_back(i);
    size_t at = 0;
    while (at < rest.size()) {
        const int b0 = rest[at];
        if (!eligible(blocks[b0])) {
            add({b0}, 0);
            ++at;
            continue;
        }
        if (n < kReorderQubits || rules.keep_order) {
            std::vector<int> take;
            uint64_t on = 0;
            while (at < rest.size() && take.size() < kMaxSweepBlocks && eligible(blocks[rest[at]]) && fits(on | qubit_mask(blocks[rest[at]]))) {
                on |= qubit_mask(blocks[rest[at]]);
                take.push_back(rest[at++]);
            }
            add(std::move(take), on);
            continue;
        }
        // a block may join a sweep ahead of blocks left behind whose targets
        // it does not touch and that do not touch its targets (they commute); of the first ready seeds, the one
        // whose sweep takes most blocks
        const size_t hi = std::min(rest.size(), at + kReorderWindow);
        std::vector<int> best;
        uint64_t best_on = 0;
        int seeds = 0;
        uint64_t before = 0, before_t = 0;  // qubits and targets of the blocks passed over
        for (size_t s = at; s < hi && seeds < 8; ++s) {
            const uint64_t qs = qubit_mask(blocks[rest[s]]);
            const uint64_t ts = touched_mask(blocks[rest[s]]);
            const bool ready = !(qs & before) && !(ts & before_t) && eligible(blocks[rest[s]]);
            before |= ts;
            before_t |= qs;
            if (!ready) continue;
            ++seeds;
            std::vector<int> take{rest[s]};
            uint64_t on = qs;
            bool coupled = blocks[rest[s]].n_couple > 0;
            std::vector<char> in(hi - at, 0);
            in[s - at] = 1;
            while (take.size() < kMaxSweepBlocks) {
                int pick = -1, cost = 65;
                uint64_t blocked = 0, blocked_t = 0;
                for (size_t j = at; j < hi; ++j) {
                    if (in[j - at]) continue;
                    const uint64_t q = qubit_mask(blocks[rest[j]]);
                    const uint64_t touched = touched_mask(blocks[rest[j]]);
                    if (!(q & blocked) && !(touched & blocked_t) && eligible(blocks[rest[j]]) &&
                        fits(on | q, coupled || blocks[rest[j]].n_couple > 0)) {
                        const int c = __builtin_popcountll((on | q) >> lo);
                        if (c < cost) {
                            cost = c;
                            pick = int(j);
                        }
                    }
                    blocked |= touched;
                    blocked_t |= q;
                }
                if (pick < 0) break;
                in[pick - at] = 1;
                on |= qubit_mask(blocks[rest[pick]]);
                coupled = coupled || blocks[rest[pick]].n_couple > 0;
                take.push_back(rest[pick]);
            }
            if (take.size() > best.size()) {
                best = take;
                best_on = on;
            }
        }
        // program order inside the sweep
        std::sort(best.begin(), best.end());
        size_t w = hi;
        for (size_t j = hi; j-- > at;)
            if (!std::binary_search(best.begin(), best.end(), rest[j])) rest[--w] = rest[j];
        at = w;
        add(std::move(best), best_on);
    }
    return steps;
}

namespace {

uint32_t slot_bytes(sv_dtype_t dt, uint32_t a) { return dt == SV_C64 ? 8u * slot<float>(a) : 16u * slot<double>(a); }

// Byte offsets (grp) and positions (pos) of the group index's bits: the tile
// bits outside `used`, those of the state's n qubits first, the lanes' first of these;
// returns their number.  The first 4 (complex64; complex128 3) lane bits are to be
// independent in the 32 banks a write sees, and one more with them in the 64
// of a read, as far as there are such bits.
int choose_lanes(sv_dtype_t dt, int T, int n_qubits, uint32_t used, uint32_t* grp, int* pos)
{
    const int width = dt == SV_C64 ? 5 : 4;
    uint32_t left = ((1u << T) - 1u) & ~used;
    // the vectors taken, reduced: basis[i] has its top bit at i
    uint32_t low[5] = {}, full[5] = {};
    auto add = [](uint32_t* basis, uint32_t v) {
        while (v) {
            const int i = 31 - __builtin_clz(v);
            if (!basis[i]) {
                basis[i] = v;
                return true;
            }
            v ^= basis[i];
        }
        return false;
    };
    int n = 0;
    auto take = [&](int p) {
        left &= ~(1u << p);
        pos[n] = p;
        grp[n++] = slot_bytes(dt, 1u << p);
    };
    auto bank = [&](int p) { return (dt == SV_C64 ? slot<float>(1u << p) : slot<double>(1u << p)) & ((1u << width) - 1u); };
    const int own = std::min(T, n_qubits);
    for (int p = 0; p < own && n < width - 1; ++p)
        if (((left >> p) & 1) && add(low, bank(p) & ((1u << (width - 1)) - 1u))) {
            add(full, bank(p));
            take(p);
        }
    for (int p = 0; p < own && n < width; ++p)
        if (((left >> p) & 1) && add(full, bank(p))) take(p);
    for (int p = 0; p < T; ++p)
        if ((left >> p) & 1) take(p);
    return n;
}

// Place of matrix entry (i, c) in a part of the packed operands.  complex64:
// float4 [q][lane] of A[i][2(4q + j) + half], lane = i + 32 half; complex128:
// double2 [rt 4 + s/2][lane] of A[16 rt + i][4s + q], lane = i + 16 q.
struct PackOrder {
    uint16_t f32[1024], f64[1024];
    PackOrder()
    {
        for (int i = 0; i < 32; ++i)
            for (int c = 0; c < 32; ++c) {
                f32[i * 32 + c] = uint16_t(((c >> 3) * 64 + i + 32 * (c & 1)) * 4 + ((c >> 1) & 3));
                f64[i * 32 + c] =
                    uint16_t((((i >> 4) * 4 + (c >> 3)) * 64 + (i & 15) + 16 * (c & 3)) * 2 + ((c >> 2) & 1));
            }
    }
};
const PackOrder kPackOrder;

// Packed A operands of the five-qubit sweep of M (x) I (M on the block's k
// qubits, the padding qubits the high matrix bits): parts Re M, Im M and, for
// complex64, Re M + Im M (of the entries as given for states of fewer than
// 12 qubits, else of the rounded ones, as their single-block kernels take it).
template <typename R>
void pack5(const FusedBlock& b, int n, R* o)
{
    const uint16_t* at = sizeof(R) == 4 ? kPackOrder.f32 : kPackOrder.f64;
    const int parts = sizeof(R) == 4 ? 3 : 2, d = 1 << b.k;
    if (b.k < 5) std::fill(o, o + parts * 1024, R(0));
    for (int e = 0; e < 32; e += d)  // the diagonal blocks of M (x) I
        for (int i = 0; i < d; ++i) {
            const double* row = b.m + 2 * size_t(i) * d;
            const uint16_t* to = at + (e + i) * 32 + e;
            for (int c = 0; c < d; ++c) {
                const R re = R(row[2 * c]), im = R(row[2 * c + 1]);
                o[to[c]] = re;
                o[1024 + to[c]] = im;
                if (sizeof(R) == 4) o[2048 + to[c]] = n < 12 ? R(row[2 * c] + row[2 * c + 1]) : re + im;
            }
        }
}

// The operands of block5_split: part (Re M, Im M), piece, half of the columns
// s, lane: row lane % 32, columns 8 (2 s + e / 4) + 4 (lane / 32) + e % 4 for e < 8.
// Returns whether the pieces hold the entries (those of 2^-110 and more, as far as
// the first is not rounded up to infinity).
bool pack5_split(const FusedBlock& b, uint16_t* o)
{
    const int d = 1 << b.k;
    bool hold = true;
    std::fill(o, o + 6 * 1024, uint16_t(0));
    for (int e = 0; e < 32; e += d)  // the diagonal blocks of M (x) I
        for (int i = 0; i < d; ++i)
            for (int c = 0; c < d; ++c)
                for (int part = 0; part < 2; ++part) {
                    const int row = e + i, j = e + c;
                    const int at = ((j >> 4) * 64 + row + 32 * ((j >> 2) & 1)) * 8 + ((j >> 3) & 1) * 4 + (j & 3);
                    float v = float(b.m[2 * (size_t(i) * d + c) + part]);
                    for (int q = 0; q < 3; ++q) {
                        uint32_t w;
                        std::memcpy(&w, &v, 4);
                        w = (w + 0x7fffu + ((w >> 16) & 1u)) & 0xffff0000u;
                        o[(part * 3 + q) * 1024 + at] = uint16_t(w >> 16);
                        float f;
                        std::memcpy(&f, &w, 4);
                        v -= f;
                    }
                    hold &= v == 0.f;
                }
    return hold;
}

// The same matrix for FP32 products (kSweepFp32): part, step r, lane: row lane % 32,
// column 8 (r / 4) + 4 (lane / 32) + r % 4.
void pack5_fp32(const FusedBlock& b, float* o)
{
    const int d = 1 << b.k;
    for (int part = 0; part < 2; ++part)
        for (int r = 0; r < 16; ++r)
            for (int lane = 0; lane < 64; ++lane) {
                const int row = lane % 32, c = 8 * (r / 4) + 4 * (lane / 32) + r % 4;
                o[(part * 16 + r) * 64 + lane] =
                    row / d == c / d ? float(b.m[2 * (size_t(row % d) * d + c % d) + part]) : 0.f;
            }
}

}  // namespace

// Bytes from one block's matrix to the next's in a step's buffer.
size_t matrix_stride(sv_dtype_t dt, const SweepStep& st)
{
    return sweep_matrix_stride(dt == SV_C64) + (st.coupled ? sizeof(SweepCouple) : 0);
}

size_t sweep_bytes(sv_dtype_t dt, const SweepStep& st)
{
    return ((sizeof(SweepBlock) * st.blocks.size() + 255) & ~size_t(255)) +
           matrix_stride(dt, st) * st.blocks.size();
}

void pack_sweep(sv_dtype_t dt, const SweepStep& st, const FusedBlock* blocks, void* dst)
{
    pack_sweep(dt, st, blocks, static_cast<SweepBlock*>(dst),
               static_cast<char*>(dst) + ((sizeof(SweepBlock) * st.blocks.size() + 255) & ~size_t(255)));
}

void pack_sweep(sv_dtype_t dt, const SweepStep& st, const FusedBlock* blocks, SweepBlock* desc, char* mat)
{
    const int L = st.args.L, T = st.tile_bits, n = 63 - __builtin_clzll(st.args.amps);
    for (size_t j = 0; j < st.blocks.size(); ++j, mat += matrix_stride(dt, st)) {
        const FusedBlock& b = blocks[st.blocks[j]];
        const int k = st.padded ? 5 : b.k;
        SweepBlock s{};
        s.kind = k < 5 ? k : (dt == SV_C128 && n < 11) ? kSweepRows5 : kSweepMfma5;
        // tile-local positions of the targets, then of the padding qubits
        // (the lowest positions that are free)
        int pos[5] = {}, group[12] = {};
        uint32_t used = 0;
        for (int a = 0; a < b.k; ++a) {
            int p = b.targets[a];
            if (p >= L) {
                int r = 0;
                while (st.hi_pos[r] != p) ++r;
                p = L + r;
            }
            pos[a] = p;
            used |= 1u << p;
        }
        for (int a = b.k, p = 0; a < k; ++p)
            if (!((used >> p) & 1)) {
                pos[a++] = p;
                used |= 1u << p;
            }
        const int left = choose_lanes(dt, T, n, used, s.grp, group);
        if (b.n_couple > 0) s.kind |= kSweepCoupled;
        if (st.coupled) {
            // turns of each target's phase, by the coupled qubit's place: a bit
            // of the group index, or outside the tile
            SweepCouple cp{};
            for (int a = 0; a < b.k; ++a)
                for (int c = 0; c < b.n_couple; ++c) {
                    const int q = b.couple_q[c];
                    if (q >= n) continue;  // no such qubit: never set
                    double turn = b.couple[a * b.n_couple + c] / 6.283185307179586476925286766559;
                    turn -= std::floor(turn);
                    int p = q;
                    if (q >= L) {
                        int r = 0;
                        while (r < st.args.n_hi && st.hi_pos[r] != q) ++r;
                        p = r < st.args.n_hi ? L + r : -1;
                    }
                    const uint64_t u = uint64_t(std::llround(std::ldexp(turn, 62))) << 2;  // (2^64 does not fit)
                    if (p < 0) cp.out[a][q] = u;
                    for (int j = 0; j < left; ++j) {
                        if (group[j] != p) continue;
                        if (j < 5)
                            for (int l = 0; l < 32; ++l) cp.lane[a][l] += (l >> j) & 1 ? u : 0;
                        else
                            for (int w = 0; w < 8; ++w) cp.wave[a][w] += (w >> (j - 5)) & 1 ? u : 0;
                    }
                }
            std::memcpy(mat + sweep_matrix_stride(true), &cp, sizeof cp);
        }
        for (int a = 0; a < k; ++a) s.bit[a] = slot_bytes(dt, 1u << pos[a]);
        if (s.kind == kSweepRows5)
            std::memcpy(mat, b.m, 1024 * 2 * sizeof(double));
        else if (k < 5)
            pack_matrix(dt, 12, k, 0, b.m, 0, mat);
        else if (st.split) {
            if (few_products(b) || !pack5_split(b, reinterpret_cast<uint16_t*>(mat))) {
                s.kind |= kSweepFp32;
                pack5_fp32(b, reinterpret_cast<float*>(mat));
            }
        } else if (dt == SV_C64)
            pack5(b, n, reinterpret_cast<float*>(mat));
        else
            pack5(b, n, reinterpret_cast<double*>(mat));
        desc[j] = s;
    }
}

void launch_sweep(sv_handle_s* h, sv_dtype_t dt, void* psi_v, const SweepStep& st, const void* buffer)
{
    char* psi = static_cast<char*>(psi_v);
    const auto* blocks = static_cast<const SweepBlock*>(buffer);
    const auto* mats = static_cast<const char*>(buffer) + ((sizeof(SweepBlock) * st.blocks.size() + 255) & ~size_t(255));
    const SweepArgs& a = st.args;
    const dim3 grid{unsigned((a.n_tiles + a.tiles_per_wg - 1) / a.tiles_per_wg)};
    const bool small = a.amps < (uint64_t(1) << kPadQubits);
    const bool large_tile = st.tile_bits > tile_bits(dt);
#define SV_SWEEP(...) \
    hipLaunchKernelGGL((k_sweep<__VA_ARGS__>), grid, dim3(large_tile ? 512 : 256), 0, h->stream, psi, blocks, mats, a)
    if (dt == SV_C64) {
        if (large_tile && small)
            SV_SWEEP(float, 13, 512, true);
        else if (small)
            SV_SWEEP(float, 12, 256, true);
        else if (large_tile && st.coupled)
            SV_SWEEP(float, 13, 512, false, true, true);
        else if (large_tile)
            SV_SWEEP(float, 13, 512, false, true);
        else if (st.coupled)
            SV_SWEEP(float, 12, 256, false, true, true);
        else if (st.split)
            SV_SWEEP(float, 12, 256, false, true);
        else
            SV_SWEEP(float, 12, 256, false);
    } else {
        if (large_tile && small)
            SV_SWEEP(double, 12, 512, true);
        else if (small)
            SV_SWEEP(double, 11, 256, true);
        else if (large_tile)
            SV_SWEEP(double, 12, 512, false);
        else
            SV_SWEEP(double, 11, 256, false);
    }
#undef SV_SWEEP
    SV_HIP(hipGetLastError());
}

void launch_batch_level(hipStream_t stream, const BatchArgs& a, uint64_t first, uint32_t n_entries, bool first_level)
{
    char* states = static_cast<char*>(a.states);
    if (first_level)
        hipLaunchKernelGGL(k_batch_level<true>, dim3(n_entries), dim3(256), 0, stream, states, a.sweeps, a.entries + first,
                           a.sweep_blocks, a.sweep_mats, a.z_masks, a.partials);
    else
        hipLaunchKernelGGL(k_batch_level<false>, dim3(n_entries), dim3(256), 0, stream, states, a.sweeps,
                           a.entries + first, a.sweep_blocks, a.sweep_mats, a.z_masks, a.partials);
    SV_HIP(hipGetLastError());
}

}  // namespace sv

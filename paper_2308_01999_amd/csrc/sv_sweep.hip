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
// mixes) and multiplies them in the same order of operations as the
// single-block sweeps (sv_tile.h, sv_apply.hip), so a state has the same bits
// whichever sweep ran.
//
// What bounds it: a block alone is bound by HBM (the 30-qubit complex64 sweep:
// 2.9 ms).  In a sweep of several, the matrix cores take about 1.7 ms a block
// there, and they share their issue slots with the vector ALUs (a vector
// instruction costs the matrix pipe 2.7 cycles with several waves on a SIMD), so the
// kernel keeps the address work to one XOR per LDS access.  32 KiB tiles and
// 256 threads: the runs of 128 bytes that they leave for eight free bits
// stream at 4.6-5.4 TB/s, and three workgroups a CU overlap one's loads with
// another's products; tiles of 64 and 128 KiB (fewer sweeps) measured slower,
// 2.4 and 2.5 ms for two blocks on 29 qubits against 2.35.
// Measured, before (a sweep per block) and after: 30-qubit brickwork circuit
// of depth 20, complex64, 52 blocks in 20 sweeps, 156 -> 115 ms; 28-qubit
// random CNOT/CP circuit, complex128, 71 -> 53 ms; 19-qubit circuit on random
// pairs, complex128, 660 -> 323 us; 14 qubits complex64 as a recorded graph,
// 155 -> 92 us; 12 qubits complex128 194 -> 117 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "sv_batch.h"
#include "sv_tile.h"

namespace sv {
namespace {

using namespace tile;

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// LDS slot of tile-local amplitude a: bits 1-4 XORed with bits 6-9.  Bit 0
// stays, so a pair (i, i + 1) keeps its order and stages as one 16-byte
// slot without a swap.  The XOR is linear over bits, so the slot of a group's
// amplitude r is slot(base) ^ slot(off(r)): one XOR per access with the
// host's swizzled offset as the scalar operand.
__host__ __device__ __forceinline__ uint32_t slot(uint32_t a) { return a ^ ((a >> 5) & 30u); }

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

// Group index -> tile-local base: a zero inserted at each target position
// (v + the bits at and above the position, which moves them up by one).
template <int K>
__device__ __forceinline__ uint32_t spread(uint32_t v, const uint32_t* ins)
{
#pragma unroll
    for (int j = 0; j < K; ++j) v += v & ins[j];
    return v;
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
            re[q] = m[q * 64 + lane];
            im[q] = m[256 + q * 64 + lane];
            if (SUM) sum[q] = m[512 + q * 64 + lane];
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
            re[h] = m[(rt * 4 + h) * 64 + lane];
            im[h] = m[(8 + rt * 4 + h) * 64 + lane];
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
                                       uint32_t g0, int lane)
{
    const int col = lane & 31, half = lane >> 5;
    if (!READY) o.load<SUM>(m, lane);
    const uint32_t base = 8u * slot(spread<5>(uint32_t(col), b.ins)) ^ 8u * slot(spread<5>(g0, b.ins));
    uint32_t in = base ^ (half ? b.off[1] : 0u), out = base ^ (half ? b.off[4] : 0u);
    asm volatile("" : "+v"(in), "+v"(out));  // keep (base ^ half part) ^ uniform part: one XOR per access
    f32x2 x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = *reinterpret_cast<const f32x2*>(lds + (in ^ b.off[2 * j]));
    f32x16 p1 = {0}, p2 = {0}, p3 = {0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 vs = SUM ? o.sum[q] : o.re[q] + o.im[q];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const f32x2 xv = x[4 * q + jj];
            p1 = __builtin_amdgcn_mfma_f32_32x32x2f32(o.re[q][jj], xv.x, p1, 0, 0, 0);
            p2 = __builtin_amdgcn_mfma_f32_32x32x2f32(o.im[q][jj], xv.y, p2, 0, 0, 0);
            p3 = __builtin_amdgcn_mfma_f32_32x32x2f32(vs[jj], xv.x + xv.y, p3, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
        *reinterpret_cast<f32x2*>(lds + (out ^ b.off[8 * (r / 4) + (r % 4)])) =
            f32x2{p1[r] - p2[r], p3[r] - p1[r] - p2[r]};
}

// complex64, four qubits, on v_mfma_f32_16x16x4_f32 (the chain of
// k_tile_c64_k4), `steps` column tiles of 16 groups per wave.
__device__ __forceinline__ void block4(char* lds, const SweepBlock& b, const f32x4* __restrict__ m, uint32_t g0, int steps,
                                       int lane)
{
    const int col = lane & 15, q = lane >> 4;
    const f32x4 ar = m[lane], ai = m[64 + lane], as = m[128 + lane];
    const uint32_t lin = ((q & 1) ? b.off[1] : 0u) ^ ((q & 2) ? b.off[2] : 0u);
    const uint32_t lout = ((q & 1) ? b.off[4] : 0u) ^ ((q & 2) ? b.off[8] : 0u);
    for (int c = 0; c < steps; ++c) {
        const uint32_t base = 8u * slot(spread<4>(g0 + uint32_t(c * 16 + col), b.ins));
        f32x2 x[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) x[s] = *reinterpret_cast<const f32x2*>(lds + (base ^ lin ^ b.off[4 * s]));
        f32x4 p1 = {0}, p2 = {0}, p3 = {0};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            p1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[s], x[s].x, p1, 0, 0, 0);
            p2 = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[s], x[s].y, p2, 0, 0, 0);
            p3 = __builtin_amdgcn_mfma_f32_16x16x4f32(as[s], x[s].x + x[s].y, p3, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<f32x2*>(lds + (base ^ lout ^ b.off[r])) = f32x2{p1[r] - p2[r], p3[r] - p1[r] - p2[r]};
    }
}

// complex128, five qubits, on v_mfma_f64_16x16x4_f64: one column tile of 16
// groups per wave, two row tiles (the chain of k_tile_c128_k5).  The lane's
// inputs are matrix columns 4s + q, its outputs rows 16 rt + 4v + q.
template <bool SUM, bool READY>
__device__ __forceinline__ void block5(char* lds, const SweepBlock& b, const f64x2* __restrict__ m, Ops<double>& o,
                                       uint32_t g0, int lane)
{
    const int col = lane & 15, q = lane >> 4;
    const uint32_t base = 16u * slot(spread<5>(uint32_t(col), b.ins)) ^ 16u * slot(spread<5>(g0, b.ins));
    uint32_t at = base ^ ((q & 1) ? b.off[1] : 0u) ^ ((q & 2) ? b.off[2] : 0u);
    asm volatile("" : "+v"(at));
    f64x2 x[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) x[s] = *reinterpret_cast<const f64x2*>(lds + (at ^ b.off[4 * s]));
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
            *reinterpret_cast<f64x2*>(lds + (at ^ b.off[16 * rt + 4 * v])) =
                f64x2{p1[v] - p2[v], p3[v] - p1[v] - p2[v]};
    };
    if (!READY) o.load_rows(m, lane, 0);
    rows(0, o);
    if (!READY) second.load_rows(m, lane, 1);
    rows(1, second);
}

// k <= 3 (complex64) or k <= 4 (complex128) on the vector units, one group
// per thread and step, in the order of k_apply_dense.
template <typename R, int K>
__device__ __forceinline__ void block_small(char* lds, const SweepBlock& b, const typename Amp<R>::V* __restrict__ m,
                                            uint32_t groups, int nt)
{
    using V = typename Amp<R>::V;
    constexpr int D = 1 << K;
    for (uint32_t g = threadIdx.x; g < groups; g += uint32_t(nt)) {
        asm volatile("" ::: "memory");  // the matrix stays out of the registers
        const uint32_t base = Amp<R>::kBytes * slot(spread<K>(g, b.ins));
        V v[D];
#pragma unroll
        for (int c = 0; c < D; ++c) v[c] = *reinterpret_cast<const V*>(lds + (base ^ b.off[c]));
#pragma unroll
        for (int r = 0; r < D; ++r) {
            R re = 0, im = 0;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                const V e = m[r * D + c];
                re = fma(e.x, v[c].x, re);
                re = fma(-e.y, v[c].y, re);
                im = fma(e.x, v[c].y, im);
                im = fma(e.y, v[c].x, im);
            }
            *reinterpret_cast<V*>(lds + (base ^ b.off[r])) = V{re, im};
        }
    }
}

// complex128, five qubits, states of fewer than 11 qubits: on the vector units
// in the order of k_apply_dense, one group per lane and 8 rows per wave (64
// groups, four waves).  Every wave reads its groups' inputs before any writes.
__device__ __forceinline__ void block5_rows(char* lds, const SweepBlock& b, const f64x2* __restrict__ m, int wave, int lane)
{
    const uint32_t base = 16u * slot(spread<5>(uint32_t(lane), b.ins));
    f64x2 v[32], y[8];
#pragma unroll
    for (int c = 0; c < 32; ++c) v[c] = *reinterpret_cast<const f64x2*>(lds + (base ^ b.off[c]));
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const f64x2* row = m + (wave * 8 + r) * 32;
        double re = 0, im = 0;
#pragma unroll
        for (int c = 0; c < 32; ++c) {
            re = fma(row[c].x, v[c].x, re);
            re = fma(-row[c].y, v[c].y, re);
            im = fma(row[c].x, v[c].y, im);
            im = fma(row[c].y, v[c].x, im);
        }
        y[r] = f64x2{re, im};
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 8; ++r) *reinterpret_cast<f64x2*>(lds + (base ^ b.off[wave * 8 + r])) = y[r];
}

// A block's descriptor from the wave's copy of it (lane l holds word l).
__device__ __forceinline__ SweepBlock unpack_block(uint32_t words)
{
    auto word = [&](int i) { return uint32_t(__builtin_amdgcn_readlane(int(words), i)); };
    SweepBlock b;
#pragma unroll
    for (int j = 0; j < 5; ++j) b.ins[j] = word(j);
    b.kind = int32_t(word(5));
#pragma unroll
    for (int r = 0; r < 32; ++r) b.off[r] = word(6 + r);
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
    double c[16];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(lds + 8u * slot(uint32_t(u * NT + tid) * 2));
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
        *reinterpret_cast<f64x2*>(lds + 8u * slot(uint32_t(u * NT + tid) * 2)) = f64x2{c[2 * u], c[2 * u + 1]};
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
                *reinterpret_cast<const double*>(lds + 8u * slot(uint32_t((k >> 1) * NT + tid) * 2) + 8 * (k & 1));
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
template <typename R, int T, int NT, bool SMALL, bool FIRST = false, bool SUMS = false>
__device__ __forceinline__ void sweep_tiles(char* __restrict__ psi, const SweepBlock* __restrict__ blocks,
                                            const char* __restrict__ mats, const SweepArgs& a, uint64_t wg,
                                            char* lds, const ZSums& zs)
{
    using A = Amp<R>;
    using W = typename A::W;
    constexpr int NV = (1 << T) / A::kPerVec / NT;       // 16-byte vectors per thread
    constexpr int kCols = sizeof(R) == 4 ? 32 : 16;      // groups per wave
    constexpr uint32_t kStride = sweep_matrix_stride(sizeof(R) == 4);
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
    char* base = psi + A::kBytes * tile_origin(t0, a);
    W buf[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
        if (FIRST || (SMALL && uint64_t(u * NT + tid) * A::kPerVec >= a.amps))
            buf[u] = W{};
        else
            buf[u] = __builtin_nontemporal_load(reinterpret_cast<const W*>(base + roff[u] + loff));
    }
    if (FIRST && base == psi && tid == 0) buf[0][0] = 1;
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
        if (FIRST && base != psi) {
            // |0..0> is zero on every tile but the first, and so is its image:
            // such a tile is only written
#pragma unroll
            for (int u = 0; u < NV; ++u) __builtin_nontemporal_store(W{}, reinterpret_cast<W*>(base + roff[u] + loff));
            if (t + 1 < t1) base = psi + A::kBytes * tile_origin(t + 1, a);
            continue;
        }
#pragma unroll
        for (int u = 0; u < NV; ++u)
            *reinterpret_cast<W*>(lds + A::kBytes * slot(uint32_t(u * NT + tid) * A::kPerVec)) = buf[u];
        __syncthreads();
        char* nbase = base;
        if (!SMALL && t + 1 < t1) {
            nbase = psi + A::kBytes * tile_origin(t + 1, a);
            if (!FIRST) {
#pragma unroll
                for (int u = 0; u < NV; ++u)
                    buf[u] = __builtin_nontemporal_load(reinterpret_cast<const W*>(nbase + roff[u] + loff));
            }
        }
        if constexpr (!SMALL) {
            for (int i = 0; i < a.n_blocks; ++i) {
                Ops<R> o;
                block5<false, false>(lds, blocks[i], matrix(i), o, uint32_t(wave * kCols), lane);
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
                    block5<true, true>(lds, b, matrix(i), now, uint32_t(wave * kCols), lane);
                    return;
                }
                const auto* mv = reinterpret_cast<const typename A::V*>(matrix(i));
                if constexpr (sizeof(R) == 8 && NT == 256)
                    if (b.kind == kSweepRows5) block5_rows(lds, blocks[i], mv, wave, lane);
                if (b.kind == 1) block_small<R, 1>(lds, b, mv, 1u << (T - 1), NT);
                if (b.kind == 2) block_small<R, 2>(lds, b, mv, 1u << (T - 2), NT);
                if (b.kind == 3) block_small<R, 3>(lds, b, mv, 1u << (T - 3), NT);
                if (b.kind == 4) {
                    if constexpr (sizeof(R) == 8)
                        block_small<R, 4>(lds, b, mv, 1u << (T - 4), NT);
                    else
                        block4(lds, b, matrix(i), uint32_t(wave * 64), 4, lane);
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
                *reinterpret_cast<const W*>(lds + A::kBytes * slot(uint32_t(u * NT + tid) * A::kPerVec)),
                reinterpret_cast<W*>(base + roff[u] + loff));
        }
        if constexpr (SUMS)
            if (zs.n_terms >= 0) add_z_sums(lds, a, zs, uint64_t(base - psi + int64_t(roff[0]) + loff) / A::kBytes, tid);
        base = nbase;
        __syncthreads();
    }
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

template <typename R, int T, int NT, bool SMALL>
__global__ __launch_bounds__(NT, SMALL ? 1 : 3) void k_sweep(char* __restrict__ psi, const SweepBlock* __restrict__ blocks,
                                                            const char* __restrict__ mats, SweepArgs a)
{
    __shared__ __align__(16) char lds[Amp<R>::kBytes << T];
    sweep_tiles<R, T, NT, SMALL>(psi, blocks, mats, a, blockIdx.x, lds, ZSums{nullptr, -1, nullptr, nullptr});
}

// Level path of a batch: workgroup w sweeps its tiles of one step of one
// circuit; on a circuit's last step it also leaves the Z-type sums of its
// tiles.  FIRST: the states are |0..0>.  Bound by HBM and the matrix pipe
// about equally: a step holds two blocks in the mean (in program order, since
// a swap would change the states' bits), so that a batch of 512 circuits of 8-20
// qubits moves half the bytes of one sweep per block: 13.5 -> 10.6 ms.
template <bool FIRST>
__global__ __launch_bounds__(256, 3) void k_batch_level(char* __restrict__ states, const BatchSweep* __restrict__ sweeps,
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
    sweep_tiles<float, 12, 256, false, FIRST, true>(states + 8 * d.state_off, blocks + d.block0,
                                                    mats + uint64_t(d.block0) * sweep_matrix_stride(true), d.a, e.wg,
                                                    lds, zs);
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
// their bits).
constexpr int kReorderQubits = 22;
constexpr int kReorderWindow = 96;

// Shortest runs of a tile: 128 bytes, the line of the L2.  (Runs of 64 bytes
// below 22 qubits, for 7% fewer sweeps, measured no faster: 339 us against 324
// on 19 qubits complex128.)
constexpr int min_run_bits(sv_dtype_t dt) { return dt == SV_C64 ? 4 : 3; }

// Most blocks of one sweep: its descriptors and matrices fit a segment of the
// handle's matrix ring (16 KiB a block at most, 1 MiB).
constexpr size_t kMaxSweepBlocks = 48;

// Largest state of multi-block sweeps: the lanes' part of an address (three
// index bits below the fifth highest one) fits 32 bits.
constexpr int kMaxSweepQubitsC64 = 34, kMaxSweepQubitsC128 = 33;

uint64_t qubit_mask(const FusedBlock& b)
{
    uint64_t m = 0;
    for (int a = 0; a < b.k; ++a) m |= uint64_t(1) << b.targets[a];
    return m;
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
    uint64_t per = a.n_tiles / (uint64_t(cu_count) * SV_TILE_WGS_PER_CU);
    per = std::max<uint64_t>(1, std::min<uint64_t>(per, SV_TILES_PER_WG_MAX_K5));
    a.tiles_per_wg = per;
    if ((per & (per - 1)) == 0)
        while ((uint64_t(1) << a.trot) < per) ++a.trot;
}

}  // namespace

std::vector<SweepStep> plan_sweeps(sv_dtype_t dt, int n, int cu_count, const FusedBlock* blocks, int first, int end,
                                   const SweepRules& rules)
{
    std::vector<SweepStep> steps;
    const bool one_tile = n <= tile_bits(dt) + (rules.pad_all ? 0 : 1);
    const int T = std::max(tile_bits(dt), one_tile ? n : 0);
    const int lo = min_run_bits(dt);
    auto eligible = [&](const FusedBlock& b) {
        if (b.diagonal || b.n_couple > 0 || b.k > 5) return false;
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
    auto fits = [&](uint64_t on) { return one_tile || __builtin_popcountll(on >> lo) <= T - lo; };
    auto add = [&](std::vector<int>&& take, uint64_t on) {
        SweepStep st;
        st.multi = take.size() > 1 || ((n < kReorderQubits || rules.pad_all) && eligible(blocks[take[0]]));
        st.blocks = std::move(take);
        st.padded = rules.pad_all || n >= kPadQubits;
        if (st.multi) {
            st.tile_bits = T;
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
        // a block may join a sweep ahead of blocks left behind that share no
        // qubit with it (they commute); of the first ready seeds, the one
        // whose sweep takes most blocks
        const size_t hi = std::min(rest.size(), at + kReorderWindow);
        std::vector<int> best;
        uint64_t best_on = 0;
        int seeds = 0;
        uint64_t before = 0;
        for (size_t s = at; s < hi && seeds < 8; ++s) {
            const uint64_t qs = qubit_mask(blocks[rest[s]]);
            const bool ready = !(qs & before) && eligible(blocks[rest[s]]);
            before |= touched_mask(blocks[rest[s]]);
            if (!ready) continue;
            ++seeds;
            std::vector<int> take{rest[s]};
            uint64_t on = qs;
            std::vector<char> in(hi - at, 0);
            in[s - at] = 1;
            while (take.size() < kMaxSweepBlocks) {
                int pick = -1, cost = 65;
                uint64_t blocked = 0;
                for (size_t j = at; j < hi; ++j) {
                    if (in[j - at]) continue;
                    const uint64_t q = qubit_mask(blocks[rest[j]]);
                    if (!(q & blocked) && eligible(blocks[rest[j]]) && fits(on | q)) {
                        const int c = __builtin_popcountll((on | q) >> lo);
                        if (c < cost) {
                            cost = c;
                            pick = int(j);
                        }
                    }
                    blocked |= touched_mask(blocks[rest[j]]);
                }
                if (pick < 0) break;
                in[pick - at] = 1;
                on |= qubit_mask(blocks[rest[pick]]);
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

}  // namespace

size_t sweep_bytes(sv_dtype_t dt, const SweepStep& st)
{
    return ((sizeof(SweepBlock) * st.blocks.size() + 255) & ~size_t(255)) +
           sweep_matrix_stride(dt == SV_C64) * st.blocks.size();
}

void pack_sweep(sv_dtype_t dt, const SweepStep& st, const FusedBlock* blocks, void* dst)
{
    pack_sweep(dt, st, blocks, static_cast<SweepBlock*>(dst),
               static_cast<char*>(dst) + ((sizeof(SweepBlock) * st.blocks.size() + 255) & ~size_t(255)));
}

void pack_sweep(sv_dtype_t dt, const SweepStep& st, const FusedBlock* blocks, SweepBlock* desc, char* mat)
{
    const int L = st.args.L, T = st.tile_bits, n = 63 - __builtin_clzll(st.args.amps);
    for (size_t j = 0; j < st.blocks.size(); ++j, mat += sweep_matrix_stride(dt == SV_C64)) {
        const FusedBlock& b = blocks[st.blocks[j]];
        const int k = st.padded ? 5 : b.k;
        SweepBlock s{};
        s.kind = k < 5 ? k : (dt == SV_C128 && n < 11) ? kSweepRows5 : kSweepMfma5;
        // tile-local positions of the targets, then of the padding qubits
        // (the lowest positions that are free)
        int pos[5] = {};
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
        int w = 0;
        for (int p = 0; p < T; ++p)
            if ((used >> p) & 1) s.ins[w++] = ~((1u << p) - 1u);
        for (int r = 0; r < (1 << k); ++r) {
            uint32_t o = 0;
            for (int a = 0; a < k; ++a)
                if ((r >> a) & 1) o |= 1u << pos[a];
            s.off[r] = (dt == SV_C64 ? 8u : 16u) * slot(o);
        }
        desc[j] = s;
        if (s.kind == kSweepRows5)
            std::memcpy(mat, b.m, 1024 * 2 * sizeof(double));
        else if (k < 5)
            pack_matrix(dt, 12, k, 0, b.m, 0, mat);
        else if (dt == SV_C64)
            pack5(b, n, reinterpret_cast<float*>(mat));
        else
            pack5(b, n, reinterpret_cast<double*>(mat));
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
#define SV_SWEEP(R, T, NT, SMALL) \
    hipLaunchKernelGGL((k_sweep<R, T, NT, SMALL>), grid, dim3(NT), 0, h->stream, psi, blocks, mats, a)
    if (dt == SV_C64) {
        if (large_tile)
            SV_SWEEP(float, 13, 512, true);
        else if (small)
            SV_SWEEP(float, 12, 256, true);
        else
            SV_SWEEP(float, 12, 256, false);
    } else {
        if (large_tile)
            SV_SWEEP(double, 12, 512, true);
        else if (small)
            SV_SWEEP(double, 11, 256, true);
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

// Device-side helpers shared by the gfx950 kernels of libtq.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include "tq.h"
#include "tq_layout.h"

namespace tq {

constexpr int kGroup = 8;            // elements served by one Philox4x32 call = one lane's work item
constexpr int kBlock = 256;          // threads per workgroup (4 wavefronts of 64)
constexpr int kTile = kBlock * kGroup;  // elements per workgroup tile (2048)

// a ^ b ^ c in one instruction (the three-input bitwise operation of this ISA, truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies whose
// halves are crossed over and xored with a Weyl-sequence round key.  Operands that are
// uniform over the wavefront (key, worker, step, high counter word) stay in SGPRs and
// their multiplies run on the scalar unit; only the lane's counter word c0 is per-lane.
// The xors of the first three rounds are grouped so that the uniform pair is combined on
// the scalar unit (first round: c1, c2, c3 uniform; second: c0, c1; third: c3); from then
// on every word differs per lane and each output word is one three-input xor.
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t h0 = (uint32_t)(p0 >> 32), h1 = (uint32_t)(p1 >> 32);
        uint32_t n0, n2;
        if (r == 0) { n0 = h1 ^ c1 ^ k0; n2 = h0 ^ (c3 ^ k1); }
        else if (r == 1) { n0 = h1 ^ (c1 ^ k0); n2 = c3 ^ (h0 ^ k1); }
        else if (r == 2) { n0 = xor3(h1, c1, k0); n2 = h0 ^ (c3 ^ k1); }
        else { n0 = xor3(h1, c1, k0); n2 = xor3(h0, c3, k1); }
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Pointer table of a batched launch: blockIdx.y selects the tensor (one simulated worker, or
// one of several same-shaped tensors of one worker).  Passed by value in the kernel arguments.
constexpr int kMaxBatch = TQ_MAX_WORKERS;
struct PtrTable {
    const void* p[kMaxBatch];
};
struct MutPtrTable {
    void* p[kMaxBatch];
};

// A launch of `nblocks` workgroups.  The dispatch packet counts work-items per dimension in 32
// bits, so blocks * threads of one dimension must stay below 2^32: long grids are folded into
// (x, z), grid.y being the tensor of a batch.  Workgroups past `nblocks` (the last z-row is
// padded) find nothing to do and exit; every kernel tests for that before touching memory.
__device__ __forceinline__ uint32_t linear_block() { return blockIdx.x + blockIdx.z * gridDim.x; }

// Builds with -DTQ_TEST_GRID_FOLD (the test build only) read TQ_TEST_MAX_GRID_X from the
// environment, once, to lower the fold point, so that tests can drive the folded path of every
// kernel with small inputs; the product build has no such hook.
inline bool fold_grid(uint64_t nblocks, unsigned threads, unsigned count, dim3& grid)
{
#ifdef TQ_TEST_GRID_FOLD
    static const uint64_t forced = [] {
        const char* e = getenv("TQ_TEST_MAX_GRID_X");
        return e ? strtoull(e, nullptr, 10) : 0ull;
    }();
#else
    constexpr uint64_t forced = 0;
#endif
    uint64_t max_x = (1ull << 31) / threads;                       // x * threads <= 2^31
    if (forced > 0 && forced < max_x) max_x = forced;
    if (nblocks == 0 || nblocks > 0xFFFFFFFFull) return false;
    const uint64_t gx = nblocks < max_x ? nblocks : max_x;
    const uint64_t gz = (nblocks + gx - 1) / gx;
    if (gz > 65535 || gx * gz > 0xFFFFFFFFull) return false;
    grid = dim3((unsigned)gx, count, (unsigned)gz);
    return true;
}

// Whether an fp32 output of so many bytes is stored past the caches (non-temporally).  Well above half the
// 256 MiB of the memory-side cache little of it would be found there by whoever reads it next, and
// written back late it costs more than written out at once.  The average of N payloads, us, through / past the caches,
// repeated alone, after another kernel has left the cache full of its own dirty lines, and there with a reader of the
// output behind it:
//   40 M  b = 2, N = 8   39 / 40    65 / 61    116 / 127        b = 4, N = 1   27.5 / 27   39 / 37.5   91 / 110
//   50 M                 57 / 49    80 / 75.5  149.5 / 152                     33.5 / 33.5 47 / 45     123 / 130.5
//   80 M                 92 / 77    110 / 116  225 / 222                       63 / 51     70 / 70     190 / 191
//   124 M                135 / 114  154 / 183  325 / 333                       94.5 / 78   101 / 105   280 / 281
// So the call by itself gains or, after such a kernel, loses, and from 50 M on what follows it gets that back: a whole
// step of 8 x 124 M 1438 / 1409.  Below, a reader pays up to a quarter.
inline bool output_past_caches(uint64_t bytes) { return bytes > (160ull << 20); }

typedef float float4_native __attribute__((ext_vector_type(4)));

// Exchanges a wavefront's 32 bytes per lane between two layouts (it undoes itself; the whole wavefront is active):
// x = the lane's own group of 8 fp32 values, and x = the pieces of 16 bytes with which a load or store instruction
// covers 1 KiB in one piece: piece wave_piece(lane) of the wavefront's first 64 in x[0..3], of its second in x[4..7].
// The lower half holds the even pieces of the first load (a group's first half), the upper half the odd ones, so one
// v_permlane32_swap per register is all it takes.
__device__ __forceinline__ uint32_t wave_piece(uint32_t lane) { return 2u * (lane & 31u) + (lane >> 5); }
__device__ __forceinline__ void swap_pieces(float (&x)[8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {                              // the upper half of x[j] against the lower half of x[4 + j]
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[j]), __float_as_uint(x[4 + j]), false, false);
        x[j] = __uint_as_float(r[0]);
        x[4 + j] = __uint_as_float(r[1]);
    }
}

// 32 bytes per lane, stored by a WHOLE wavefront (every lane owns a group; `o` is lane
// 0's address).  Stored directly, each of the wavefront's two 16-byte store instructions would
// touch every line of its 2 KiB half-way; as pieces each writes 1 KiB in one piece (the
// aggregate of 8 x 124 M elements 139 us -> 118, of 8 x 11.2 M 20.8 -> 15.6).  Two ways to lay the pieces out, neither better
// everywhere: in registers, beside the look-ups whose LDS reads bound many launches, or through LDS, which takes fewer
// registers where two tiles' values are live at once (16 workers at b = 2: 62 against 70, 8 wavefronts per SIMD against 7).
// Who takes which: lds_above (tq_decode.hip); the simulation takes LDS.
template <bool STREAM>
__device__ __forceinline__ void store_pieces(float4_native* p, float4_native a, float4_native b)
{
    if constexpr (STREAM) {
        __builtin_nontemporal_store(a, p);
        __builtin_nontemporal_store(b, p + 64);
    } else {
        p[0] = a;
        p[64] = b;
    }
}

// `x` = the lane's pieces already.
template <bool STREAM>
__device__ __forceinline__ void store_lane_pieces(float* o, uint32_t lane, const float (&x)[8])
{
    const float4_native a = {x[0], x[1], x[2], x[3]}, b = {x[4], x[5], x[6], x[7]};
    store_pieces<STREAM>(reinterpret_cast<float4_native*>(o) + wave_piece(lane), a, b);
}

template <bool STREAM>
__device__ __forceinline__ void store8_wave(float* o, uint32_t lane, const float (&x)[8])
{
    float y[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = x[j];
    swap_pieces(y);
    store_lane_pieces<STREAM>(o, lane, y);
}

// `wb` is the wavefront's own 2 KiB of LDS; a wavefront's LDS operations complete in order, so no
// barrier.
template <bool STREAM>
__device__ __forceinline__ void store8_wave_lds(float* o, uint32_t lane, const float (&x)[8], float4_native* wb)
{
    wb[2 * lane] = float4_native{x[0], x[1], x[2], x[3]};
    wb[2 * lane + 1] = float4_native{x[4], x[5], x[6], x[7]};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // other lanes' halves: the compiler keeps the order, no instruction
    const float4_native a = wb[lane], b = wb[64 + lane];
    store_pieces<STREAM>(reinterpret_cast<float4_native*>(o) + lane, a, b);
}

// The same, added to what the lane's pieces held.
template <bool STREAM>
__device__ __forceinline__ void store8_wave_lds(float* o, uint32_t lane, const float (&x)[8], float4_native* wb, const float (&held)[8])
{
    wb[2 * lane] = float4_native{x[0], x[1], x[2], x[3]};
    wb[2 * lane + 1] = float4_native{x[4], x[5], x[6], x[7]};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const float4_native c = wb[lane], d = wb[64 + lane];
    const float4_native a = {held[0] + c.x, held[1] + c.y, held[2] + c.z, held[3] + c.w};
    const float4_native b = {held[4] + d.x, held[5] + d.y, held[6] + d.z, held[7] + d.w};
    store_pieces<STREAM>(reinterpret_cast<float4_native*>(o) + lane, a, b);
}

// Inclusive prefix sums over a wavefront by moves inside the vector unit: inside rows of 16 lanes, then the
// rows' totals handed on (lane 15 of a row to the next row, lane 31 to the upper half).  6 steps of a few clocks each,
// where a shuffle through LDS takes about a hundred.  Lanes without a source see 0.  The whole wavefront is active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_or_zero(unsigned long long v)
{
    return (unsigned long long)dpp_or_zero<CTRL, ROWS>((uint32_t)v) |
           (unsigned long long)dpp_or_zero<CTRL, ROWS>((uint32_t)(v >> 32)) << 32;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
    return __hiloint2double(hi, lo);
}
template <typename T>
__device__ __forceinline__ T row_scan(T v)
{
    v += dpp_or_zero<0x111, 0xf>(v);
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    return v;
}
template <typename T>
__device__ __forceinline__ T wave_scan(T v)
{
    v = row_scan(v);
    v += dpp_or_zero<0x142, 0xa>(v);
    v += dpp_or_zero<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ unsigned long long lane_value(unsigned long long v, int lane)
{
    return (unsigned long long)lane_value((uint32_t)v, lane) | (unsigned long long)lane_value((uint32_t)(v >> 32), lane) << 32;
}
__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

}  // namespace tq

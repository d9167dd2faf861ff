// tq_compress: Alg. 1 client step of arXiv 2402.01798 -- truncate (Eq. 1), locate the cell
// and its rounding probability, round stochastically (Eq. 2), pack b-bit codes.
//
// One lane owns 8 consecutive elements: they share one Philox4x32-10 call (8 x 16 random
// bits) and their codes are exactly b bytes of the payload, so a wavefront reads 2 KiB
// (fp32) or 1 KiB (bf16) of gradient and writes 64*b contiguous bytes.
#include <type_traits>

#include "tq_device.h"


namespace tq {

// NT: non-temporal loads.  In the main path this is the last read of the gradient.  While the batch is small enough
// that the memory-side cache still holds much of what the statistics pass read, the hint keeps this kernel's misses
// from displacing the lines it is about to hit (-6 % on 8 x 45 MB); a larger batch gains by it too, if its
// lines are read whole (see load_groups_wave).
template <int DTYPE, bool NT>
__device__ __forceinline__ void load_group(const void* g, uint64_t e0, float (&x)[8])
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    if constexpr (DTYPE == TQ_F32) {
        const f4* p = reinterpret_cast<const f4*>(static_cast<const float*>(g) + e0);
        f4 a, b;
        if constexpr (NT) { a = __builtin_nontemporal_load(p); b = __builtin_nontemporal_load(p + 1); }
        else { a = p[0]; b = p[1]; }
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    } else {
        const u4* p = reinterpret_cast<const u4*>(static_cast<const uint16_t*>(g) + e0);
        u4 v;
        if constexpr (NT) v = __builtin_nontemporal_load(p);
        else v = p[0];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = __uint_as_float(w[i] << 16);
            x[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
}

// fp32, a whole wavefront whose lanes own the 64 groups from element `base` on: the two loads read 1 KiB in one piece
// each, and swap_pieces gives every lane the two pieces of its own group.  A non-temporal line is not kept for a second load that wants its other
// half: 8 x 124 M at b = 2, one step, a lane's own 32 bytes through the caches / past them / this way past them
// 1356 / 1441 / 1338 us (with 68 layers 1458 / 1516 / 1406), 16 x 25.6 M at b = 3 with tables 642 / 664 / 625; pieces in the
// lanes' order exchanged by DPP moves 1338 / 1410 / 628.  On batches that the memory-side cache still holds the lane's own
// 32 bytes are as good or better: 8 x 11.2 M 144.3 / 147.0.
__device__ __forceinline__ void load_groups_wave(const void* g, uint64_t base, uint32_t lane, float (&x)[8])
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4* p = reinterpret_cast<const f4*>(static_cast<const float*>(g) + base) + wave_piece(lane);
    const f4 a = __builtin_nontemporal_load(p), b = __builtin_nontemporal_load(p + 64);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}

template <int DTYPE>
__device__ __forceinline__ float load_one(const void* g, uint64_t e)
{
    if constexpr (DTYPE == TQ_F32) return static_cast<const float*>(g)[e];
    return __uint_as_float((uint32_t) static_cast<const uint16_t*>(g)[e] << 16);
}

// Levels and inverse widths of one bucket, kept in LDS for the per-lane look-ups of the
// level-table path: entry j = (l_j, inv_w[j], pivot_j, -), 16 bytes, where pivot_j = l_j for
// j < s and +inf from j = s on: the table the cell search walks.  The search carries the
// BYTE offset of its current entry, so no look-up needs an index-to-address shift.
struct LevelLds {
    float4 e[16];
};

__device__ __forceinline__ void fill_level_lds(LevelLds& tab, const tq_params_t* P, uint32_t s)
{
    if (threadIdx.x < 16) {
        const float l = P->level[threadIdx.x];
        tab.e[threadIdx.x] = make_float4(l, P->inv_w[threadIdx.x], threadIdx.x < s ? l : __builtin_inff(), 0.0f);
    }
}

// NaN -> +0 for a lane's 8 values.  NaN is rare, so the test is made as cheap as it can be:
// one unordered compare per PAIR of values, and the replacement itself only in wavefronts
// in which some lane saw one.
__device__ __forceinline__ void replace_nan(float (&x)[8])
{
    unsigned long long any = 0ull;                             // lane masks, combined on the scalar unit
#pragma unroll
    for (int i = 0; i < 4; ++i) any |= __builtin_amdgcn_ballot_w64(__builtin_isunordered(x[2 * i], x[2 * i + 1]));
    if (any != 0ull) {
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = (x[j] != x[j]) ? 0.0f : x[j];
    }
}

// Eq. (1) then Eq. (2) for one element; `rf` is the element's 16-bit draw as a float.
// Any codebook: cell k by comparison with the levels, p_r = (x - l_k) * inv_w[k] (two
// roundings), the upper end iff u = 1 - (rf + 1/2) / 2^16 <= p_r.  The uniform codebook: the
// same rounding stated through the position in units of cells, floor(t + U), U = (rf + 1/2) / 2^16.
// Uniform codebook: the code of one element.
template <int BITS>
__device__ __forceinline__ uint32_t quantize_uniform(float x, float rf, float alpha, float inv_step)
{
    constexpr uint32_t S = (1u << BITS) - 1u;
    const float xc = __builtin_amdgcn_fmed3f(x, -alpha, alpha);  // Eq. (1); the caller has replaced NaN
    // position in units of cells from -alpha, plus the dither's half grain; then the draw
    const float u = fmaf(xc, inv_step, 0.5f * (float)S + 1.0f / 131072.0f);
    const float v = fmaf(rf, 1.0f / 65536.0f, u);              // floor(v) = k + [rnd >= 1 - frac]
    const uint32_t code = (uint32_t)v;
    return code > S ? S : code;
}

// Level-table path: 16 * k for the cell k that holds x (l_k <= x < l_{k+1}; levels ascending),
// i.e. the byte offset of the cell's entry in LevelLds.
template <int BITS>
__device__ __forceinline__ uint32_t cell_offset(float x, const float (&lv)[16], const LevelLds& tab)
{
    uint32_t a;
    if constexpr (BITS == 2) {
        a = (x >= lv[1]) ? 16u : 0u;                           // two selects, no adds
        a = (x >= lv[2]) ? 32u : a;
    } else {
        // binary search over the pivots (padded with +inf to 2^b entries): the first pivot is a
        // scalar, the second a select between two scalars, the others are read from LDS at
        // (current entry + step), the step folded into the instruction's offset field
        constexpr uint32_t HALF = 1u << (BITS - 1), QUARTER = HALF >> 1;
        const bool top = x >= lv[HALF];
        const float pivot = top ? lv[HALF + QUARTER] : lv[QUARTER];
        a = top ? 16u * HALF : 0u;
        a |= (x >= pivot) ? 16u * QUARTER : 0u;
        const char* base = reinterpret_cast<const char*>(tab.e);
#pragma unroll
        for (uint32_t h = QUARTER >> 1; h >= 1; h >>= 1) {
            const float pv = *reinterpret_cast<const float*>(base + a + (16u * h + 8u));
            a |= (x >= pv) ? 16u * h : 0u;
        }
    }
    return a;
}

// Level-table path: does the element take the upper end of its cell?  p_r and the draw.
__device__ __forceinline__ bool rounds_up(float x, float rf, uint32_t a, const LevelLds& tab)
{
    const float2 cell = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(tab.e) + a);
    const float p_r = (x - cell.x) * cell.y;                   // (g - l_k) / |Delta_k| of Eq. (2)
    const float u = fmaf(rf, -1.0f / 65536.0f, 1.0f - 1.0f / 131072.0f);   // 1 - (r + 1/2) / 2^16, exact
    return u <= p_r;
}

template <int BITS, int GRID>
__device__ __forceinline__ uint32_t quantize(float x, float rf, float alpha, float inv_step,
                                             const float (&lv)[16], const LevelLds& tab)
{
    if constexpr (GRID == TQ_GRID_UNIFORM) {
        return quantize_uniform<BITS>(x, rf, alpha, inv_step);
    } else {
        const float xc = __builtin_amdgcn_fmed3f(x, -alpha, alpha);  // Eq. (1)
        const uint32_t a = cell_offset<BITS>(xc, lv, tab);
        return (a >> 4) + (rounds_up(xc, rf, a, tab) ? 1u : 0u);
    }
}

// Codes of one lane's 8 elements, packed little-endian into the low 8*BITS bits.
// PARTIAL: only the first n_valid elements exist; the others encode as 0 (pad bits).
// CLAMP (level tables): whether the truncation of Eq. (1) is written out; see truncates_itself.
template <int BITS, int GRID, bool PARTIAL, bool CLAMP = true>
__device__ __forceinline__ uint32_t encode_group(const float (&x)[8], const uint32_t (&rw)[4], int n_valid,
                                                 float alpha, float inv_step, const float (&lv)[16],
                                                 const LevelLds& tab)
{
    if constexpr (GRID == TQ_GRID_UNIFORM) {
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t r = (j & 1) ? (rw[j >> 1] >> 16) : (rw[j >> 1] & 0xFFFFu);
            uint32_t code = quantize_uniform<BITS>(x[j], (float)r, alpha, inv_step);
            if (PARTIAL && j >= n_valid) code = 0;
            word |= code << (j * BITS);
        }
        return word;
    } else {
        // code = k + up: the cells' offsets 16 k are merged into one word (shifted into place,
        // four bits too high), the upward roundings into another; their sum is the packed group
        uint32_t cells = 0, ups = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t r = (j & 1) ? (rw[j >> 1] >> 16) : (rw[j >> 1] & 0xFFFFu);
            const float xc = CLAMP ? __builtin_amdgcn_fmed3f(x[j], -alpha, alpha) : x[j];   // Eq. (1); NaN is gone
            uint32_t a = cell_offset<BITS>(xc, lv, tab);
            bool up = rounds_up(xc, (float)r, a, tab);
            if (PARTIAL && j >= n_valid) { a = 0; up = false; }
            cells |= (j * BITS >= 4) ? a << (j * BITS - 4) : a >> (4 - j * BITS);
            ups |= up ? 1u << (j * BITS) : 0u;
        }
        return cells + ups;
    }
}

// ---- the level-table path of regular codebooks ---------------------------------------------
//
// The general path above costs 18 (b = 3) or 13 (b = 2) vector instructions per element beside the
// draw's 5, many of them compares whose mask the next instruction needs (this ISA wants two other
// instructions in between, else s_nop).  For a REGULAR codebook -- every cell's stored reciprocal
// fits its width and the levels mirror each other about 0, as in every designed one -- the same codes
// come from 14 or 10 instructions without a single mask:
//   * the cell is searched on |x| (half the levels) by the SIGN BITS of |x| - l_j, which v_alignbit
//     shifts into the index one by one; the element's own sign completes it;
//   * the cell's LDS entry holds l_k, inv_w[k] 2^(32-b) and a word with k in its top b bits plus the
//     draw's half grain.  floor(p_r 2^(32-b)) (converted with saturation), the draw times 2^(16-b)
//     and that word add up to a number whose top b bits ARE the code: u <= p_r is the same as
//     p_r + (r + 1/2) / 2^16 >= 1, and dropping p_r's bits below 2^-(32-b) cannot change it (the other
//     terms are multiples of 2^(15-b), 1 is 2^(32-b)).  A negative p_r converts to 0 and the sum saturates at the
//     last code, so nothing is clamped;
//   * v_alignbit shifts the top b bits of each sum into the packed word.
// p_r itself is still a subtraction and a multiplication, each rounded (scaling by 2^(32-b) is exact).
//
// Regular (checked once per workgroup with the very arithmetic of p_r): for every cell k, with
// p_k(x) = (x - l_k) inv_w[k], and lo_k, hi_k the ends the search gives it,
//   |p_k(l_{k+1}) - 1| <= 2^-18,  |p_k(hi_k) - 1| <= 2^-18,  |p_k(lo_k)| <= 2^-18,  0 < inv_w[k] <= 2^90,
// and no level lies beyond +-alpha, so that the codes saturate where Eq. (1) truncates.
// p_k is monotone and 2^-17 <= u <= 1 - 2^-17.  So inside a cell no sum reaches the code k + 2, and where the
// search and the definition disagree about the cell (levels that mirror each other only to within
// rounding) they agree about the code: a value that the search leaves in cell k although it has reached
// l_{k+1} is encoded k + 1 by both (p_k >= u and p_{k+1} < u for every draw), and one that the search
// puts into cell k although it is below l_k is encoded k by both (p_k < u and p_{k-1} >= u).  The empty and the
// lopsided codebooks take the general path.
//
// Measured, general path -> this, with the same tiles: 16 x 25.6 M at b = 3 fp32 326 -> 300 us, bf16 263 -> 227, 25.6 M
// bf16 at b = 3 19.9 -> 16.8, at b = 2 15.0 -> 14.6; where it does not pay it is not checked for (mirrored_pays: b = 2 and
// 3 only).  What bounds it now is the pattern of its memory traffic: with the draws left out, the encoding left out, both,
// a launch of 16 x 25.6 M fp32 of 320 us took 313 / 309 / 307, one of 4 x 10^9 bf16 at b = 2 of 1780 1640 / 1625 / 1618.
struct CellLds {
    float4 e[8];             // entry neg * H + (H - 1 - i): cell m + i (x >= 0) or m - i, H = 2^(b-1), m = H - 1
    uint32_t regular;
};

constexpr float kRegularSlack = 3.814697265625e-06f;           // 2^-18
constexpr float kRegularMaxInv = 1.2379400392853803e27f;       // 2^90

// What one lane of the filling wavefront reads of the record (requested before anything is known about it).
struct CellReads { float l, l_next, inv, outer, inner; };

template <int BITS>
__device__ __forceinline__ CellReads read_cells(const tq_params_t* P, uint32_t lane)
{
    constexpr uint32_t H = 1u << (BITS - 1), M = H - 1;
    const uint32_t j = lane & (2u * H - 1u), i = H - 1u - (j & (H - 1u)), k = (j & H) ? M - i : M + i;
    return CellReads{P->level[k], P->level[k + 1], P->inv_w[k], P->level[M + 1u + i], P->level[i ? M + i : M + 1u]};
}

// Called by one whole wavefront (lane = its lane).
template <int BITS>
__device__ __forceinline__ void fill_cells(CellLds& tab, const CellReads& c, float alpha, uint32_t lane)
{
    constexpr uint32_t H = 1u << (BITS - 1), M = H - 1;
    const uint32_t j = lane & (2u * H - 1u), i = H - 1u - (j & (H - 1u));
    const bool neg = (j & H) != 0u;
    const uint32_t k = neg ? M - i : M + i;
    const float inner = i ? c.inner : -c.inner;                // this entry is |x| in [inner, outer)
    const float lo = neg ? -c.outer : inner, hi = neg ? -inner : c.outer;
    const float p_next = (c.l_next - c.l) * c.inv, p_hi = (hi - c.l) * c.inv, p_lo = (lo - c.l) * c.inv;
    const bool ok = fabsf(p_next - 1.0f) <= kRegularSlack && fabsf(p_hi - 1.0f) <= kRegularSlack &&
                    fabsf(p_lo) <= kRegularSlack && c.inv > 0.0f && c.inv <= kRegularMaxInv &&
                    fabsf(c.l) <= alpha && fabsf(c.l_next) <= alpha;
    if (lane < 2u * H)
        tab.e[j] = make_float4(c.l, c.inv * (float)(1u << (32 - BITS)),
                               __uint_as_float((k << (32 - BITS)) + (1u << (15 - BITS))), 0.0f);
    const bool regular = __builtin_amdgcn_ballot_w64(!ok) == 0ull;
    if (lane == 0) tab.regular = regular ? 1u : 0u;
}

// (index << 1) | sign bit of d
__device__ __forceinline__ uint32_t push_sign(uint32_t index, float d)
{
    return __builtin_amdgcn_alignbit(index, __float_as_uint(d), 31);
}

// The element's sum: its code in the top BITS bits.  HIGH: the draw is the high half of rw.
template <int BITS, bool HIGH>
__device__ __forceinline__ uint32_t code_on_top(float x, uint32_t rw, const float (&pv)[3], const CellLds& tab)
{
    const float y = __builtin_fabsf(x);
    uint32_t index = __float_as_uint(x) >> 31;
    if constexpr (BITS == 2) {
        index = push_sign(index, y - pv[0]);
    } else {
        // |x| below l_4 / l_5 / l_6: the two index bits are [below l_5] and, of the three signs, their parity
        const float d0 = y - pv[0], d1 = y - pv[1], d2 = y - pv[2];
        index = push_sign(index, d1);
        index = push_sign(index, __uint_as_float(xor3(__float_as_uint(d0), __float_as_uint(d1), __float_as_uint(d2))));
    }
    const float4 c = tab.e[index];
    const float p_r = (x - c.x) * c.y;                         // p_r * 2^(32-b), the two roundings of the definition
    uint32_t whole;                                            // 0 below, saturated far above: what v_cvt_u32_f32 does
    asm("v_cvt_u32_f32 %0, %1" : "=v"(whole) : "v"(p_r));
    uint32_t base;                                             // draw * 2^(16-b) + k and the half grain
    if constexpr (HIGH)
        asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(base) : "v"(rw), "s"(1u << (16 - BITS)), "v"(__float_as_uint(c.z)));
    else
        asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(base) : "v"(rw), "s"(1u << (16 - BITS)), "v"(__float_as_uint(c.z)));
    return __builtin_elementwise_add_sat(whole, base);
}

// The packed codes of one lane's whole group, regular codebook.
template <int BITS>
__device__ __forceinline__ uint32_t encode_regular(const float (&x)[8], const uint32_t (&rw)[4], const float (&pv)[3],
                                                   const CellLds& tab)
{
    uint32_t word = 0;
#pragma unroll
    for (int j = 7; j >= 0; --j) {
        const uint32_t t = (j & 1) ? code_on_top<BITS, true>(x[j], rw[j >> 1], pv, tab)
                                   : code_on_top<BITS, false>(x[j], rw[j >> 1], pv, tab);
        word = __builtin_amdgcn_alignbit(word, t, 32 - BITS);
    }
    return word;
}

// The levels the search compares |x| with first (wave-uniform: scalar loads).
template <int BITS>
__device__ __forceinline__ void load_pivots(const tq_params_t* P, float (&pv)[3])
{
    if constexpr (BITS == 2) { pv[0] = P->level[2]; pv[1] = pv[2] = 0.0f; }
    else { pv[0] = P->level[4]; pv[1] = P->level[5]; pv[2] = P->level[6]; }
}

// `room` = bytes of the payload from `out` on.  A payload is a multiple of 16 bytes, so a
// group's 2 or 4 bytes are either wholly inside or wholly outside; its 3 bytes at b = 3 can
// straddle the end (the last, ragged group of a short tensor), hence the per-byte test.
template <int BITS>
__device__ __forceinline__ void store_codes(uint8_t* out, uint32_t word, uint64_t room = 4)
{
    if constexpr (BITS == 4) {
        *reinterpret_cast<uint32_t*>(out) = word;
    } else if constexpr (BITS == 2) {
        *reinterpret_cast<uint16_t*>(out) = (uint16_t)word;
    } else {
        out[0] = (uint8_t)word;
        if (room > 1) out[1] = (uint8_t)(word >> 8);
        if (room > 2) out[2] = (uint8_t)(word >> 16);
    }
}

// The codes of a wavefront whose lanes all own whole groups inside the payload (`out` = the lane's place).
// PAST_CACHES: non-temporal stores, for payloads that would not be found in a cache by whoever
// reads them: they leave the caches to the gradient and go out as they come.  8 x 124 M fp32 uniform at
// b = 2 / 3 / 4: 671 -> 641, 689 -> 672, 700 -> 677 us; with a payload that the decode finds in the
// memory-side cache the hint costs the decode more than it gives here (4 x 11.2 M at b = 3: 1 us
// against 3.6), so the host turns it on with the whole-line loads (compress_cached).
// b = 3: the 12 bytes of four lanes leave as three 4-byte stores of the first three (bytes sent past
// the caches one by one cost 1.6 times the whole launch); through the caches single bytes are as good.
template <int BITS, bool PAST_CACHES>
__device__ __forceinline__ void store_codes_wave(uint8_t* out, uint32_t word)
{
    if constexpr (!PAST_CACHES) {
        store_codes<BITS>(out, word);
    } else if constexpr (BITS == 4) {
        __builtin_nontemporal_store(word, reinterpret_cast<uint32_t*>(out));
    } else if constexpr (BITS == 2) {
        __builtin_nontemporal_store((uint16_t)word, reinterpret_cast<uint16_t*>(out));
    } else {
        const uint32_t r = threadIdx.x & 3u;                   // the lane's 3 bytes start at byte 3 r of the quad's 12
        const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0xF9, 0xf, 0xf, false);   // from lane r + 1
        const uint32_t dword = (word >> (8u * r)) | (next << (24u - 8u * r));
        if (r < 3u) __builtin_nontemporal_store(dword, reinterpret_cast<uint32_t*>(out + r));
    }
}

// Tiles per workgroup (256 threads, every thread one group in every tile, all reads requested
// first).  The two codebook families want different numbers, measured on MI355X:
//   * the uniform path runs at the speed of its memory traffic when the running wavefronts together
//     cover a small window of the gradient: on 8 x 124 M fp32, 670 us (641 with the payload stored past the
//     caches) with one tile per workgroup against 745 us with two, whether the two are requested
//     together, one after the other, adjacent or far apart;
//   * the level-table path sets up its codebook before the first read, once per workgroup, and needs reads in
//     flight while it computes: with one / two / four tiles 16 x 25.6 M fp32 at b = 3 take 370 / 300 / 325 us, with two /
//     four / six 4 x 10^9 bf16 at b = 2 (a bf16 tile is half the bytes) 1970 / 1775 / 1819.
// The family is a property of the parameter records, which live on the device, so the host
// chooses by the family the caller names (tq_compress's `grid`); the kernel itself reads every
// bucket's record and computes what the record says, whatever shape it was launched in.
constexpr int compress_tiles(int dtype, bool table_tiles)
{
    return dtype == TQ_F32 ? (table_tiles ? 2 : 1) : (table_tiles ? 4 : 2);
}

// The same for segments, whose family the caller does not name: the level table's numbers.  One step of
// 8 x 124 M with 68 layers, one (two at bf16) / two (four) / three / four (six) tiles: fp32 b = 2 tables 1605 / 1555 /
// 1566 / 1577 us, b = 3 1866 / 1688 / 1671 / 1663, bf16 b = 2 1088 / 1013 / 1035 / 1003; fp32 b = 2 uniform
// 1497 / 1529 / 1600 / 1586.
constexpr int segment_tiles(int dtype) { return compress_tiles(dtype, true); }

// What a workgroup knows of its record.
struct Codebook {
    float alpha, inv_step;
    bool nonuniform, regular;                                  // the same in the whole workgroup
    float pv[3];
};

// Reads the record and, for a level table, fills `cells` (one barrier).  The codebook is read before the record's
// family is known: the launch expects a level table.
template <int BITS>
__device__ __forceinline__ Codebook set_up_codebook(const tq_params_t* P, CellLds& cells, uint32_t lane)
{
    Codebook cb;
    CellReads reads = {};
    if (lane < 64) reads = read_cells<BITS>(P, lane);
    load_pivots<BITS>(P, cb.pv);
    cb.alpha = P->alpha;
    cb.inv_step = P->inv_w[0];
    cb.nonuniform = P->grid != TQ_GRID_UNIFORM;
    cb.regular = true;
    if (cb.nonuniform) {
        if (lane < 64) fill_cells<BITS>(cells, reads, cb.alpha, lane);
        // compared from vector registers: with a scalar operand the subtraction runs at 36 T/s, without at 59
        asm volatile("" : "+v"(cb.pv[0]), "+v"(cb.pv[1]), "+v"(cb.pv[2]));
        __syncthreads();
        cb.regular = __builtin_amdgcn_readfirstlane((int)cells.regular) != 0;
    }
    return cb;
}

// The draws of one tile whose first element is ebase: one Philox call per lane; the high counter word
// stays scalar unless the low word wraps inside the tile.
template <uint32_t LANES = kBlock>
__device__ __forceinline__ void draw_tile(uint64_t ebase, uint32_t lane, uint32_t worker, uint32_t step,
                                          uint32_t seed_lo, uint32_t seed_hi, uint32_t (&rw)[4])
{
    const uint64_t qb = ebase >> 3;                            // first group of the tile (uniform)
    const uint32_t qb_lo = (uint32_t)qb, qb_hi = (uint32_t)(qb >> 32);
    const uint32_t q_lo = qb_lo + lane;
    if (qb_lo <= 0xFFFFFFFFu - LANES) philox4x32_10(q_lo, qb_hi, worker, step, seed_lo, seed_hi, rw);
    else philox4x32_10(q_lo, qb_hi + (q_lo < qb_lo ? 1u : 0u), worker, step, seed_lo, seed_hi, rw);
}

template <int BITS>
__device__ __forceinline__ uint32_t encode_uniform(const float (&x)[8], const uint32_t (&rw)[4], const Codebook& cb)
{
    uint32_t word = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t r = (j & 1) ? (rw[j >> 1] >> 16) : (rw[j >> 1] & 0xFFFFu);
        word |= quantize_uniform<BITS>(x[j], (float)r, cb.alpha, cb.inv_step) << (j * BITS);
    }
    return word;
}

// The packed codes of a lane's whole group, uniform or regular codebook.
template <int BITS>
__device__ __forceinline__ uint32_t encode_whole(const float (&x)[8], const uint32_t (&rw)[4], const Codebook& cb,
                                                 const CellLds& cells)
{
    return cb.nonuniform ? encode_regular<BITS>(x, rw, cb.pv, cells) : encode_uniform<BITS>(x, rw, cb);
}

// The general path's table: 16 scalar levels and, behind one barrier, the entries in LDS.
template <int BITS>
__device__ __forceinline__ void set_up_levels(const tq_params_t* P, LevelLds& tab, float (&lv)[16])
{
    fill_level_lds(tab, P, (1u << BITS) - 1u);
#pragma unroll
    for (int j = 0; j < 16; ++j) lv[j] = P->level[j];           // wave-uniform: scalar loads
    __syncthreads();
}

// Whether a level table encodes every value as it encodes the truncated one, so that Eq. (1) need not be written out
// (one of 13 to 18 instructions per element: 16 x 25.6 M fp32 at b = 4 351 -> 344 us).  Below -alpha the cell is the
// first one, not empty, and p_r < 0; beyond +alpha it is the last one and p_r at least the largest u, 1 - 2^-17, or 0
// if it is empty (Inf times a zero reciprocal is NaN, and u <= NaN is false).
template <int BITS>
__device__ __forceinline__ bool truncates_itself(const tq_params_t* P, float alpha)
{
    constexpr int S = (1 << BITS) - 1;
    const float first = P->level[0], last = P->level[S], inv = P->inv_w[S - 1];
    const bool full = (last - P->level[S - 1]) * inv >= 1.0f - 7.62939453125e-06f;
    return P->level[1] > first && first >= -alpha && P->inv_w[0] >= 0.0f && last <= alpha && (full || inv == 0.0f);
}

__device__ __forceinline__ Codebook read_codebook(const tq_params_t* P)
{
    Codebook cb;
    cb.alpha = P->alpha;
    cb.inv_step = P->inv_w[0];
    cb.nonuniform = P->grid != TQ_GRID_UNIFORM;                // uniform over the workgroup
    cb.regular = false;
    cb.pv[0] = cb.pv[1] = cb.pv[2] = 0.0f;
    return cb;
}

// A lane's whole group on the general path.
template <int BITS, bool CLAMP>
__device__ __forceinline__ uint32_t encode_general(const float (&x)[8], const uint32_t (&rw)[4], const Codebook& cb,
                                                   const float (&lv)[16], const LevelLds& tab)
{
    return cb.nonuniform ? encode_group<BITS, TQ_GRID_NONUNIFORM, false, CLAMP>(x, rw, 8, cb.alpha, cb.inv_step, lv, tab)
                         : encode_group<BITS, TQ_GRID_UNIFORM, false>(x, rw, 8, cb.alpha, cb.inv_step, lv, tab);
}

// N tiles from `base` on in which every lane owns a whole group: all reads first, the draws under them (requesting the
// reads even earlier, before the codebook is set up, was slower: 708 us against 668 on 8 x 124 M fp32).
// THROUGH: bf16 lines are read through the caches (reads_through).
template <int DTYPE, int BITS, bool CACHED, int N, bool THROUGH = false, int TILE = kTile, typename Draw, typename Encode>
__device__ __forceinline__ void encode_tiles(const void* g, uint8_t* payload, uint64_t base, uint32_t lane, Draw draw, Encode encode)
{
    constexpr bool kLines = DTYPE == TQ_F32 && !CACHED;
    float x[N][8];
    uint32_t rw[N][4];
#pragma unroll
    for (int t = 0; t < N; ++t) {
        const uint64_t tile = base + (uint64_t)t * TILE;
        if constexpr (kLines) load_groups_wave(g, tile + (lane & ~63u) * kGroup, lane & 63u, x[t]);
        else load_group<DTYPE, !THROUGH>(g, tile + (uint64_t)lane * kGroup, x[t]);
    }
#pragma unroll
    for (int t = 0; t < N; ++t) {
        draw(base + (uint64_t)t * TILE, rw[t]);
        asm volatile("" : "+v"(rw[t][0]));                     // computed here, under the loads
    }
#pragma unroll
    for (int t = 0; t < N; ++t) {
        if constexpr (kLines) swap_pieces(x[t]);
        replace_nan(x[t]);
        const uint32_t word = encode(x[t], rw[t]);
        store_codes_wave<BITS, !CACHED>(payload + (((base + (uint64_t)t * TILE) >> 3) + lane) * (uint64_t)BITS, word);
    }
}

// A workgroup's T whole tiles on the general path.
template <int DTYPE, int BITS, bool CACHED, int T, bool MIRROR, typename Draw>
__device__ __forceinline__ void encode_tiles_general(const void* g, uint8_t* payload, uint64_t base, uint32_t lane, Draw draw,
                                                     const tq_params_t* P, const Codebook& cb, const float (&lv)[16], const LevelLds& tab)
{
    auto clamped = [&](const float (&x)[8], const uint32_t (&rw)[4]) { return encode_general<BITS, true>(x, rw, cb, lv, tab); };
    auto plain = [&](const float (&x)[8], const uint32_t (&rw)[4]) { return encode_general<BITS, false>(x, rw, cb, lv, tab); };
    if constexpr (MIRROR) {                                    // two tiles at a time: no more registers than the mirrored path
        constexpr int N = T < 2 ? T : 2;
#pragma unroll 1
        for (int t = 0; t < T; t += N) encode_tiles<DTYPE, BITS, CACHED, N>(g, payload, base + (uint64_t)t * kTile, lane, draw, clamped);
    } else {
        if (T == compress_tiles(DTYPE, true) && cb.nonuniform && truncates_itself<BITS>(P, cb.alpha))
            encode_tiles<DTYPE, BITS, CACHED, T>(g, payload, base, lane, draw, plain);
        else
            encode_tiles<DTYPE, BITS, CACHED, T>(g, payload, base, lane, draw, clamped);
    }
}

// MIRROR: level tables are checked for the mirrored path and take it if they are regular; else every record is
// encoded on the general one.
template <int DTYPE, int BITS, bool CACHED, int T, bool MIRROR, bool THROUGH>
__global__ __launch_bounds__(kBlock, !MIRROR && T <= 2 && !(DTYPE == TQ_BF16 && BITS == 4) ? 8 : 1) void tq_compress_kernel(
    const PtrTable g_tab, uint64_t d, uint64_t d_pad, uint64_t bucket_elems,
    uint32_t groups_per_bucket, const PtrTable params_tab, uint32_t seed_lo,
    uint32_t seed_hi, uint32_t first_worker, uint32_t step, const MutPtrTable payload_tab,
    uint64_t payload_bytes)
{
    const uint32_t blk = linear_block();
    const uint32_t bucket = blk / groups_per_bucket;
    const uint32_t grp = blk - bucket * groups_per_bucket;
    const uint64_t bstart = (uint64_t)bucket * bucket_elems;
    const uint64_t bend = bstart + bucket_elems < d_pad ? bstart + bucket_elems : d_pad;
    const uint64_t gbase = bstart + (uint64_t)grp * T * kTile;            // first element of the workgroup
    if (gbase >= bend) return;                                 // idle workgroup of a short last bucket
    // blockIdx.y = tensor of the batch; its worker id keys the random draws
    const void* __restrict__ g = g_tab.p[blockIdx.y];
    uint8_t* __restrict__ payload = static_cast<uint8_t*>(payload_tab.p[blockIdx.y]);
    const uint32_t worker = first_worker + blockIdx.y;
    const tq_params_t* P = static_cast<const tq_params_t*>(params_tab.p[blockIdx.y]) + bucket;
    const uint32_t lane = threadIdx.x;                         // this thread's group within a tile
    auto draw = [&](uint64_t ebase, uint32_t (&rw)[4]) { draw_tile(ebase, lane, worker, step, seed_lo, seed_hi, rw); };

    const uint64_t lim = bend < d ? bend : d;
    const bool whole = gbase + (uint64_t)T * kTile <= lim;

    Codebook cb;
    if constexpr (MIRROR) {
        __shared__ CellLds cells;
        cb = set_up_codebook<BITS>(P, cells, lane);
        if (cb.regular && whole) {
            encode_tiles<DTYPE, BITS, CACHED, T>(g, payload, gbase, lane, draw, [&](const float (&x)[8], const uint32_t (&rw)[4]) {
                return encode_whole<BITS>(x, rw, cb, cells);
            });
            return;
        }
    } else {
        cb = read_codebook(P);
        // bf16: the uniform codebook apart from the tables' code, which costs it 1 us of 14 on 25.6 M at b = 3 and 4 (fp32
        // the other way round: tables at b = 2 20.9 us with it, 21.9 without)
        if (DTYPE == TQ_BF16 && whole && !cb.nonuniform) {
            encode_tiles<DTYPE, BITS, CACHED, T, THROUGH>(g, payload, gbase, lane, draw, [&](const float (&x)[8], const uint32_t (&rw)[4]) {
                return encode_uniform<BITS>(x, rw, cb);
            });
            return;
        }
    }
    __shared__ LevelLds tab;
    float lv[16];
    if (cb.nonuniform) set_up_levels<BITS>(P, tab, lv);
    if (whole) {
        encode_tiles_general<DTYPE, BITS, CACHED, T, MIRROR>(g, payload, gbase, lane, draw, P, cb, lv, tab);
        return;
    }

    // the last workgroup of a bucket: tile by tile, lanes past the end idle, the tensor's
    // ragged last group element by element
    for (int t = 0; t < T; ++t) {
        const uint64_t ebase = gbase + (uint64_t)t * kTile;
        const uint64_t e0 = ebase + (uint64_t)lane * kGroup;
        const uint64_t byte_off = ((ebase >> 3) + lane) * (uint64_t)BITS;
        if (e0 >= bend || byte_off >= payload_bytes) continue;
        uint32_t word = 0;                                     // groups wholly in the padding encode as 0
        if (e0 + kGroup <= d) {
            float x[8];
            load_group<DTYPE, false>(g, e0, x);
            uint32_t rw[4];
            draw(ebase, rw);
            replace_nan(x);
            word = encode_general<BITS, true>(x, rw, cb, lv, tab);
        } else if (e0 < d) {
            const int n_valid = (int)(d - e0);
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = (j < n_valid) ? load_one<DTYPE>(g, e0 + j) : 0.0f;
            uint32_t rw[4];
            draw(ebase, rw);
            replace_nan(x);
            word = cb.nonuniform ? encode_group<BITS, TQ_GRID_NONUNIFORM, true>(x, rw, n_valid, cb.alpha, cb.inv_step, lv, tab)
                                 : encode_group<BITS, TQ_GRID_UNIFORM, true>(x, rw, n_valid, cb.alpha, cb.inv_step, lv, tab);
        }
        store_codes<BITS>(payload + byte_off, word, payload_bytes - byte_off);
    }
}

// ---- bf16 and a level table: the encoding of every value, looked up ---------------------------
//
// A bf16 gradient has few different values.  From alpha down to 2^-32 alpha there are 4096 magnitudes; all larger ones encode
// like alpha, all smaller ones like 0 (checked, below).  A workgroup works out the encoding of each of them, of either sign,
// once, by the general path's own arithmetic, and keeps it in LDS:
//   entry = k 2^(32-b) + f 2^(16-b),   f = the number of the 65536 draws that take the upper end of cell k,
// so that entry + draw 2^(16-b) has the code in its top b bits: draw r takes the upper end iff r >= 65536 - f.  An element
// then costs 5.5 vector instructions beside its draw's 5 -- two elements' magnitudes are clamped at a time -- where the mirrored
// path takes 11 (b = 2) or 15 (b = 3), and any table will do, regular or not.
//   f: u(r) = 1 - (r + 1/2) / 2^16 <= p_r  <=>  r >= 65535.5 - 2^16 p_r, so f = floor(2^16 p_r + 1/2), within 0 .. 2^16 (0 where
//   p_r is no number); in fp64 that is exact.
//   Magnitudes below the smallest of the 4096 encode like it and like 0 if those two lie in one cell with the same f, the
//   difference, the product and f being monotone inside a cell.  If they do not (always where the cell at 0 is narrower than
//   2^-17 alpha, seldom where it is wide), the workgroup encodes on the general path, a tile at a time (two take more than 64
//   registers), which with so few workgroups is slower than tq_compress_kernel, us: 4 x 250 M at b = 2 460 / 531, b = 3 554 / 653,
//   b = 4 711 / 711, 1 x 70 M at b = 3 43.6 / 67, b = 4 54 / 71, 1 x 34 M 30.5 / 52.9.  So do uniform records that the caller took
//   for tables: 399 / 445, 425 / 464, 397 / 471, 34.5 / 47.5, 33.4 / 45.6, 18.7 / 33.8.  (The next tile requested ahead: narrow cells
//   546 -> 537, 1 x 70 M 67 -> 62 and 71 -> 66, but uniform records at b = 4 471 -> 477: not done.)
// What bounds it: instruction issue (12.6 vector instructions per element in all; 18.6 on the mirrored path at b = 2) and, past it, memory:
// a loop that only reads and writes in this pattern takes 1580 to 1720 us for 4 x 10^9 elements, one-shot workgroups 1400 to 1480
// (which the time to fill the entries rules out).  A wavefront takes two groups at a time: with one, the chain of the draws is
// exposed (2200 us).  Workgroups of 1024 threads 1750 to 1770 us, of 512 1690 to 1780, of 256 (fewer wavefronts: the entries fill the LDS) 1726.
// Ranges taken tile by tile in turn by 64 to 1024 workgroups 1670 to 1860.  Rules and times by size: look_tiles.
constexpr int kLookBlock = 512;                                // threads; a tile is one group of each
constexpr int kLookTile = kLookBlock * kGroup;
constexpr uint32_t kLookMagnitudes = 4096;
typedef uint16_t ushort2_native __attribute__((ext_vector_type(2)));

struct LookLds {
    uint32_t entry[2 * kLookMagnitudes];                       // 2 * (magnitude - lowest) + sign
};

// The entry of one value, and the cell it lies in.
template <int BITS>
__device__ __forceinline__ uint32_t look_entry(float x, float alpha, const float (&lv)[16], const LevelLds& tab, uint32_t& cell)
{
    const float xc = __builtin_amdgcn_fmed3f(x, -alpha, alpha);          // Eq. (1)
    cell = cell_offset<BITS>(xc, lv, tab);
    const float2 c = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(tab.e) + cell);
    const float p_r = (xc - c.x) * c.y;                        // (g - l_k) / |Delta_k| of Eq. (2)
    double f = __builtin_floor((double)p_r * 65536.0 + 0.5);
    f = f > 0.0 ? (f < 65536.0 ? f : 65536.0) : 0.0;
    return ((cell >> 4) << (32 - BITS)) + ((uint32_t)f << (16 - BITS));
}

// The entries of a lane's 8 elements (two to a word).  lowest and span: twice the smallest magnitude that has
// an entry, twice the number of those above it, in both halves.
__device__ __forceinline__ void look_up(const uint32_t (&w)[4], uint32_t lowest, uint32_t span, const LookLds& L, uint32_t (&entry)[8])
{
    // twice the magnitudes; NaN -> +0 (it counts as nothing), tested on all of a wavefront's values at once
    ushort2_native twice[4], sign[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const ushort2_native v = __builtin_bit_cast(ushort2_native, w[i]);
        twice[i] = v << 1;
        sign[i] = v >> 15;
    }
    const ushort2_native inf = {0xFF00u, 0xFF00u};
    const ushort2_native top = __builtin_elementwise_max(__builtin_elementwise_max(twice[0], twice[1]), __builtin_elementwise_max(twice[2], twice[3]));
    if (__builtin_amdgcn_ballot_w64(__builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(top, inf)) != 0u) != 0ull) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool nan = twice[i][h] > 0xFF00u;
                twice[i][h] = nan ? (uint16_t)0u : twice[i][h];
                sign[i][h] = nan ? (uint16_t)0u : sign[i][h];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        ushort2_native m = __builtin_elementwise_sub_sat(twice[i], __builtin_bit_cast(ushort2_native, lowest));
        m = __builtin_elementwise_min(m, __builtin_bit_cast(ushort2_native, span));
        uint32_t at = __builtin_bit_cast(uint32_t, (ushort2_native)(m | sign[i]));
        asm("" : "+v"(at));                                    // each half is then taken and scaled in one instruction
        entry[2 * i] = L.entry[at & 0xFFFFu];
        entry[2 * i + 1] = L.entry[at >> 16];
    }
}

// The packed codes, from the entries and the draws.
template <int BITS>
__device__ __forceinline__ uint32_t pack_looked_up(const uint32_t (&entry)[8], const uint32_t (&rw)[4])
{
    uint32_t sum[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(sum[2 * i]) : "v"(rw[i]), "s"(1u << (16 - BITS)), "v"(entry[2 * i]));
        asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(sum[2 * i + 1]) : "v"(rw[i]), "s"(1u << (16 - BITS)), "v"(entry[2 * i + 1]));
    }
    uint32_t word = 0;
#pragma unroll
    for (int j = 7; j >= 0; --j) word = __builtin_amdgcn_alignbit(word, sum[j], 32 - BITS);
    return word;
}

// `tiles` tiles of one bucket per workgroup, two at a time.
template <int BITS, bool CACHED>
__global__ __launch_bounds__(kLookBlock, 8) void tq_compress_lookup_kernel(
    const PtrTable g_tab, uint64_t d, uint64_t d_pad, uint64_t bucket_elems, uint32_t groups_per_bucket, uint32_t tiles,
    const PtrTable params_tab, uint32_t seed_lo, uint32_t seed_hi, uint32_t first_worker, uint32_t step, const MutPtrTable payload_tab,
    uint64_t payload_bytes)
{
    const uint32_t blk = linear_block();
    const uint32_t bucket = blk / groups_per_bucket;
    const uint32_t grp = blk - bucket * groups_per_bucket;
    const uint64_t bstart = (uint64_t)bucket * bucket_elems;
    const uint64_t bend = bstart + bucket_elems < d_pad ? bstart + bucket_elems : d_pad;
    const uint64_t gbase = bstart + (uint64_t)grp * tiles * kLookTile;    // first element of the workgroup
    if (gbase >= bend) return;                                 // idle workgroup of a short last bucket
    const uint16_t* __restrict__ g = static_cast<const uint16_t*>(g_tab.p[blockIdx.y]);
    uint8_t* __restrict__ payload = static_cast<uint8_t*>(payload_tab.p[blockIdx.y]);
    const uint32_t worker = first_worker + blockIdx.y;
    const tq_params_t* P = static_cast<const tq_params_t*>(params_tab.p[blockIdx.y]) + bucket;
    const uint32_t lane = threadIdx.x;
    const uint64_t whole_end = bend < d ? bend : d;            // the groups before it are whole

    __shared__ LookLds L;
    __shared__ LevelLds tab;
    const Codebook cb = read_codebook(P);
    float lv[16];
    uint32_t lowest = 0, span = 0;
    bool looked_up = false;
    if (cb.nonuniform) {
        set_up_levels<BITS>(P, tab, lv);
        // the smallest magnitude that is not below alpha, and 4095 before it
        const uint32_t alpha_bits = __float_as_uint(cb.alpha);
        const uint32_t high = alpha_bits >= 0x7F800000u ? 0x7F80u : (alpha_bits + 0xFFFFu) >> 16;
        const uint32_t low = high > kLookMagnitudes - 1u ? high - (kLookMagnitudes - 1u) : 0u;
        {   // every wavefront by itself: lanes 0 and 1 look at the smallest magnitude, 2 and 3 at 0
            uint32_t cell;
            const uint32_t sign = (lane & 1u) << 31;
            const uint32_t entry = look_entry<BITS>(__uint_as_float((lane & 2u ? 0u : low << 16) | sign), cb.alpha, lv, tab, cell);
            const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)entry, 0x4E, 0xf, 0xf, true);   // lane ^ 2
            const uint32_t other_cell = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)cell, 0x4E, 0xf, 0xf, true);
            looked_up = (__builtin_amdgcn_ballot_w64(entry == other && cell == other_cell) & 3ull) == 3ull;
        }
        if (looked_up) {                                       // the same in every wavefront
#pragma unroll 1
            for (uint32_t e = lane; e < 2u * kLookMagnitudes; e += kLookBlock) {
                uint32_t cell;
                const uint32_t bits_e = ((low + (e >> 1)) << 16) | (e & 1u) << 31;
                L.entry[e] = look_entry<BITS>(__uint_as_float(bits_e), cb.alpha, lv, tab, cell);
            }
            __syncthreads();
        }
        lowest = 2u * low * 0x10001u;
        span = 2u * (high - low) * 0x10001u;
    }
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    constexpr int N = 2;
    uint64_t base = gbase;
    uint32_t left = tiles;
    if (looked_up) {
        // N tiles at a time, the next ones requested before these are stored: a wavefront's loads and stores complete in order,
        // and a request behind a store would wait for it
        const uint64_t fit = whole_end > gbase ? (whole_end - gbase) / kLookTile : 0;     // whole tiles
        uint32_t turns = (uint32_t)(fit < tiles ? fit : tiles) / N;
        auto request = [&](u4 (&v)[N], uint64_t at) {
#pragma unroll
            for (int t = 0; t < N; ++t)
                v[t] = __builtin_nontemporal_load(reinterpret_cast<const u4*>(g + (at + t * (uint64_t)kLookTile)) + lane);
        };
        auto turn = [&](const u4 (&v)[N], u4 (&next)[N], bool more) {
            uint32_t rw[N][4];
            request(next, more ? base + N * (uint64_t)kLookTile : base);    // no branch: where its paths joined, all loads would be waited for
            __builtin_amdgcn_sched_barrier(0);
            uint32_t entry[N][8];                              // on their way from LDS while the draws are computed
#pragma unroll
            for (int t = 0; t < N; ++t) {
                const uint32_t w[4] = {v[t].x, v[t].y, v[t].z, v[t].w};
                look_up(w, lowest, span, L, entry[t]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < N; ++t) draw_tile<kLookBlock>(base + t * (uint64_t)kLookTile, lane, worker, step, seed_lo, seed_hi, rw[t]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < N; ++t) {
                const uint32_t word = pack_looked_up<BITS>(entry[t], rw[t]);
                store_codes_wave<BITS, !CACHED>(payload + ((base + t * (uint64_t)kLookTile) >> 3) * BITS + lane * BITS, word);
            }
            base += N * (uint64_t)kLookTile;
        };
        u4 a[N], b[N];
        if (turns > 0) request(a, base);
        left -= turns * N;
#pragma unroll 1
        for (; turns > 0; turns -= 2) {
            turn(a, b, turns > 1);
            if (turns == 1) break;
            turn(b, a, turns > 2);
        }
    }
    if (!looked_up) {
        auto draw = [&](uint64_t ebase, uint32_t (&rw)[4]) { draw_tile<kLookBlock>(ebase, lane, worker, step, seed_lo, seed_hi, rw); };
#pragma unroll 1
        for (; left > 0 && base + kLookTile <= whole_end; base += kLookTile, --left) {
            encode_tiles<TQ_BF16, BITS, CACHED, 1, false, kLookTile>(g, payload, base, lane, draw, [&](const float (&x)[8], const uint32_t (&rw)[4]) {
                return encode_general<BITS, true>(x, rw, cb, lv, tab);
            });
        }
    }
    // the tiles that are left: lanes past the end idle, the tensor's ragged last group element by element
#pragma unroll 1
    for (; left > 0 && base < bend; base += kLookTile, --left) {
        const uint64_t e0 = base + (uint64_t)lane * kGroup;
        const uint64_t byte_off = ((base >> 3) + lane) * (uint64_t)BITS;
        if (e0 >= bend || byte_off >= payload_bytes) continue;
        const int n_valid = e0 >= d ? 0 : (d - e0 < kGroup ? (int)(d - e0) : kGroup);
        uint32_t w[4], rw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = 0;
        if (n_valid == kGroup) {
            const u4 v = *reinterpret_cast<const u4*>(g + e0);
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 7; ++j)
                if (j < n_valid) w[j >> 1] |= (uint32_t)g[e0 + j] << (16 * (j & 1));
        }
        draw_tile<kLookBlock>(base, lane, worker, step, seed_lo, seed_hi, rw);
        uint32_t word;
        if (looked_up) {
            uint32_t entry[8];
            look_up(w, lowest, span, L, entry);
            word = pack_looked_up<BITS>(entry, rw);
        } else {
            float x[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) { x[2 * i] = __uint_as_float(w[i] << 16); x[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u); }
            replace_nan(x);
            word = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float r = (float)((j & 1) ? rw[j >> 1] >> 16 : rw[j >> 1] & 0xFFFFu);
                const uint32_t code = cb.nonuniform ? quantize<BITS, TQ_GRID_NONUNIFORM>(x[j], r, cb.alpha, cb.inv_step, lv, tab)
                                                    : quantize_uniform<BITS>(x[j], r, cb.alpha, cb.inv_step);
                word |= code << (j * BITS);
                __builtin_amdgcn_sched_barrier(0);             // one after the other, in few registers
            }
        }
        if (n_valid < kGroup) word &= (1u << (n_valid * BITS)) - 1u;      // the others encode as 0
        store_codes<BITS>(payload + byte_off, word, payload_bytes - byte_off);
    }
}

// Wavefronts per SIMD of the segments' kernel: held to the registers of one more where that needs no scratch memory
// (8 x 124 M fp32 with 68 layers at b = 2, one step: 1532 -> 1506 us).
constexpr int segment_waves(int dtype, int bits, int tiles)
{
    if (tiles == 1) return 6;
    return bits == 2 ? (dtype == TQ_F32 ? 7 : 6) : (dtype == TQ_F32 ? 6 : 5);
}

// tq_compress_segments: the same client step with one (alpha, codebook) per variable-size
// segment of the flat gradient (Sec. V: the layers of a network are quantized independently).
// T tiles per workgroup wherever the segments fall.  Large layers are the rule: nearly every workgroup's
// range lies inside one segment and is encoded like a bucket's.  The others take their tiles one by
// one, and the segments that overlap a tile one after the other (a lane's group of 8 lies in exactly
// one, the offsets being multiples of 128).  The last segment also owns the
// padding up to a multiple of 128 elements.  No access depends on the table being well-formed:
// the segment index stays inside [0, nseg) and every element access is bounded by d.
template <int DTYPE, int BITS, bool CACHED, int T, bool MIRROR>
__global__ __launch_bounds__(kBlock, segment_waves(DTYPE, BITS, T)) void tq_compress_segments_kernel(
    const PtrTable g_tab, uint64_t d, uint64_t d_pad, const uint64_t* __restrict__ seg_off, uint32_t nseg,
    const SegHints hints, const PtrTable params_tab, uint32_t seed_lo, uint32_t seed_hi, uint32_t first_worker, uint32_t step,
    const MutPtrTable payload_tab, uint64_t payload_bytes)
{
    const uint64_t gbase = (uint64_t)linear_block() * T * kTile;
    if (gbase >= d_pad) return;                                // padding of a folded grid
    // blockIdx.y = tensor of the batch; its worker id keys the random draws
    const void* __restrict__ g = g_tab.p[blockIdx.y];
    const tq_params_t* __restrict__ params = static_cast<const tq_params_t*>(params_tab.p[blockIdx.y]);
    uint8_t* __restrict__ payload = static_cast<uint8_t*>(payload_tab.p[blockIdx.y]);
    const uint32_t worker = first_worker + blockIdx.y;
    const uint32_t lane = threadIdx.x;
    __shared__ LevelLds tab;
    auto draw = [&](uint64_t ebase, uint32_t (&rw)[4]) { draw_tile(ebase, lane, worker, step, seed_lo, seed_hi, rw); };

    // One tile: the values are requested and the draws computed before the segment is looked up, a chain of
    // dependent scalar loads (they depend on the lane's position alone).
    float x[8];
    uint32_t rw[4];
    auto request = [&](uint64_t ebase) {
        const uint64_t e0 = ebase + (uint64_t)lane * kGroup;
        if (e0 + kGroup <= d) {
            load_group<DTYPE, false>(g, e0, x);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = e0 + j < d ? load_one<DTYPE>(g, e0 + j) : 0.0f;
        }
        draw(ebase, rw);
        asm volatile("" : "+v"(rw[0]));                        // computed here, under the loads
    };
    if constexpr (T == 1) request(gbase);

    const uint32_t s0 = find_segment(seg_off, nseg, gbase < d ? gbase : d - 1, hints);
    // The test uses the very segment ends the loop below uses, so both ways write the same bytes.
    uint64_t seg_lo = seg_off[s0];
    uint64_t seg_hi = s0 + 1 < nseg ? seg_off[s0 + 1] : d_pad;
    {
        const uint64_t gend = gbase + (uint64_t)T * kTile;
        if (seg_lo <= gbase && seg_hi >= gend && gend <= d) {  // whole groups, and their codes lie inside the payload
            const tq_params_t* P = params + s0;
            Codebook cb;
            if constexpr (MIRROR) {
                __shared__ CellLds cells;
                cb = set_up_codebook<BITS>(P, cells, lane);
                if (cb.regular) {
                    encode_tiles<DTYPE, BITS, CACHED, T>(g, payload, gbase, lane, draw, [&](const float (&v)[8], const uint32_t (&r)[4]) {
                        return encode_whole<BITS>(v, r, cb, cells);
                    });
                    return;
                }
            } else {
                cb = read_codebook(P);
            }
            float lv[16];
            if (cb.nonuniform) set_up_levels<BITS>(P, tab, lv);
            if constexpr (T == 1) {
                replace_nan(x);
                store_codes_wave<BITS, !CACHED>(payload + ((gbase >> 3) + lane) * (uint64_t)BITS, encode_general<BITS, true>(x, rw, cb, lv, tab));
            } else {
                encode_tiles_general<DTYPE, BITS, CACHED, T, MIRROR>(g, payload, gbase, lane, draw, P, cb, lv, tab);
            }
            return;
        }
    }
    bool table_used = false;                                   // the same for the whole workgroup
    for (int t = 0; t < T; ++t) {
        const uint64_t ebase = gbase + (uint64_t)t * kTile;
        if (ebase >= d_pad) break;
        // positions inside the tile are 32-bit offsets from its first element (which is the same for
        // the whole workgroup): the tensor's end, the payload's end and the segments' ends as such
        const uint32_t rel = lane * kGroup;                                              // this lane's group
        const uint32_t tile_len = (uint32_t)(ebase + kTile < d_pad ? kTile : d_pad - ebase);   // multiple of 128
        const uint32_t d_rel = ebase < d ? (uint32_t)(d - ebase < (uint64_t)kTile ? d - ebase : kTile) : 0u;
        const uint64_t tile_byte = (ebase >> 3) * (uint64_t)BITS;                         // payload offset of the tile
        const uint32_t pay_rel =                                                          // payload bytes from there on, capped
            tile_byte < payload_bytes ? (uint32_t)(payload_bytes - tile_byte < (uint64_t)kTile ? payload_bytes - tile_byte : kTile) : 0u;
        const uint32_t byte_rel = lane * (uint32_t)BITS;
        const int n_valid = rel >= d_rel ? 0 : (d_rel - rel >= (uint32_t)kGroup ? kGroup : (int)(d_rel - rel));
        if constexpr (T > 1) request(ebase);
        uint32_t s = s0;
        if (t > 0) {
            s = find_segment(seg_off, nseg, ebase < d ? ebase : d - 1, hints);
            seg_lo = seg_off[s];
            seg_hi = s + 1 < nseg ? seg_off[s + 1] : d_pad;
        }
        replace_nan(x);
        for (;;) {
            // the part of the tile that belongs to this segment, as offsets from the tile's start
            const uint32_t lo_rel = (uint32_t)(seg_lo > ebase ? (seg_lo - ebase < (uint64_t)tile_len ? seg_lo - ebase : tile_len) : 0);
            const uint32_t hi_rel = (uint32_t)(seg_hi > ebase ? (seg_hi - ebase < (uint64_t)tile_len ? seg_hi - ebase : tile_len) : 0);
            const tq_params_t* P = params + s;
            float lv[16];
            const float alpha = P->alpha;
            const float inv_step = P->inv_w[0];
            const bool nonuniform = P->grid != TQ_GRID_UNIFORM;    // uniform over the workgroup
            if (nonuniform) {
                if (table_used) __syncthreads();               // the table of the segment before is done with
                table_used = true;
                fill_level_lds(tab, P, (1u << BITS) - 1u);
#pragma unroll
                for (int j = 0; j < 16; ++j) lv[j] = P->level[j];   // wave-uniform: scalar loads
                __syncthreads();
            }
            if (rel >= lo_rel && rel < hi_rel && byte_rel < pay_rel) {
                uint32_t word = 0;                                 // a group wholly in the padding encodes as 0
                if (n_valid == kGroup)
                    word = nonuniform ? encode_group<BITS, TQ_GRID_NONUNIFORM, false>(x, rw, 8, alpha, inv_step, lv, tab)
                                      : encode_group<BITS, TQ_GRID_UNIFORM, false>(x, rw, 8, alpha, inv_step, lv, tab);
                else if (n_valid > 0)
                    word = nonuniform ? encode_group<BITS, TQ_GRID_NONUNIFORM, true>(x, rw, n_valid, alpha, inv_step, lv, tab)
                                      : encode_group<BITS, TQ_GRID_UNIFORM, true>(x, rw, n_valid, alpha, inv_step, lv, tab);
                store_codes<BITS>(payload + tile_byte + byte_rel, word, (uint64_t)(pay_rel - byte_rel));
            }
            if (hi_rel >= tile_len || s + 1 >= nseg) break;
            ++s;
            seg_lo = seg_hi;
            seg_hi = s + 1 < nseg ? seg_off[s + 1] : d_pad;
        }
    }
}

// tq_quantize_dequantize: out[e] = Q[T_alpha(g[e])] as the server would reconstruct it from
// this worker's message (the level of the code tq_compress_kernel would have written: same
// draws, same arithmetic), without the round trip through a payload.  T tiles per workgroup, the compress kernel's
// general path, and the decode kernel's whole-line stores wherever a whole wavefront has whole
// groups.  Large outputs (PAST_CACHES, simulate_past) are written past the caches, and so is read what is read, old sums
// in the pieces that are stored.  Bound by its memory traffic and, at 25 M elements, by filling and draining the
// chip.  The mirrored path of the compress kernel, half-line stores / this: 61,706 fp32 at b = 3 3.8 / 3.4 / 2.9 us, 25.6 M
// bf16 24.4 / 26.1 / 24.5, accumulating 37.5 / 40.1 / 37.3, in buckets of 1024 64 / 31.6 / 31.1, 124 M bf16 104 / 138 / 103.5.
// Whole lines laid out through LDS, of which it reads little otherwise; in registers / through LDS, bf16 25.6 M at b = 4 26.7 / 26.0, 60 M
// 57.1 / 55.2, 124 M 117.0 / 112.9 (b = 3 108.9 / 105.0, b = 2 107.0 / 106.5), fp32 the same.
template <int DTYPE, int BITS, bool ACC, bool PAST_CACHES, int T>
__global__ __launch_bounds__(kBlock) void tq_simulate_kernel(
    const void* __restrict__ g, uint64_t d, uint64_t d_pad, uint64_t bucket_elems, uint32_t groups_per_bucket,
    const tq_params_t* __restrict__ params, uint32_t seed_lo, uint32_t seed_hi, uint32_t worker, uint32_t step,
    float* __restrict__ out)
{
    constexpr uint32_t S = (1u << BITS) - 1u;
    const uint32_t blk = linear_block();
    const uint32_t bucket = blk / groups_per_bucket;
    const uint32_t grp = blk - bucket * groups_per_bucket;
    const uint64_t bstart = (uint64_t)bucket * bucket_elems;
    uint64_t bend = bstart + bucket_elems < d_pad ? bstart + bucket_elems : d_pad;
    bend = bend < d ? bend : d;
    const uint64_t gbase = bstart + (uint64_t)grp * T * kTile;
    if (gbase >= bend) return;
    const tq_params_t* P = params + bucket;

    __shared__ LevelLds tab;                                   // the table, and what a code stands for
    __shared__ float4_native xbuf[kBlock / 64][128];           // store8_wave_lds's exchange buffers
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const Codebook cb = read_codebook(P);
    float lv[16];
    set_up_levels<BITS>(P, tab, lv);
    const uint64_t wave_base = gbase + (uint64_t)wave * (64 * kGroup);    // this wavefront's part of the first tile
    if (wave_base >= bend) return;                             // and of the others

    // all reads first, the draws under them
    // past the caches a lane's 32 bytes of fp32 are read as whole lines, of which half is not kept for the other half: a lane's
    // own / whole lines, 62 M in buckets of 2176 126 / 112 us, of 1024 86.2 / 82.5, of 16384 80.1 / 77.8, 124 M 163 / 154.5
    constexpr bool kLines = DTYPE == TQ_F32 && PAST_CACHES;
    float x[T][8], prev[T][8];
    uint32_t rw[T][4];
    // the old sum: past the caches a whole wavefront reads the 16-byte pieces that it will store, otherwise each lane its own
    auto load_prev = [&](int t) {
        const uint64_t base = wave_base + (uint64_t)t * kTile, e0 = base + (uint64_t)lane * kGroup;
        if (e0 + kGroup <= bend) {
            const bool pieces = PAST_CACHES && base + 64 * kGroup <= bend;
            const float4_native* pa = reinterpret_cast<const float4_native*>(out + (pieces ? base + 4u * lane : e0));
            const float4_native* pb = pa + (pieces ? 64 : 1);
            float4_native a, b;
            if constexpr (PAST_CACHES) { a = __builtin_nontemporal_load(pa); b = __builtin_nontemporal_load(pb); }
            else { a = *pa; b = *pb; }
            prev[t][0] = a.x; prev[t][1] = a.y; prev[t][2] = a.z; prev[t][3] = a.w;
            prev[t][4] = b.x; prev[t][5] = b.y; prev[t][6] = b.z; prev[t][7] = b.w;
        } else if (e0 < bend) {
#pragma unroll
            for (int j = 0; j < 7; ++j)
                if (e0 + j < bend) prev[t][j] = out[e0 + j];
        }
    };
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const uint64_t base = wave_base + (uint64_t)t * kTile, e0 = base + (uint64_t)lane * kGroup;
#pragma unroll
        for (int j = 0; j < 8; ++j) { x[t][j] = 0.0f; prev[t][j] = 0.0f; }
        if (kLines && base + 64 * kGroup <= bend) {
            load_groups_wave(g, base, lane, x[t]);
        } else if (e0 + kGroup <= bend) {
            load_group<DTYPE, PAST_CACHES && !kLines>(g, e0, x[t]);
        } else if (e0 < bend) {
#pragma unroll
            for (int j = 0; j < 7; ++j)                        // a ragged group has at most 7 elements
                if (e0 + j < bend) x[t][j] = load_one<DTYPE>(g, e0 + j);
        }
        if constexpr (ACC) load_prev(t);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
        draw_tile(gbase + (uint64_t)t * kTile, tid, worker, step, seed_lo, seed_hi, rw[t]);
        asm volatile("" : "+v"(rw[t][0]));                     // computed here, under the loads
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const uint64_t base = wave_base + (uint64_t)t * kTile, e0 = base + (uint64_t)lane * kGroup;
        if (base >= bend) break;
        if (kLines && base + 64 * kGroup <= bend) swap_pieces(x[t]);
        replace_nan(x[t]);
        const uint32_t word = encode_general<BITS, true>(x[t], rw[t], cb, lv, tab);
        float y[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            y[j] = tab.e[(word >> (j * BITS)) & S].x;
        }
        if (ACC && PAST_CACHES && base + 64 * kGroup <= bend) {
            store8_wave_lds<PAST_CACHES>(out + base, lane, y, xbuf[wave], prev[t]);
            continue;
        }
        if constexpr (ACC) {
#pragma unroll
            for (int j = 0; j < 8; ++j) y[j] = prev[t][j] + y[j];
        }
        if (base + 64 * kGroup <= bend) {
            store8_wave_lds<PAST_CACHES>(out + base, lane, y, xbuf[wave]);
        } else if (e0 + kGroup <= bend) {
            reinterpret_cast<float4*>(out + e0)[0] = make_float4(y[0], y[1], y[2], y[3]);
            reinterpret_cast<float4*>(out + e0)[1] = make_float4(y[4], y[5], y[6], y[7]);
        } else if (e0 < bend) {
#pragma unroll
            for (int j = 0; j < 7; ++j)
                if (e0 + j < bend) out[e0 + j] = y[j];
        }
    }
}

}  // namespace tq

namespace {

// Whether the memory-side cache (256 MiB) can still hold much of the batch from the statistics pass: up to twice its size.
// Then a lane reads its own 32 bytes past the caches and the payload is stored through them, else fp32 lines are read whole
// (load_groups_wave) and the payload goes past them (store_codes_wave).  Beside that: ranges that are cut and the one-tile
// segments kernel read a lane's own 32 bytes through the caches at any size; see reads_through too.
// fp32, a lane's own 32 bytes through the caches / whole lines, launches by themselves, us: uniform, one record 8 x 124 M at
// b = 2 699 / 670, at b = 4 743 / 695, buckets of 4096 2 x 400 M 550 / 524, but of 2^20 8 x 124 M 634 / 660 and 677 / 692, 900 M
// 574 / 600 (behind the statistics one step of 8 x 124 M at b = 2 1356 / 1338).  Level tables at b = 4 are slower with whole lines,
// for the exchange's instructions: 140 M 113 / 121 (the client's three calls 312 / 315), 8 x 37.5 M 238 / 249 (one step
// 502 / 492), 8 x 62 M 390 / 402 (768 / 759), 2 x 310 M 494 / 502 (1117 / 1083), 16 x 62 M 793 / 812 (1508 / 1516), in layers
// 8 x 124 M 799 / 797 (1559 / 1531).  The steps around the slower launches gain more often than they lose.
bool compress_cached(int count, uint64_t d, int dtype)
{
    return (uint64_t)count * d * (dtype == TQ_F32 ? 4u : 2u) <= (512ull << 20);
}

// Whether the uniform codebook at bf16, b = 4, reads through the caches: batches above 2 GiB.  Past them it loses up to a
// seventh of its speed at some sizes there (us, through / past, and the step around it): 12 x 110 M 575 / 617 (1174 / 1180),
// 32 x 62 M 897 / 1020 (1726 / 1760), 8 x 248 M 886 / 983 (1837 / 1881), 4 x 10^9 1761 / 1770 (3969 / 4028); below, 4 x 100 M
// 175 / 174 (409 / 398), 8 x 100 M 345 / 340 (747 / 738).  At b = 2 and 3 and with tables reading past them is as good or better.
bool reads_through(int count, uint64_t d) { return (uint64_t)count * d * 2u > (2ull << 30); }

// Whether level tables are checked for the mirrored path.  Its fewer instructions pay at b = 3 and, for bf16, at b = 2; the
// general path otherwise reads a lighter table and starts sooner.  General / mirrored, us: 16 x 25.6 M fp32 at
// b = 2 / 3 / 4 279 / 278, 326 / 300, 333 / 336, bf16 196 / 196, 263 / 227, 274 / 284; 11.2 M at b = 2 fp32 10.4 / 10.8,
// bf16 8.9 / 8.5.
constexpr bool mirrored_pays(int dtype, int bits) { return bits == 3 || (bits == 2 && dtype == TQ_BF16); }

struct CompressShape { bool table_tiles, mirror; };

// Tiles (4096 elements) of a workgroup of tq_compress_lookup_kernel, or 0 where the launch takes the tables as before.  Its 8192
// entries cost a workgroup as much as five of its tiles, so it wants many of them, in workgroups enough to fill the chip a few
// times.  us, as before / with 16 / 24 / 32 / 64 / 128 tiles, one record:
//   b = 2  124 M 60 / 63 / 61 / 64 / 63 / 74, 8 x 25.6 M 95 / 104 / 101 / 101 / 111 / 116, 4 x 124 M 220 / 219 / 217 / 218 / 244 / 255,
//          8 x 124 M 432 / 463 / 430 / 421 / 441 / 482, 4 x 10^9 1956 / 1907 / 1791 / 1739 / 1696 / 1688
//   b = 3  40 M 27 / 29 / 29 / 35 / 39 / 70, 60 M 37.6 / 36.8 / 39.5 / 36.4 / 41 / 71, 124 M 73 / 72 / 65 / 66 / 67 / 78, 8 x 124 M 519 / 494 /
//          468 / 475 / 500 / 531, 4 x 10^9 2304 / 2058 / 1931 / 1901 / 1882 / 1939
//   b = 4  20 M 18.9 / 20.8 / 19.3 / 22.8 / 37 / 67, 40 M 33.6 / 29.1 / 28.2 / 33.7 / 39 / 69, 124 M 91 / 72 / 64 / 67 / 64 / 75, 8 x 124 M 696 / 486 /
//          456 / 467 / 482 / 517, 4 x 10^9 2758 / 2050 / 1932 / 1955 / 1906 / 1912
// A bucket is cut into equal ranges of at least so many tiles, or taken whole: 4 x 124 M in buckets of 65536 (16 tiles) at b = 3
// 265 / 241, b = 4 332 / 234, of 16384 270 / 384 and 339 / 400; b = 2 4 x 140 M in buckets of 65536 266 / 264, of 98304 256 / 248, 4 x 250 M
// 460 / 452 and 457 / 430.
uint32_t look_tiles(int dtype, int bits, uint64_t bucket_elems, uint64_t elements)
{
    const uint64_t least = bits == 2 ? 1ull << 29 : (bits == 3 ? 1ull << 26 : 1ull << 25);
    const uint64_t of_bucket = (bucket_elems - 1) / tq::kLookTile + 1;
    if (dtype != TQ_BF16 || elements < least || of_bucket < 16) return 0;
    uint64_t wanted = elements / tq::kLookTile / 8192;
    wanted = wanted < 24 ? 24 : (wanted > 64 ? 64 : wanted);
    const uint64_t ranges = of_bucket < wanted ? 1 : of_bucket / wanted;
    return (uint32_t)((of_bucket - 1) / ranges + 1);
}

// The shape of a launch of level tables.
//   * Launches whose workgroups are all resident at once wait for latencies and take the tiles and the general path
//     of the uniform codebook: up to 512 tiles (fp32; 1024 at b = 3) or 4096 (bf16; at b = 3 the mirrored path from 1024 on).  General
//     with few tiles / general / mirrored with many, us: 250,000 fp32 at b = 3 2.9 / 3.5 / 3.4, 1.2 M 4.0 / 3.9 / 4.2,
//     3 M 4.7 / 4.7 / 4.4; 1.2 M bf16 at b = 4 4.4 / 5.7 / 6.1, 8 M 8.3 / 8.9 / 9.0, 11.2 M at b = 3 10.0 / 10.9 / 9.1.
//   * So do buckets shorter than a tile (fp32) or of at most two (bf16), of which every larger range is a cut one: 25.6 M at
//     b = 3 in buckets of 1024 fp32 30.4 / 33.0 / 35.2, bf16 31.5 / 43.3 / 44.1, of 4096 bf16 20.3 / 23.2 / 23.1 (but of 6144, a
//     whole and a half range in the smaller shape, 25.3 / 22.8 / 22.8).
CompressShape table_shape(int dtype, int bits, uint64_t bucket_elems, uint64_t all_tiles)
{
    const bool f32 = dtype == TQ_F32;
    if (f32 ? bucket_elems < (uint64_t)tq::kTile : bucket_elems <= 2 * (uint64_t)tq::kTile) return {false, false};
    if (all_tiles <= (f32 ? (bits == 3 ? 1024u : 512u) : 4096u)) return {false, !f32 && bits == 3 && all_tiles > 1024};
    return {true, mirrored_pays(dtype, bits)};
}

struct CompressArgs {
    dim3 blocks;
    hipStream_t st;
    tq::PtrTable g, params;
    tq::MutPtrTable payload;
    uint64_t d, d_pad, be, seed, pbytes;
    uint32_t groups_per_bucket, first_worker, step;
    bool through;
    uint32_t look;                                             // tiles of a workgroup that looks its codes up, or 0
};

template <int DTYPE, int BITS, bool CACHED, bool TABLE_TILES, bool MIRROR, bool THROUGH = false>
void launch_as(const CompressArgs& a)
{
    hipLaunchKernelGGL((tq::tq_compress_kernel<DTYPE, BITS, CACHED, tq::compress_tiles(DTYPE, TABLE_TILES), MIRROR, THROUGH>), a.blocks,
                       dim3(tq::kBlock), 0, a.st, a.g, a.d, a.d_pad, a.be, a.groups_per_bucket, a.params, (uint32_t)a.seed,
                       (uint32_t)(a.seed >> 32), a.first_worker, a.step, a.payload, a.pbytes);
}

template <int BITS, bool CACHED>
void launch_lookup(const CompressArgs& a)
{
    hipLaunchKernelGGL((tq::tq_compress_lookup_kernel<BITS, CACHED>), a.blocks, dim3(tq::kLookBlock), 0, a.st, a.g, a.d, a.d_pad, a.be,
                       a.groups_per_bucket, a.look, a.params, (uint32_t)a.seed, (uint32_t)(a.seed >> 32), a.first_worker, a.step,
                       a.payload, a.pbytes);
}

template <int DTYPE, int BITS, bool CACHED>
hipError_t launch(const CompressShape& shape, const CompressArgs& a)
{
    if constexpr (DTYPE == TQ_BF16 && !(BITS == 2 && CACHED)) {    // 2^29 elements are never read through the caches
        if (a.look) { launch_lookup<BITS, CACHED>(a); return hipGetLastError(); }
    }
    if constexpr (mirrored_pays(DTYPE, BITS)) {
        if (shape.mirror && shape.table_tiles) { launch_as<DTYPE, BITS, CACHED, true, true>(a); return hipGetLastError(); }
        if constexpr (DTYPE == TQ_BF16 && BITS == 3) {
            if (shape.mirror) { launch_as<DTYPE, BITS, CACHED, false, true>(a); return hipGetLastError(); }
        }
    } else if (shape.table_tiles) {
        launch_as<DTYPE, BITS, CACHED, true, false>(a);
        return hipGetLastError();
    }
    if constexpr (DTYPE == TQ_BF16 && BITS == 4 && !CACHED) {
        if (a.through) { launch_as<DTYPE, BITS, CACHED, false, false, true>(a); return hipGetLastError(); }
    }
    launch_as<DTYPE, BITS, CACHED, false, false>(a);
    return hipGetLastError();
}

}  // namespace

// Host side of tq_compress / tq_compress_multi after the argument checks of the C entry
// points: `count` same-shaped tensors in one launch (grid.y), workers first_worker + 0..count-1.
// `grid` (the family the caller names) only chooses the number of tiles per workgroup.
hipError_t tq_launch_compress(const void* const* g, int count, int dtype, uint64_t d, uint64_t bucket_elems,
                              const tq_params_t* const* params, int bits, int grid, uint64_t seed,
                              uint32_t first_worker, uint32_t step, void* const* payload, hipStream_t st)
{
    const uint64_t d_pad = (d + 127) / 128 * 128;
    const uint64_t be = bucket_elems ? bucket_elems : d_pad;
    const uint64_t nb = (d_pad + be - 1) / be;
    const uint64_t tiles = (be + tq::kTile - 1) / tq::kTile;                  // of a bucket
    CompressShape shape{false, false};
    if (grid != TQ_GRID_UNIFORM) shape = table_shape(dtype, bits, be, nb * tiles * (uint64_t)(count < 1 ? 1 : count));
    const uint64_t tt = (uint64_t)tq::compress_tiles(dtype, shape.table_tiles);
    CompressArgs a{};
    a.look = grid == TQ_GRID_UNIFORM ? 0u : look_tiles(dtype, bits, be < d_pad ? be : d_pad, d * (uint64_t)(count < 1 ? 1 : count));
    const uint64_t range = a.look ? (uint64_t)a.look * tq::kLookTile : tt * tq::kTile;      // elements of a workgroup
    const uint64_t ranges = (be - 1) / range + 1;              // of a bucket
    a.groups_per_bucket = (uint32_t)ranges;
    if (count < 1 || count > tq::kMaxBatch ||
        !tq::fold_grid(nb * ranges, a.look ? tq::kLookBlock : tq::kBlock, (unsigned)count, a.blocks))
        return hipErrorInvalidValue;
    for (int i = 0; i < count; ++i) { a.g.p[i] = g[i]; a.params.p[i] = params[i]; a.payload.p[i] = payload[i]; }
    a.st = st;
    a.d = d; a.d_pad = d_pad; a.be = be; a.seed = seed;
    a.pbytes = tq_payload_bytes(d, bits);
    a.first_worker = first_worker; a.step = step;
    const bool cached = compress_cached(count, d, dtype);
    a.through = reads_through(count, d);
#define TQ_LAUNCH_COMPRESS(DT, B) (cached ? launch<DT, B, true>(shape, a) : launch<DT, B, false>(shape, a))
#define TQ_LAUNCH_COMPRESS_B(DT) \
    (bits == 2 ? TQ_LAUNCH_COMPRESS(DT, 2) : (bits == 3 ? TQ_LAUNCH_COMPRESS(DT, 3) : TQ_LAUNCH_COMPRESS(DT, 4)))
    return dtype == TQ_F32 ? TQ_LAUNCH_COMPRESS_B(TQ_F32) : TQ_LAUNCH_COMPRESS_B(TQ_BF16);
#undef TQ_LAUNCH_COMPRESS_B
#undef TQ_LAUNCH_COMPRESS
}

// Whether a simulated gradient goes past the caches: outputs above 96 MiB, sums above 64 MiB.  us, through / past them, by itself, with an
// elementwise kernel behind it that reads the result, and with one that subtracts the gradient from it; above the
// lines the three together gain (bf16 20 M gains in sum, too, but the plain reader loses more there than the call gains):
//   bf16 (past: two tiles a workgroup)  20 M 25.1 / 23.7  47.7 / 49.8  102 / 97    25.2 M 29.9 / 28.4  59.3 / 60.0  87.7 / 74.8
//         25.6 M 30.4 / 29.1  60.3 / 61.0  114 / 94     30 M 34.5 / 32.9  71.2 / 69.4  102 / 91    40 M 44.1 / 41.8  96.7 / 97.4  144 / 138
//         62 M 67.0 / 62.5  152 / 146  180 / 175
//   fp32  22 M 31.2 / 29.3  57.7 / 58.8  68.7 / 71.1    25.6 M 35.9 / 33.5  70.9 / 66.7  83.9 / 87.4    40 M 55.0 / 51.1  111 / 107  139 / 135
//   sums  bf16 16 M 26.1 / 26.2  45.7 / 46.5  87.0 / 91.2    18 M 30.5 / 29.1  51.4 / 52.0  104 / 98    25.6 M 45.4 / 40.8  74.8 / 73.3  130 / 109
//         fp32 16 M 33.0 / 31.2  52.3 / 51.6  60.6 / 62.7    18 M 38.5 / 34.9  58.9 / 57.4  68.5 / 69.2    25.6 M 54.7 / 48.7  88.7 / 81.7  102 / 104
// Buckets of less than a wavefront's 512 elements hold no whole line to store: there the
// reads keep to the caches, sums of 25.6 M fp32 in buckets of 384 66.8 / 69.7.  62 M in buckets of 1024 and 2176: fp32 82.3 / 81.8
// and 110.5 / 111.7, sums 126 / 112 and 172 / 143, bf16 77.2 / 74.1 and 107.3 / 104.4, sums 105 / 97.8 and 148 / 125.
bool simulate_past(uint64_t d, uint64_t be, int accumulate)
{
    return be >= 512 && d * sizeof(float) > ((accumulate ? 64ull : 96ull) << 20);
}

// Host side of tq_quantize_dequantize after the argument checks of the C entry point.
hipError_t tq_launch_simulate(const void* g, int dtype, uint64_t d, uint64_t bucket_elems, const tq_params_t* params,
                              int bits, uint64_t seed, uint32_t worker, uint32_t step, int accumulate, float* out,
                              hipStream_t st)
{
    const uint64_t d_pad = (d + 127) / 128 * 128;
    const uint64_t be = bucket_elems ? bucket_elems : d_pad;
    const uint64_t nb = (d_pad + be - 1) / be;
    const bool past = simulate_past(d, be, accumulate);
    // one tile per workgroup; two for bf16 past the caches, in buckets of at least four.  One / two, at b = 3 by itself and with the two kernels
    // above behind it: 25.6 M 28.3 / 29.1  61.4 / 61.0  96.5 / 94.4, 40 M 42.0 / 41.8  99.2 / 97.4  138 / 138, 80 M 82.7 / 80.2  188 / 186  238 / 236;
    // but through the caches 25.6 M 24.5 / 25.7, and 124 M in buckets of 2048 111 / 174
    const bool two = dtype == TQ_BF16 && past && !accumulate && be >= 4 * (uint64_t)tq::kTile;
    const uint64_t tt = two ? 2 : 1;
    const uint64_t tpb = ((be + tq::kTile - 1) / tq::kTile + tt - 1) / tt;    // workgroups per bucket
    const uint64_t nblocks = nb * tpb;
    dim3 blocks;
    if (!tq::fold_grid(nblocks, tq::kBlock, 1, blocks)) return hipErrorInvalidValue;
    const uint32_t slo = (uint32_t)seed, shi = (uint32_t)(seed >> 32);
    const dim3 threads(tq::kBlock);
#define TQ_LAUNCH_SIM_AS(DT, B, ACC, PAST, T)                                                                       \
    hipLaunchKernelGGL((tq::tq_simulate_kernel<DT, B, ACC, PAST, T>), blocks, threads, 0, st, g, d, d_pad, be,      \
                       (uint32_t)tpb, params, slo, shi, worker, step, out)
#define TQ_LAUNCH_SIM(DT, B)                                                   \
    do {                                                                       \
        if (accumulate && past) TQ_LAUNCH_SIM_AS(DT, B, true, true, 1);        \
        else if (accumulate) TQ_LAUNCH_SIM_AS(DT, B, true, false, 1);          \
        else if (two) TQ_LAUNCH_SIM_AS(DT, B, false, true, DT == TQ_BF16 ? 2 : 1); \
        else if (past) TQ_LAUNCH_SIM_AS(DT, B, false, true, 1);                \
        else TQ_LAUNCH_SIM_AS(DT, B, false, false, 1);                         \
    } while (0)
#define TQ_LAUNCH_SIM_B(DT)                      \
    switch (bits) {                              \
        case 2: TQ_LAUNCH_SIM(DT, 2); break;     \
        case 3: TQ_LAUNCH_SIM(DT, 3); break;     \
        default: TQ_LAUNCH_SIM(DT, 4); break;    \
    }
    if (dtype == TQ_F32) { TQ_LAUNCH_SIM_B(TQ_F32) } else { TQ_LAUNCH_SIM_B(TQ_BF16) }
#undef TQ_LAUNCH_SIM_B
#undef TQ_LAUNCH_SIM
#undef TQ_LAUNCH_SIM_AS
    return hipGetLastError();
}


namespace {

// One tile per workgroup, requested before its segment is looked up, on the general path; else two (fp32) or four.
//   * Launches that are resident at once: 61,706 fp32 at b = 3 4.2 us against 5.2, bf16 4.3 against 8.3; 3 M fp32 5.6 / 6.2,
//     5 M 8.7 / 8.6; 11.2 M bf16 in segments of 20,000 13.1 / 16.1, of 10^6 11.6 / 13.3, 25.6 M 28.1 / 27.1 and 23.7 / 20.2.
//   * Segments so short that most larger ranges are cut and taken tile by tile: 124 M in segments of 5000 at b = 2 fp32 154 /
//     164, bf16 144 / 151, at b = 3 bf16 176 / 190, but fp32 178 / 163 and at b = 4 205 / 187 and 204 / 193; of 20,000 at
//     b = 2 121 / 109 and 114 / 86.
bool segments_one_tile(int count, int dtype, int bits, uint64_t d, uint64_t nseg)
{
    const uint64_t tiles = (uint64_t)(count < 1 ? 1 : count) * ((d + tq::kTile - 1) / tq::kTile);
    if (tiles <= (dtype == TQ_F32 ? 2048u : 8192u)) return true;
    return d / nseg < 12288 && (bits == 2 || (bits == 3 && dtype == TQ_BF16));
}

}  // namespace

// Host side of tq_compress_segments after the argument checks of the C entry point.
hipError_t tq_launch_compress_segments(const void* const* g, int count, int dtype, uint64_t d, const uint64_t* seg_off,
                                       const uint64_t* seg_host, uint64_t nseg, const tq_params_t* const* params, int bits, uint64_t seed,
                                       uint32_t first_worker, uint32_t step, void* const* payload, hipStream_t st)
{
    const uint64_t d_pad = (d + 127) / 128 * 128;
    const bool one_tile = segments_one_tile(count, dtype, bits, d, nseg);
    const uint64_t range = (one_tile ? 1u : (uint64_t)tq::segment_tiles(dtype)) * tq::kTile;        // elements per workgroup
    const uint64_t nblocks = (d_pad + range - 1) / range;
    dim3 blocks;
    if (count < 1 || count > tq::kMaxBatch || nseg > 0xFFFFFFFFull ||
        !tq::fold_grid(nblocks, tq::kBlock, (unsigned)count, blocks))
        return hipErrorInvalidValue;
    tq::PtrTable gt{}, pt{};
    tq::MutPtrTable yt{};
    for (int i = 0; i < count; ++i) { gt.p[i] = g[i]; pt.p[i] = params[i]; yt.p[i] = payload[i]; }
    const uint32_t slo = (uint32_t)seed, shi = (uint32_t)(seed >> 32);
    const uint64_t pbytes = tq_payload_bytes(d, bits);
    const dim3 threads(tq::kBlock);
    const tq::SegHints hints = tq::make_seg_hints(seg_host, nseg, d);
    const bool cached = compress_cached(count, d, dtype);
#define TQ_LAUNCH_CSEG(DT, B, ST, T, MI)                                                                        \
    hipLaunchKernelGGL((tq::tq_compress_segments_kernel<DT, B, ST, T, MI>), blocks, threads, 0, st, gt, d,      \
                       d_pad, seg_off, (uint32_t)nseg, hints, pt, slo, shi, first_worker, step, yt, pbytes)
#define TQ_LAUNCH_CSEG_T(DT, B, ST)                                                                    \
    do {                                                                                               \
        if (one_tile) TQ_LAUNCH_CSEG(DT, B, ST, 1, false);                                             \
        else TQ_LAUNCH_CSEG(DT, B, ST, tq::segment_tiles(DT), mirrored_pays(DT, B));                   \
    } while (0)
#define TQ_LAUNCH_CSEG_ST(DT, B) if (cached) TQ_LAUNCH_CSEG_T(DT, B, true); else TQ_LAUNCH_CSEG_T(DT, B, false)
#define TQ_LAUNCH_CSEG_B(DT)                         \
    switch (bits) {                                  \
        case 2: TQ_LAUNCH_CSEG_ST(DT, 2); break;     \
        case 3: TQ_LAUNCH_CSEG_ST(DT, 3); break;     \
        default: TQ_LAUNCH_CSEG_ST(DT, 4); break;    \
    }
    if (dtype == TQ_F32) { TQ_LAUNCH_CSEG_B(TQ_F32) } else { TQ_LAUNCH_CSEG_B(TQ_BF16) }
#undef TQ_LAUNCH_CSEG_B
#undef TQ_LAUNCH_CSEG_ST
#undef TQ_LAUNCH_CSEG_T
#undef TQ_LAUNCH_CSEG
    return hipGetLastError();
}

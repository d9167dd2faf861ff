// tq_decompress_aggregate and tq_decompress_aggregate_update: Alg. 1 server steps of
// arXiv 2402.01798,
//   g_bar[e] = sum_i w_i * L_i[code_i(e)],   then out = g_bar or theta <- theta - eta * g_bar,
// for all N workers in one pass.  Each lane owns 8 consecutive output elements: it reads the
// b bytes that hold their codes from every worker's stream, looks the levels up in LDS, adds
// them in worker order and writes 32 contiguous bytes of fp32 once.
//
// Two kernels share that shape:
//   tq_decode_fast_kernel    the fast path (N <= 16; N <= 8 at b = 4): per worker a table
//                            indexed by TWO adjacent codes (2^(2b) entries of float2), so one
//                            8-byte LDS read serves two elements; a single memory round trip
//                            per workgroup.
//   tq_decode_many_kernel    any N up to 64 at any b: the workers taken eight at a time.
#include <type_traits>

#include "tq_device.h"
#include "tq_layout.h"

namespace tq {

struct DecodeArgs {
    const uint8_t* payload[TQ_MAX_WORKERS];
    const tq_params_t* params[TQ_MAX_WORKERS];
    float weight[TQ_MAX_WORKERS];
};

// The word that holds the 8 codes of a group, as code_load (tq_layout.h) places it.  Nothing
// here depends on the loaded value, so the load stays in flight until the codes are used; the
// caller shifts by CodeLoad::first_bit (non-zero only for the last groups of a 3-bit payload).
// PAST (b = 4, whose loads of a wavefront are whole lines): past the caches, see payloads_past.
template <int BITS, bool PAST = false>
__device__ __forceinline__ uint32_t load_code_word(const uint8_t* stream, const CodeLoad& c)
{
    if constexpr (PAST) return __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(stream + c.load_off));
    if constexpr (BITS == 2) return *reinterpret_cast<const uint16_t*>(stream + c.load_off);
    uint32_t w;
    __builtin_memcpy(&w, stream + c.load_off, 4);          // b = 3: byte-aligned only
    return w;
}

// What happens to the aggregate g_bar of an element (the MODE of the kernels below):
//   kStore        out = g_bar                           Alg. 1, server step "aggregate"
//   kStoreStream  the same, stored with the non-temporal hint (small and very large outputs, see streams_output)
//   kAccumulate   out = out + g_bar
//   kSgd          theta = theta - eta * u,  u = g_bar + weight_decay * theta
//                                                       Alg. 1, server step "update", fused
//   kSgdMomentum  v = momentum * v + u;  theta = theta - eta * v
//                                                       the momentum SGD of the Sec. V experiments
// every product and sum rounded once to binary32, in that order.  MODE is a template parameter
// on purpose: with a run-time flag the read-modify-write branch leaves "a load may be pending"
// on every path, and the compiler then waits for ALL outstanding memory operations -- the
// tile's own stores included -- before the next tile.
//   ... | kPast   the modes that read back, past the caches: what they read and write is too much for them (reads_past)
enum { kStore = 0, kAccumulate = 1, kSgd = 2, kSgdMomentum = 3, kStoreStream = 4, kPast = 8 };
constexpr bool reads_back(int mode) { return mode != kStore && mode != kStoreStream; }
constexpr bool has_velocity(int mode) { return (mode & ~kPast) == kSgdMomentum; }

struct Update {
    float eta, momentum, weight_decay;
    float* velocity;
};

template <int MODE>
__device__ __forceinline__ float finish(float g_bar, float prev, float& vel, const Update& up)
{
    if constexpr (!reads_back(MODE)) {
        return g_bar;
    } else if constexpr ((MODE & ~kPast) == kAccumulate) {
        return prev + g_bar;
    } else {
        float u = g_bar;
        if (up.weight_decay != 0.0f) {
            const float decay = up.weight_decay * prev;
            u = g_bar + decay;
        }
        if constexpr (has_velocity(MODE)) {
            const float carried = up.momentum * vel;
            u = carried + u;
            vel = u;
        }
        const float delta = up.eta * u;
        return prev - delta;
    }
}

__device__ __forceinline__ void load8(const float* p, float (&x)[8])
{
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}

// STREAM: stored with the non-temporal hint.  Here, in ranges that are cut, the two 16-byte halves of a lane's 32 bytes
// leave L2 as separate partial writes with it; whole wavefronts store whole lines (store8_wave).  Storing the halves
// through the caches instead: 124 M in buckets of 1536 128 -> 132 us and in segments of 2176 142 -> 215, 11.2 M in buckets
// of 384 36.5 -> 38.8, but in segments of 512 29.4 -> 26.2.
template <bool STREAM>
__device__ __forceinline__ void store8(float* p, const float (&x)[8])
{
    if constexpr (STREAM) {
        float4_native a = {x[0], x[1], x[2], x[3]}, b = {x[4], x[5], x[6], x[7]};
        __builtin_nontemporal_store(a, reinterpret_cast<float4_native*>(p));
        __builtin_nontemporal_store(b, reinterpret_cast<float4_native*>(p) + 1);
    } else {
        reinterpret_cast<float4*>(p)[0] = make_float4(x[0], x[1], x[2], x[3]);
        reinterpret_cast<float4*>(p)[1] = make_float4(x[4], x[5], x[6], x[7]);
    }
}

// A lane's whole group: prev (and vel) were loaded by the caller, early, when MODE needs them.
template <int MODE>
__device__ __forceinline__ void finish_group(float* o, uint64_t e0, float (&acc)[8], const float (&prev)[8],
                                             float (&vel)[8], const Update& up)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = finish<MODE>(acc[j], prev[j], vel[j], up);
    store8<MODE == kStoreStream>(o, acc);
    if constexpr (has_velocity(MODE)) store8<false>(up.velocity + e0, vel);
}

// What the epilogue reads back (the old output, the parameters, the velocity) is requested with the code words, by the lanes
// that own a whole group.  PIECES and a workgroup whose lanes all do: a lane's two loads are not its own 32 bytes but the
// pieces that it will store (wave_piece), so that each load reads 1 KiB in one piece and nothing but the aggregate
// has to be exchanged; such lines can be read and written past the caches, which is where this pays (reads_past).
template <bool PIECES>
struct ReadBack {
    uint64_t first, second;                                // elements of the two loads
    bool any;
    __device__ __forceinline__ ReadBack(uint64_t e0, uint32_t lane, bool whole, uint64_t bend)
    {
        const bool pieces = PIECES && whole;
        first = pieces ? e0 - (uint64_t)lane * kGroup + wave_piece(lane) * 4u : e0;
        second = first + (pieces ? 256u : 4u);
        any = e0 + kGroup <= bend;
    }
    template <bool PAST>
    __device__ __forceinline__ void load(const float* p, float (&x)[8]) const
    {
        const float4_native *pa = reinterpret_cast<const float4_native*>(p + first), *pb = reinterpret_cast<const float4_native*>(p + second);
        float4_native a, b;
        if constexpr (PAST) { a = __builtin_nontemporal_load(pa); b = __builtin_nontemporal_load(pb); }
        else { a = *pa; b = *pb; }
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    }
};

// `prev` and `vel` hold the lane's pieces (modes that read back), `acc` its group.
template <int MODE, bool LDS, bool PIECES>
__device__ __forceinline__ void finish_group_wave(float* out, uint64_t e0, uint32_t lane, float (&acc)[8],
                                                  const float (&prev)[8], float (&vel)[8], const Update& up,
                                                  float4_native* wb)
{
    const uint64_t wave_e0 = e0 - (uint64_t)lane * kGroup;
    if constexpr (PIECES && reads_back(MODE)) {
        swap_pieces(acc);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = finish<MODE>(acc[j], prev[j], vel[j], up);
        store_lane_pieces<(MODE & kPast) != 0>(out + wave_e0, lane, acc);
        if constexpr (has_velocity(MODE)) store_lane_pieces<(MODE & kPast) != 0>(up.velocity + wave_e0, lane, vel);
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = finish<MODE>(acc[j], prev[j], vel[j], up);
        if constexpr (LDS) store8_wave_lds<MODE == kStoreStream>(out + wave_e0, lane, acc, wb);
        else store8_wave<MODE == kStoreStream>(out + wave_e0, lane, acc);
        if constexpr (has_velocity(MODE)) store8_wave<false>(up.velocity + wave_e0, lane, vel);
    }
}

// The ragged end of the tensor, element by element (only in the last workgroup of the tensor;
// the workgroups whose lanes all own whole groups take a separate, straight-line path, so
// that whatever the compiler makes of these predicated stores does not touch theirs).
template <int MODE>
__device__ __forceinline__ void finish_ragged(float* o, uint64_t e0, const float (&acc)[8], int n_valid,
                                              const Update& up)
{
#pragma unroll
    for (int j = 0; j < 7; ++j) {                          // a ragged group has at most 7 elements
        if (j < n_valid) {
            float prev = 0.0f, vel = 0.0f;
            if constexpr (reads_back(MODE)) prev = o[j];
            if constexpr (has_velocity(MODE)) vel = up.velocity[e0 + j];
            o[j] = finish<MODE>(acc[j], prev, vel, up);
            if constexpr (has_velocity(MODE)) up.velocity[e0 + j] = vel;
        }
    }
}

// Plain level tables of one bucket: row i = worker i's 16 levels, pre-multiplied by w_i
// when explicit weights are given (one rounding per level, as the weighted sum is defined).
__device__ __forceinline__ void fill_level_rows(float* table, const DecodeArgs& args, int N, int weighted,
                                                uint64_t bucket)
{
    for (int idx = threadIdx.x; idx < N * 16; idx += kBlock) {
        const int i = idx >> 4;
        float l = args.params[i][bucket].level[idx & 15];
        if (weighted) l = args.weight[i] * l;
        table[idx] = l;
    }
}

// tq_decode_fast_kernel<BITS, U, T, MODE>: U = workers handled (N rounded up to 1, 2, 4, 8 or 16;
// the rows of the missing workers are zero and their stream is worker 0's, so they add 0),
// T = tiles per workgroup, MODE = what is done with the aggregate (see above).
//
// One shot per workgroup, no loop over tiles: on this ISA loads and stores retire through ONE
// in-order counter, so a wave that stores a tile and then waits for further loads also waits
// for its stores to reach memory; a wave that ends after its stores waits for nothing.  What
// is left on the critical path is one memory round trip, so the kernel is arranged to make it
// exactly one: the code words of all T tiles are requested first; meanwhile each wavefront
// fetches the level rows of "its" workers through a scalar (wave-uniform) pointer, expands
// them to pair entries with two cross-lane reads and writes them to LDS; one barrier.
//
// SEG: the records are those of variable-size segments instead of buckets.  A workgroup takes
// T tiles wherever they fall; its reads are requested before the segment is looked up, and
// when its whole range lies inside one segment (nearly always) the rest is the bucketed code
// with that segment's record.  Otherwise it takes its tiles one by one, the segments that
// overlap a tile one after the other, with plain level rows -- the same sums in the same order.
//
// LDS: whole wavefronts lay their results out through LDS instead of in registers (lds_above).
template <int BITS, int U, int T, int MODE, bool SEG, bool LDS>
__global__ __launch_bounds__(kBlock) void tq_decode_fast_kernel(
    const DecodeArgs args, int N, int weighted, float scale, uint64_t d, uint64_t d_pad, uint64_t bucket_elems,
    uint32_t groups_per_bucket, uint64_t payload_bytes, float* __restrict__ out, const Update up,
    const uint64_t* __restrict__ seg_off, uint32_t nseg, const SegHints hints)
{
    constexpr int PAIRS = 1 << (2 * BITS);
    constexpr uint32_t PMASK = PAIRS - 1;
    constexpr uint32_t CMASK = (1u << BITS) - 1u;
    __shared__ float2 pair_tab[U * PAIRS];
    float4_native* wb = nullptr;
    if constexpr (LDS) {
        __shared__ float4_native xbuf[kBlock / 64][128];
        wb = xbuf[__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))];
    }

    const uint32_t blk = linear_block();
    uint32_t bucket = 0;                                       // the record of the workgroup's range
    uint64_t gstart, bend;                                     // its first element, the end of what it may take
    if constexpr (!SEG) {
        bucket = blk / groups_per_bucket;
        const uint32_t grp = blk - bucket * groups_per_bucket;
        const uint64_t bstart = (uint64_t)bucket * bucket_elems;
        bend = bstart + bucket_elems < d_pad ? bstart + bucket_elems : d_pad;
        bend = bend < d ? bend : d;
        gstart = bstart + (uint64_t)grp * T * kTile;
    } else {
        gstart = (uint64_t)blk * T * kTile;
        bend = d;                                              // for the reads; the segment's end comes later
    }
    if (gstart >= bend) return;

    // this lane's group in each tile; lanes past the end read group 0 (always present)
    uint64_t e0[T];
    CodeLoad cl[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        e0[t] = gstart + (uint64_t)t * kTile + (uint64_t)threadIdx.x * kGroup;
        cl[t] = code_load(e0[t] < bend ? e0[t] >> 3 : 0, BITS, payload_bytes);
    }
    uint32_t w[T][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint8_t* stream = args.payload[u < N ? u : 0];
#pragma unroll
        for (int t = 0; t < T; ++t) w[t][u] = load_code_word<BITS>(stream, cl[t]);
    }
    // what the epilogue reads back (the old output, the parameters, the velocity) is requested
    // now as well, for the lanes that own a whole group
    float prev[T][8], vel[T][8];
#pragma unroll
    for (int t = 0; t < T; ++t) {
#pragma unroll
        for (int j = 0; j < 8; ++j) { prev[t][j] = 0.0f; vel[t][j] = 0.0f; }
        const ReadBack<!SEG> back(e0[t], threadIdx.x & 63u, gstart + (uint64_t)T * kTile <= bend, bend);
        if (back.any) {
            if constexpr (reads_back(MODE)) back.template load<(MODE & kPast) != 0>(out, prev[t]);
            if constexpr (has_velocity(MODE)) back.template load<(MODE & kPast) != 0>(up.velocity, vel[t]);
        }
    }

    if constexpr (SEG) {
        __shared__ float rows[16 * 16];                        // plain level rows: U <= 16 workers
        constexpr uint32_t MASK = (1u << BITS) - 1u;
        const uint32_t s0 = find_segment(seg_off, nseg, gstart, hints);
        const uint64_t lo0 = seg_off[s0];
        const uint64_t hi0 = s0 + 1 < nseg ? seg_off[s0 + 1] : d_pad;
        if (lo0 <= gstart && gstart + (uint64_t)T * kTile <= (hi0 < d ? hi0 : d)) {
            bucket = s0;                                       // one record for the whole range: as for a bucket
        } else {
            for (int t = 0; t < T; ++t) {                      // the same for the whole workgroup
                const uint64_t tbase = gstart + (uint64_t)t * kTile;
                if (tbase >= d) break;
                const uint64_t tile_end = tbase + kTile < d_pad ? tbase + kTile : d_pad;
                uint32_t s = t == 0 ? s0 : find_segment(seg_off, nseg, tbase, hints);
                for (;;) {
                    const uint64_t seg_lo = seg_off[s];
                    const uint64_t seg_hi = s + 1 < nseg ? seg_off[s + 1] : d_pad;
                    __syncthreads();                           // the rows of the segment before are done with
                    fill_level_rows(rows, args, N, weighted, s);
                    __syncthreads();
                    if (e0[t] >= seg_lo && e0[t] < seg_hi && e0[t] < d) {
                        float acc[8];
#pragma unroll
                        for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            if (u < N) {
                                const uint32_t codes = w[t][u] >> cl[t].first_bit;
#pragma unroll
                                for (int j = 0; j < 8; ++j) acc[j] = acc[j] + rows[u * 16 + ((codes >> (j * BITS)) & MASK)];
                            }
                        }
                        if (!weighted) {
#pragma unroll
                            for (int j = 0; j < 8; ++j) acc[j] = acc[j] * scale;
                        }
                        if (e0[t] + kGroup <= d) finish_group<MODE>(out + e0[t], e0[t], acc, prev[t], vel[t], up);
                        else finish_ragged<MODE>(out + e0[t], e0[t], acc, (int)(d - e0[t]), up);
                    }
                    if (seg_hi >= tile_end || s + 1 >= nseg) break;
                    ++s;
                }
            }
            return;
        }
    }

    // pair tables: wavefront `wave` expands workers wave, wave + 4, ...  The wave index is
    // read into a scalar register so that the worker's pointer and weight are scalar loads.
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    float lrow[(U + 3) / 4];
#pragma unroll
    for (int k = 0; k < (U + 3) / 4; ++k) {
        const int i = wave + 4 * k;
        lrow[k] = 0.0f;
        if (i < N) {
            const tq_params_t* P = args.params[i] + bucket;
            const float wsel = weighted ? args.weight[i] : 1.0f;   // x * 1.0f is exact
            lrow[k] = wsel * P->level[lane & 15];
        }
    }
#pragma unroll
    for (int k = 0; k < (U + 3) / 4; ++k) {
        const int i = wave + 4 * k;
        if (i < U) {
#pragma unroll
            for (int e = lane; e < PAIRS; e += 64) {
                const float lo = __shfl(lrow[k], (int)(e & CMASK), 64);
                const float hi = __shfl(lrow[k], (int)(e >> BITS), 64);
                pair_tab[i * PAIRS + e] = make_float2(lo, hi);
            }
        }
    }
    __syncthreads();
    const float post = weighted ? 1.0f : scale;                // x * 1.0f is exact

    auto lookup = [&](int t, float (&acc)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const uint32_t codes = BITS == 3 ? w[t][u] >> cl[t].first_bit : w[t][u];
                const float2 v = pair_tab[u * PAIRS + ((codes >> (2 * BITS * m)) & PMASK)];
                acc[2 * m] = acc[2 * m] + v.x;
                acc[2 * m + 1] = acc[2 * m + 1] + v.y;
            }
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = acc[j] * post;
    };

    if (gstart + (uint64_t)T * kTile <= bend) {
        // Every lane of the workgroup owns a whole group (all but the last workgroup of a
        // bucket): straight-line code, each tile stored as soon as it is looked up.
#pragma unroll
        for (int t = 0; t < T; ++t) {
            float acc[8];
            lookup(t, acc);
            finish_group_wave<MODE, LDS, !SEG>(out, e0[t], (uint32_t)lane, acc, prev[t], vel[t], up, wb);
        }
    } else {
        // the last workgroup of a bucket: tile by tile (one tile's values live at a time)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            float acc[8];
            lookup(t, acc);
            if (e0[t] + kGroup <= bend) finish_group<MODE>(out + e0[t], e0[t], acc, prev[t], vel[t], up);
            else if (e0[t] < bend) finish_ragged<MODE>(out + e0[t], e0[t], acc, (int)(bend - e0[t]), up);
        }
    }
}

// More workers than the fast kernel holds code words and pair tables for (N > 16, N > 8 at b = 4), up to
// U.  The tables of all workers are built once per workgroup -- pair entries at b = 2; at b = 3 and 4, where
// pairs take 512 B or 2 KiB a worker and their random rows meet in the banks, the plain levels, which lie
// in banks of their own -- and the workers are taken eight at a time, straight-line: the next eight's
// code words are on their way while the current ones are looked up, and every table address is a
// constant beside the masked code.  Sums in worker order.
// Bound by the rate of LDS reads (one per four clocks and compute unit, 4 bytes wide as well as 8).  11.2 M
// elements, N = 32, before (a loop over the workers, a load and eight look-ups each) -> now: b = 4 57.2 -> 44.7 us,
// b = 3 56.1 -> 45.4 (50.6 with pairs), b = 2 46.3 -> 28.7; N = 64 106 -> 79.5, N = 12 at b = 4 21.6 -> 18.9.
// PAST: the payloads are read past the caches (payloads_past).
// PART: the last eight end after the pair that holds the last worker; without it they are looked up whole.  The branches
// cost whole batches up to 6 % at b = 2 and 3 with two tiles (11.2 M, N = 24 at b = 3 28.0 -> 29.9 us) and give what the
// rows past the last worker would take: N = 9 at b = 4 20.6 -> 17.2, N = 17 28.2 -> 25.6; 61,706 elements (one tile),
// N = 17 at b = 3 7.0 -> 4.5.
template <int BITS, int U, int T, int MODE, bool PART, bool PAST>
__global__ __launch_bounds__(kBlock) void tq_decode_many_kernel(
    const DecodeArgs args, int N, int weighted, float scale, uint64_t d, uint64_t d_pad, uint64_t bucket_elems,
    uint32_t groups_per_bucket, uint64_t payload_bytes, float* __restrict__ out, const Update up)
{
    constexpr int C = 8;                                       // workers at a time
    constexpr bool PAIR = BITS == 2;
    constexpr int ENTRIES = PAIR ? 16 : 1 << BITS;             // of 8 or 4 bytes
    constexpr int ROW = ENTRIES * (PAIR ? 8 : 4);              // bytes of a worker's table
    constexpr int CMASK = (1 << BITS) - 1;
    __shared__ __align__(16) char table[U * ROW];

    const uint32_t blk = linear_block();
    const uint32_t bucket = blk / groups_per_bucket;
    const uint32_t grp = blk - bucket * groups_per_bucket;
    const uint64_t bstart = (uint64_t)bucket * bucket_elems;
    uint64_t bend = bstart + bucket_elems < d_pad ? bstart + bucket_elems : d_pad;
    bend = bend < d ? bend : d;
    const uint64_t gstart = bstart + (uint64_t)grp * T * kTile;
    if (gstart >= bend) return;

    // this lane's group in each tile; lanes past the end read group 0 (always present)
    uint64_t e0[T];
    CodeLoad cl[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        e0[t] = gstart + (uint64_t)t * kTile + (uint64_t)threadIdx.x * kGroup;
        cl[t] = code_load(e0[t] < bend ? e0[t] >> 3 : 0, BITS, payload_bytes);
    }
    // past the last worker its words again (looked up in tables of zeros)
    auto request = [&](uint32_t (&w)[T][C], int c) {
#pragma unroll
        for (int u = 0; u < C; ++u) {
            const uint8_t* stream = args.payload[c + u < N ? c + u : N - 1];
#pragma unroll
            for (int t = 0; t < T; ++t) w[t][u] = load_code_word<BITS, PAST>(stream, cl[t]);
        }
    };
    uint32_t w[2][T][C];
    request(w[0], 0);
    float prev[T][8], vel[T][8], acc[T][8];
#pragma unroll
    for (int t = 0; t < T; ++t) {
#pragma unroll
        for (int j = 0; j < 8; ++j) { prev[t][j] = 0.0f; vel[t][j] = 0.0f; acc[t][j] = 0.0f; }
        const ReadBack<true> back(e0[t], threadIdx.x & 63u, gstart + (uint64_t)T * kTile <= bend, bend);
        if (back.any) {
            if constexpr (reads_back(MODE)) back.template load<(MODE & kPast) != 0>(out, prev[t]);
            if constexpr (has_velocity(MODE)) back.template load<(MODE & kPast) != 0>(up.velocity, vel[t]);
        }
    }
    for (int idx = threadIdx.x; idx < U * ENTRIES; idx += kBlock) {
        const int i = idx / ENTRIES, e = idx % ENTRIES;
        float lo = 0.0f, hi = 0.0f;
        if (i < N) {
            const float* level = args.params[i][bucket].level;
            const float wsel = weighted ? args.weight[i] : 1.0f;   // x * 1.0f is exact
            lo = wsel * level[e & CMASK];
            if constexpr (PAIR) hi = wsel * level[e >> BITS];
        }
        if constexpr (PAIR) reinterpret_cast<float2*>(table)[idx] = make_float2(lo, hi);
        else reinterpret_cast<float*>(table)[idx] = lo;
    }
    __syncthreads();

#pragma unroll
    for (int c = 0; c < U; c += C) {
        if (c >= N) break;                                     // the same for every lane
        if (c + C < U) request(w[(c / C + 1) & 1], c + C);
#pragma unroll
        for (int u = 0; u < C; ++u) {
            // tables past the last worker hold zeros
            if (PART && u % 2 == 0 && c + u >= N) break;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint32_t word = w[(c / C) & 1][t][u];
                const uint32_t codes = BITS == 3 ? word >> cl[t].first_bit : word;
                const char* row = table + (c + u) * ROW;
                // the byte offset of an entry is the code (or two) in place, shifted and masked
                if constexpr (PAIR) {
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const uint32_t off = (m == 0 ? codes << 3 : codes >> (2 * BITS * m - 3)) & (uint32_t)(ROW - 8);
                        const float2 v = *reinterpret_cast<const float2*>(row + off);
                        acc[t][2 * m] = acc[t][2 * m] + v.x;
                        acc[t][2 * m + 1] = acc[t][2 * m + 1] + v.y;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t off = (j == 0 ? codes << 2 : codes >> (BITS * j - 2)) & (uint32_t)(ROW - 4);
                        acc[t][j] = acc[t][j] + *reinterpret_cast<const float*>(row + off);
                    }
                }
            }
        }
    }
    const float post = weighted ? 1.0f : scale;                // x * 1.0f is exact
    const uint32_t lane = threadIdx.x & 63u;
    const bool whole = gstart + (uint64_t)T * kTile <= bend;
#pragma unroll
    for (int t = 0; t < T; ++t) {
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[t][j] = acc[t][j] * post;
        if (whole) finish_group_wave<MODE, false, true>(out, e0[t], lane, acc[t], prev[t], vel[t], up, nullptr);
        else if (e0[t] + kGroup <= bend) finish_group<MODE>(out + e0[t], e0[t], acc[t], prev[t], vel[t], up);
        else if (e0[t] < bend) finish_ragged<MODE>(out + e0[t], e0[t], acc[t], (int)(bend - e0[t]), up);
    }
}

// tq_decompress_aggregate_segments: the server step with one codebook per variable-size
// segment (and worker), for more workers than the fast kernel takes.  One tile per workgroup, the
// segments that overlap it taken one after the other, each with the N workers' level rows of
// that segment in LDS.
template <int BITS, int MODE>
__global__ __launch_bounds__(kBlock) void tq_decode_segments_kernel(
    const DecodeArgs args, int N, int weighted, float scale, uint64_t d, uint64_t d_pad,
    const uint64_t* __restrict__ seg_off, uint32_t nseg, const SegHints hints, uint64_t payload_bytes,
    float* __restrict__ out, const Update up)
{
    constexpr uint32_t MASK = (1u << BITS) - 1u;
    const uint64_t ebase = (uint64_t)linear_block() * kTile;
    if (ebase >= d) return;
    const uint64_t tile_end = ebase + kTile < d_pad ? ebase + kTile : d_pad;
    const uint64_t e0 = ebase + (uint64_t)threadIdx.x * kGroup;
    __shared__ float table[TQ_MAX_WORKERS * 16];

    uint32_t s = find_segment(seg_off, nseg, ebase, hints);
    for (;;) {
        const uint64_t seg_lo = seg_off[s];
        const uint64_t seg_hi = s + 1 < nseg ? seg_off[s + 1] : d_pad;
        fill_level_rows(table, args, N, weighted, s);
        __syncthreads();
        if (e0 >= seg_lo && e0 < seg_hi && e0 < d) {
            const CodeLoad cl = code_load(e0 >> 3, BITS, payload_bytes);
            const bool whole = e0 + kGroup <= d;
            float acc[8], prev[8], vel[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) { acc[j] = 0.0f; prev[j] = 0.0f; vel[j] = 0.0f; }
            if (whole) {
                if constexpr (reads_back(MODE)) load8(out + e0, prev);
            }
            for (int i = 0; i < N; ++i) {
                const uint32_t w = load_code_word<BITS>(args.payload[i], cl) >> cl.first_bit;
                const float* row = table + i * 16;
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = acc[j] + row[(w >> (j * BITS)) & MASK];
            }
            if (!weighted) {
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = acc[j] * scale;
            }
            if (whole) finish_group<MODE>(out + e0, e0, acc, prev, vel, up);
            else finish_ragged<MODE>(out + e0, e0, acc, (int)(d - e0), up);
        }
        if (seg_hi >= tile_end || s + 1 >= nseg) break;
        ++s;
        __syncthreads();                                       // before the next segment's rows replace these
    }
}

}  // namespace tq

namespace {

// A plain aggregate is streamed past the caches when it is small -- written normally it stays behind as dirty lines of the
// memory-side cache, and their write-back competes with the next kernel's reads (12 us on the statistics launch that follows
// a 45 MB output) -- or too large for them.  The buffers of the fused update, which the next step reads again, never are.
bool streams_output(uint64_t d)
{
    return d * sizeof(float) <= (64ull << 20) || tq::output_past_caches(d * sizeof(float));
}

// Outputs of more bytes than this go through LDS on their way out, where the call is the plain average of buckets (U workers
// of tq_decode_fast_kernel); by what both ways measured over 12 M to 2 x 10^9 elements, in registers against through LDS, per cent:
//   b = 2, 16 workers  +3 .. +19 everywhere        8 workers  +2 .. +6 above 64 MiB, -3 .. +2 below
//   b = 4,  8 workers  +1 .. +5 above 160 MiB, -3 .. -11 below
//   b = 4, two and four  -4 .. +1 up to 1 GiB, +0 .. +12 above      one  -6 .. -2 up to 2 GiB, +4 .. +16 above
//   b = 2, one  -5 .. +4 up to 4.25 GiB, +5 .. +16 above            two  -5 .. +2 up to 2 GiB, +2 .. +9 above (-2 once)
//   b = 3, one  -8 .. +1 up to 2.75 GiB, +7 .. +13 above            8 workers  -5 .. -14   others  -4 .. +1
//   b = 2, four workers  -2 .. +1 up to 2.5 GiB, +1 .. +4 above by itself; behind a compress the other way round (4 x 10^9
//          bf16, one step, 3952 us in registers, 3964 through LDS), and it stays in registers
// The updates and sums lose nothing in registers (16 workers at b = 2 with SGD -5 .. -15), nor do segments (8 x 124 M at
// b = 2 in 68 layers 124 -> 114 us).
constexpr uint64_t kNever = ~0ull;
constexpr uint64_t lds_above(int bits, int U)
{
    constexpr uint64_t kMiB = 1ull << 20;
    if (U == 16) return bits == 2 ? 0 : kNever;
    if (U == 8) return bits == 2 ? 64 * kMiB : (bits == 4 ? 160 * kMiB : kNever);
    if (bits == 4) return (U == 1 ? 2048 : 1024) * kMiB;
    if (U == 1) return (bits == 2 ? 4352 : 2816) * kMiB;
    return bits == 2 && U == 2 ? 2048 * kMiB : kNever;
}

// Whether an update (or a sum) goes past the caches, in buckets of which few ranges are cut: from 96 MiB of parameters (or sum) on,
// with momentum from 88 MiB of parameters (at least 32), velocity and payloads on.  us, through / past the caches, by themselves, with an elementwise
// kernel behind them that reads the result, and with another one behind that; the lines lie where the three together gain:
//   momentum  1 x 8.5 M, b = 3 (68 MiB)    23.0 / 23.9  33.7 / 35.5  45.1 / 46.9      1 x 10 M, b = 3 (80)     26.2 / 27.6  41.2 / 41.6  54.5 / 54.7
//             8 x 8.5 M, b = 3 (89)        29.2 / 28.1  39.7 / 40.1  51.3 / 51.2      4 x 11.2 M, b = 2 (96)   33.5 / 32.0  47.6 / 47.2  61.9 / 61.0
//             16 x 8.5 M, b = 2 (97)       37.5 / 33.9  49.0 / 46.2  60.5 / 57.6      8 x 10 M, b = 4 (114)    38.2 / 35.1  51.0 / 50.2  64.5 / 63.6
//             8 x 16 M, b = 3 (168)        57.2 / 50.7  76.4 / 74.5  93.2 / 93.5      25 x 10 M, b = 3 (166)   60.8 / 57.1  72.7 / 73.2  86.0 / 85.9
//             8 x 25.6 M, b = 3 (269)      90.4 / 78.9  125 / 116    151 / 144        8 x 124 M, b = 3         430 / 383                 766 / 742
//   sgd       4 x 22 M, b = 2 (84 MiB)     34.4 / 32.7  59.9 / 61.9  85.5 / 87.5      4 x 25.6 M (98)          41.3 / 37.2  70.8 / 70.8  98.6 / 100.0
//             4 x 32 M (122)               52.5 / 45.6  93.2 / 89.6  122 / 122        4 x 62 M                 101 / 86.5   182 / 174    268 / 257
//   sums      8 x 22 M, b = 3 (84)         45.3 / 43.2  70.3 / 72.0  94.6 / 97.2      8 x 25.6 M (98)          53.0 / 49.7  85.7 / 84.0  110 / 112
//             8 x 32 M (122)               65.0 / 61.4  109 / 109    138 / 136        8 x 62 M                 122 / 115    204 / 201    291 / 286
// The same buffers again and again with nothing in between stay in the caches up to about 20 M: 8 x 16 M with momentum 45.7 / 48.1, 25.6 M
// 79.0 / 73.5.  Loads alone 92.5 -> 89.2 of 25.6 M with momentum, stores alone 93.2: it takes both.  A lane's own 32 bytes each way gave nothing.
bool reads_past(int mode, uint64_t d, uint64_t payloads, uint64_t bucket_elems)
{
    const uint64_t bytes = d * sizeof(float), all = mode == tq::kSgdMomentum ? 2 * bytes + payloads : bytes;
    return bytes > (32ull << 20) && all > ((mode == tq::kSgdMomentum ? 88ull : 96ull) << 20) && bucket_elems >= 16 * (uint64_t)tq::kTile;
}

// Whether the payloads of a launch of tq_decode_many_kernel are read past the caches: up to 16 MiB of them, and from 112 MiB on
// unless too many loads repeat the last worker's (the kernel requests eight workers' words at a time), which the caches answer.
// Through / past them at b = 4, us:
//   d       N = 9          12            16            17            25            32            64
//   1 M     4.4 / 4.4      4.6 / 4.5     5.1 / 5.0     6.2 / 6.1     7.5 / 7.2     8.2 / 7.8     13.4 / 13.0
//   4 M     8.2 / 8.2      8.8 / 8.8     10.2 / 10.3   12.1 / 13.0   14.6 / 15.3   16.6 / 17.3   30.2 / 29.2
//   8 M     13.5 / 15.3    15.7 / 17.1   17.4 / 19.0   20.8 / 23.4   27.5 / 27.2   35.5 / 33.5   62.9 / 59.5
//   11.2 M  18.1 / 20.9    19.5 / 22.4   25.6 / 25.8   28.5 / 30.7   36.3 / 34.7   43.9 / 41.5   78.0 / 72.9
//   40 M    70.0 / 68.1    76.9 / 72.8   92.2 / 86.9   96.5 / 101.6  127.6 / 121.3 156.5 / 149.8
//   80 M    118.0 / 121.2  139.1 / 133.3 168.2 / 158.6
// With momentum 12 x 5 M 19.3 / 23.4, 16 x 11.2 M 44.7 / 46.9, 32 x 11.2 M 66.3 / 64.5; added to a sum 32 x 11.2 M 58.7 / 51.1.
// At b = 2 and 3 a wavefront's load is half a line or not in place: 8 x 124 M at b = 2 120 / 133, 16 x 25.6 M at b = 3 53 / 63; and few
// workers, tq_decode_fast_kernel, lose too: 8 x 11.2 M at b = 4 17.3 / 18.4, 1 x 124 M 83 / 98.
bool payloads_past(int bits, int N, uint64_t payload_bytes)
{
    const uint64_t all = (uint64_t)N * payload_bytes;
    return bits == 4 && (all <= (16ull << 20) || (all > (112ull << 20) && 3 * ((N + 7) / 8 * 8) <= 4 * N));
}

// Whether launches of this kind can be above it: kStore is the mode of outputs of 64 to 160 MiB.
template <int MODE>
constexpr bool lds_possible(int bits, int U)
{
    return (MODE == tq::kStoreStream && lds_above(bits, U) != kNever) || (MODE == tq::kStore && lds_above(bits, U) < (160ull << 20));
}

struct DecodeGeom {
    tq::DecodeArgs args;
    int N, weighted, bits;
    float scale;
    uint64_t d, d_pad, be, nb, tpb, pbytes;
};

// One launch with the epilogue MODE fixed at compile time.
template <int MODE>
hipError_t launch_mode(const DecodeGeom& g, float* out, const tq::Update& up, hipStream_t st)
{
    const dim3 threads(tq::kBlock);
    const int N = g.N;
    if (N <= 16 && !(g.bits == 4 && N > 8)) {
        const int U = N <= 1 ? 1 : (N <= 2 ? 2 : (N <= 4 ? 4 : (N <= 8 ? 8 : 16)));
        // tiles per workgroup: two, so that the tables are built once per 4096 elements (measured
        // with 1 / 2 / 4 tiles: 8 x 124 M at b = 2 131 / 119 / 122 us; 16 x 25.6 M at b = 3, where two
        // tiles' code words take 122 registers and halve the resident wavefronts, 74 / 66 / - us)
        constexpr int T = 2;
        const uint64_t gpb = (g.tpb + T - 1) / T;
        const uint64_t nblocks = g.nb * gpb;
        dim3 blocks;
        if (!tq::fold_grid(nblocks, tq::kBlock, 1, blocks)) return hipErrorInvalidValue;
        const tq::SegHints no_hints{};
#define TQ_LAUNCH_FAST_AS(B, UU, TT, LDS)                                                                           \
    hipLaunchKernelGGL((tq::tq_decode_fast_kernel<B, UU, TT, MODE, false, LDS>), blocks, threads, 0, st, g.args, N, \
                       g.weighted, g.scale, g.d, g.d_pad, g.be, (uint32_t)gpb, g.pbytes, out, up,                   \
                       static_cast<const uint64_t*>(nullptr), 0u, no_hints)
#define TQ_LAUNCH_FAST(B, UU, TT)                                                                 \
    do {                                                                                          \
        constexpr bool may = lds_possible<MODE>(B, UU), always = may && lds_above(B, UU) == 0;    \
        if (g.d * sizeof(float) > lds_above(B, UU)) TQ_LAUNCH_FAST_AS(B, UU, TT, may);            \
        else TQ_LAUNCH_FAST_AS(B, UU, TT, always);                                                \
    } while (0)
#define TQ_LAUNCH_FAST_U(B)                                          \
    switch (U) {                                                     \
        case 1: TQ_LAUNCH_FAST(B, 1, T); break;                      \
        case 2: TQ_LAUNCH_FAST(B, 2, T); break;                      \
        case 4: TQ_LAUNCH_FAST(B, 4, T); break;                      \
        case 8: TQ_LAUNCH_FAST(B, 8, T); break;                      \
        default: TQ_LAUNCH_FAST(B, 16, T); break;  \
    }
        switch (g.bits) {
            case 2: TQ_LAUNCH_FAST_U(2) break;
            case 3: TQ_LAUNCH_FAST_U(3) break;
            default:
                switch (U) {                    // 16 workers at b = 4 would need 32 KiB of tables
                    case 1: TQ_LAUNCH_FAST(4, 1, T); break;
                    case 2: TQ_LAUNCH_FAST(4, 2, T); break;
                    case 4: TQ_LAUNCH_FAST(4, 4, T); break;
                    default: TQ_LAUNCH_FAST(4, 8, T); break;
                }
                break;
        }
#undef TQ_LAUNCH_FAST_U
#undef TQ_LAUNCH_FAST
#undef TQ_LAUNCH_FAST_AS
        return hipGetLastError();
    }

    // two tiles per workgroup, one where all workgroups are resident at once (eight per compute unit); one / two on
    // 11.2 M elements, N = 32: b = 4 45.5 / 44.7 us, b = 2 29.6 / 28.7.  So many tiles are at most 16 MiB of output, which some
    // modes are not for (streams_output, reads_past).
    constexpr bool kSmall = MODE != tq::kStore && (MODE & tq::kPast) == 0;
    const bool one_tile = kSmall && g.nb * g.tpb <= 2048, part = g.bits == 4 && N % 8 != 0;
    const bool past = payloads_past(g.bits, N, g.pbytes);
    const uint64_t gpb = one_tile ? g.tpb : (g.tpb + 1) / 2;
    dim3 blocks;
    if (!tq::fold_grid(g.nb * gpb, tq::kBlock, 1, blocks)) return hipErrorInvalidValue;
#define TQ_LAUNCH_MANY_AS(B, UU, T, PART)                                                                      \
    do {                                                                                                       \
        if (past) TQ_LAUNCH_MANY_READ(B, UU, T, PART, (B == 4));                                               \
        else TQ_LAUNCH_MANY_READ(B, UU, T, PART, false);                                                       \
    } while (0)
#define TQ_LAUNCH_MANY_READ(B, UU, T, PART, PAST)                                                              \
    hipLaunchKernelGGL((tq::tq_decode_many_kernel<B, UU, T, MODE, PART, PAST>), blocks, threads, 0, st, g.args, N, g.weighted, \
                       g.scale, g.d, g.d_pad, g.be, (uint32_t)gpb, g.pbytes, out, up)
#define TQ_LAUNCH_MANY(B, UU)                                          \
    do {                                                               \
        if constexpr (kSmall) {                                        \
            if (one_tile) { TQ_LAUNCH_MANY_AS(B, UU, 1, true); break; } \
        }                                                              \
        if (part) TQ_LAUNCH_MANY_AS(B, UU, 2, (B == 4));               \
        else TQ_LAUNCH_MANY_AS(B, UU, 2, false);                       \
    } while (0)
    switch (g.bits) {
        case 2: if (N <= 32) TQ_LAUNCH_MANY(2, 32); else TQ_LAUNCH_MANY(2, 64); break;
        case 3: if (N <= 32) TQ_LAUNCH_MANY(3, 32); else TQ_LAUNCH_MANY(3, 64); break;
        default:
            if (N <= 16) TQ_LAUNCH_MANY(4, 16);
            else if (N <= 32) TQ_LAUNCH_MANY(4, 32);
            else TQ_LAUNCH_MANY(4, 64);
            break;
    }
#undef TQ_LAUNCH_MANY
#undef TQ_LAUNCH_MANY_READ
#undef TQ_LAUNCH_MANY_AS
    return hipGetLastError();
}

}  // namespace

// Host side of tq_decompress_aggregate and tq_decompress_aggregate_update after the argument
// checks of the C entry points.  mode: 0 store, 1 accumulate, 2 SGD step on `out` (= theta),
// 3 the same with the velocity buffer.
hipError_t tq_launch_decode(const void* const* payload, const tq_params_t* const* params,
                            const float* weights, int N, uint64_t d, uint64_t bucket_elems, int bits,
                            int mode, float eta, float momentum, float weight_decay, float* velocity,
                            float* out, hipStream_t st)
{
    DecodeGeom g;
    for (int i = 0; i < TQ_MAX_WORKERS; ++i) {
        g.args.payload[i] = i < N ? static_cast<const uint8_t*>(payload[i]) : nullptr;
        g.args.params[i] = i < N ? params[i] : nullptr;
        g.args.weight[i] = (i < N && weights) ? weights[i] : 0.0f;
    }
    g.N = N;
    g.bits = bits;
    g.weighted = weights ? 1 : 0;
    g.scale = 1.0f / (float)N;
    g.d = d;
    g.d_pad = (d + 127) / 128 * 128;
    g.be = bucket_elems ? bucket_elems : g.d_pad;
    g.nb = (g.d_pad + g.be - 1) / g.be;
    g.tpb = (g.be + tq::kTile - 1) / tq::kTile;                        // tiles per bucket
    g.pbytes = tq_payload_bytes(d, bits);
    const tq::Update up{eta, momentum, weight_decay, velocity};
    if (mode == tq::kStore && streams_output(d)) mode = tq::kStoreStream;
    else if (tq::reads_back(mode) && reads_past(mode, d, (uint64_t)N * g.pbytes, g.be)) mode |= tq::kPast;
    switch (mode) {
        case tq::kStore: return launch_mode<tq::kStore>(g, out, up, st);
        case tq::kStoreStream: return launch_mode<tq::kStoreStream>(g, out, up, st);
        case tq::kAccumulate: return launch_mode<tq::kAccumulate>(g, out, up, st);
        case tq::kSgd: return launch_mode<tq::kSgd>(g, out, up, st);
        case tq::kSgdMomentum: return launch_mode<tq::kSgdMomentum>(g, out, up, st);
        case tq::kAccumulate | tq::kPast: return launch_mode<tq::kAccumulate | tq::kPast>(g, out, up, st);
        case tq::kSgd | tq::kPast: return launch_mode<tq::kSgd | tq::kPast>(g, out, up, st);
        case tq::kSgdMomentum | tq::kPast: return launch_mode<tq::kSgdMomentum | tq::kPast>(g, out, up, st);
        default: return hipErrorInvalidValue;
    }
}


// Host side of tq_decompress_aggregate_segments after the argument checks of the C entry point.
hipError_t tq_launch_decode_segments(const void* const* payload, const tq_params_t* const* params,
                                     const float* weights, int N, uint64_t d, const uint64_t* seg_off,
                                     const uint64_t* seg_host, uint64_t nseg, int bits, int accumulate, float* out,
                                     hipStream_t st)
{
    const tq::SegHints hints = tq::make_seg_hints(seg_host, nseg, d);
    tq::DecodeArgs args;
    for (int i = 0; i < TQ_MAX_WORKERS; ++i) {
        args.payload[i] = i < N ? static_cast<const uint8_t*>(payload[i]) : nullptr;
        args.params[i] = i < N ? params[i] : nullptr;
        args.weight[i] = (i < N && weights) ? weights[i] : 0.0f;
    }
    const uint64_t d_pad = (d + 127) / 128 * 128;
    const uint64_t nblocks = (d + tq::kTile - 1) / tq::kTile;
    dim3 blocks;
    if (nseg > 0xFFFFFFFFull || !tq::fold_grid(nblocks, tq::kBlock, 1, blocks)) return hipErrorInvalidValue;
    const uint64_t pbytes = tq_payload_bytes(d, bits);
    const tq::Update up{0.0f, 0.0f, 0.0f, nullptr};
    const float scale = 1.0f / (float)N;
    const int weighted = weights ? 1 : 0;
    const dim3 threads(tq::kBlock);
    if (N <= 16 && !(bits == 4 && N > 8)) {
        // the bucketed kernel's code with the segments' records: two tiles per workgroup wherever they fall
        constexpr int T = 2;
        const int U = N <= 1 ? 1 : (N <= 2 ? 2 : (N <= 4 ? 4 : (N <= 8 ? 8 : 16)));
        dim3 fblocks;
        if (!tq::fold_grid((d + (uint64_t)T * tq::kTile - 1) / ((uint64_t)T * tq::kTile), tq::kBlock, 1, fblocks))
            return hipErrorInvalidValue;
#define TQ_LAUNCH_FSEG(B, UU, M)                                                                                  \
    hipLaunchKernelGGL((tq::tq_decode_fast_kernel<B, UU, T, M, true, false>), fblocks, threads, 0, st, args, N, weighted, \
                       scale, d, d_pad, (uint64_t)0, 0u, pbytes, out, up, seg_off, (uint32_t)nseg, hints)
        const bool stream = streams_output(d);
#define TQ_LAUNCH_FSEG_M(B, UU)                               \
    if (accumulate) TQ_LAUNCH_FSEG(B, UU, tq::kAccumulate);   \
    else if (stream) TQ_LAUNCH_FSEG(B, UU, tq::kStoreStream); \
    else TQ_LAUNCH_FSEG(B, UU, tq::kStore)
#define TQ_LAUNCH_FSEG_U(B)                          \
    switch (U) {                                     \
        case 1: TQ_LAUNCH_FSEG_M(B, 1); break;       \
        case 2: TQ_LAUNCH_FSEG_M(B, 2); break;       \
        case 4: TQ_LAUNCH_FSEG_M(B, 4); break;       \
        case 8: TQ_LAUNCH_FSEG_M(B, 8); break;       \
        default: TQ_LAUNCH_FSEG_M(B, 16); break;     \
    }
        switch (bits) {
            case 2: TQ_LAUNCH_FSEG_U(2) break;
            case 3: TQ_LAUNCH_FSEG_U(3) break;
            default:
                switch (U) {
                    case 1: TQ_LAUNCH_FSEG_M(4, 1); break;
                    case 2: TQ_LAUNCH_FSEG_M(4, 2); break;
                    case 4: TQ_LAUNCH_FSEG_M(4, 4); break;
                    default: TQ_LAUNCH_FSEG_M(4, 8); break;
                }
                break;
        }
#undef TQ_LAUNCH_FSEG_U
#undef TQ_LAUNCH_FSEG_M
#undef TQ_LAUNCH_FSEG
        return hipGetLastError();
    }
#define TQ_LAUNCH_DSEG(B, M)                                                                                   \
    hipLaunchKernelGGL((tq::tq_decode_segments_kernel<B, M>), blocks, threads, 0, st, args, N, weighted, scale, \
                       d, d_pad, seg_off, (uint32_t)nseg, hints, pbytes, out, up)
#define TQ_LAUNCH_DSEG_M(B) \
    if (accumulate) TQ_LAUNCH_DSEG(B, tq::kAccumulate); else TQ_LAUNCH_DSEG(B, tq::kStore)
    switch (bits) {
        case 2: TQ_LAUNCH_DSEG_M(2); break;
        case 3: TQ_LAUNCH_DSEG_M(3); break;
        default: TQ_LAUNCH_DSEG_M(4); break;
    }
#undef TQ_LAUNCH_DSEG_M
#undef TQ_LAUNCH_DSEG
    return hipGetLastError();
}

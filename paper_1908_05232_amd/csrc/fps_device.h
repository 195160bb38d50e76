// Device helpers shared by the step kernels of libfps (header-only so every
// translation unit inlines them; no relocatable device code is needed).
#pragma once

#include "fps_internal.h"

// Pointers read from memory are generic (flat) to the compiler; a cast to
// the global address space makes their loads and stores global_* ones, which
// wait on the vector-memory counter only.
template <class T>
__device__ __forceinline__ FPS_GLOBAL T* gmem(T* p)
{
    return (FPS_GLOBAL T*)p;
}

namespace fps {

// 8 and 16 bytes of global memory in one access
typedef float Float2 __attribute__((ext_vector_type(2)));
typedef double Double2 __attribute__((ext_vector_type(2)));
typedef int Int4 __attribute__((ext_vector_type(4)));
typedef unsigned UInt4 __attribute__((ext_vector_type(4)));

// Scenario owning flattened index g: the largest s with off[s] <= g (off has
// S + 1 entries, non-decreasing).  Called with wave-uniform arguments.
__device__ __forceinline__ int find_scenario(const int* off, int S, int g)
{
    int lo = 0, hi = S - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The scenario record of a step kernel.  A launch that holds one scenario
// reads it from its kernel arguments (one round of dependent loads fewer than
// the device table the ensemble launches read).
template <bool kOne>
__device__ __forceinline__ const Scn& scn_at(const Batch& B, int sc)
{
    if constexpr (kOne) return B.one;
    else return B.scn[sc];
}

// Inclusive prefix sum over the 64 lanes of a wave by DPP lane moves (VALU
// only): shifts by 1, 2, 4 and 8 within each row of 16 lanes (lanes without a
// source add 0), then the row broadcasts of lanes 15 and 31 carry the row
// totals into the rows above.  Integer, so the result is exact.
__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
    return v;
}

// A step whose flood update is skipped: either it is the identity (nothing
// is wet, no inflow enters during the step, and the state already came out of
// a flood update, so dry cells carry no discharge; the 1 s dry step of sec. 3
// then only advances the pedestrians), or the flood is held by the caller
// (fps_set_flood_frozen: the pedestrians walk on a flood state set from
// outside).  Every kernel of the step evaluates this on the same device state
// before the finalize changes it.
__device__ __forceinline__ bool flood_skipped(int frozen, int settled, int any_wet, float inc)
{
    return frozen || (settled && !any_wet && inc == 0.0f);
}
template <class St>      // DevState, in global memory or LDS
__device__ __forceinline__ bool flood_skipped(const St* st)
{
    return flood_skipped(st->frozen, st->settled, st->any_wet, st->inc);
}

// What the kernels of a step ask the state first (wave-uniform).  All words are
// here before any is looked at: left to itself the compiler loads each where a
// branch needs it, a load and a wait at a time, and a kernel of a small grid
// is little else than its chain of waits (the march, the pedestrian step and the
// order of its loads: 512^2 with 2,000 people 23.2 -> 22.5 us a step).
struct StepState {
    int active, cur, any_wet, settled, frozen, done;
    float dt, inc;
    __device__ __forceinline__ bool skipped() const { return flood_skipped(frozen, settled, any_wet, inc); }
};
__device__ __forceinline__ StepState step_state(const FPS_GLOBAL DevState* st)
{
    StepState s{st->active, st->cur, st->any_wet, st->settled, st->frozen, st->done, st->dt, st->inc};
    int dt = __builtin_bit_cast(int, s.dt), inc = __builtin_bit_cast(int, s.inc);
    s.active = __builtin_amdgcn_readfirstlane(s.active);
    s.cur = __builtin_amdgcn_readfirstlane(s.cur);
    s.any_wet = __builtin_amdgcn_readfirstlane(s.any_wet);
    s.settled = __builtin_amdgcn_readfirstlane(s.settled);
    s.frozen = __builtin_amdgcn_readfirstlane(s.frozen);
    s.done = __builtin_amdgcn_readfirstlane(s.done);
    dt = __builtin_amdgcn_readfirstlane(dt);
    inc = __builtin_amdgcn_readfirstlane(inc);
    asm("" : "+s"(s.active), "+s"(s.cur), "+s"(s.any_wet), "+s"(s.settled), "+s"(s.frozen), "+s"(s.done),
                 "+s"(dt), "+s"(inc));
    s.dt = __builtin_bit_cast(float, dt);
    s.inc = __builtin_bit_cast(float, inc);
    return s;
}

// A parameter record by value, all of its words loaded before any is used (the
// same for the record itself: at most five vectors of 16 words).
template <class T>
__device__ __forceinline__ T all_at_once(const T& record)
{
    typedef uint32_t Words __attribute__((ext_vector_type(16)));
    constexpr int N = (sizeof(T) + 63) / 64;
    static_assert(N >= 1 && N <= 5 && sizeof(T) % 4 == 0, "what fits the scalar registers");
    Words w[5] = {};
    __builtin_memcpy(w, &record, sizeof(T));
    if constexpr (N == 1) asm("" : "+s"(w[0]));
    if constexpr (N == 2) asm("" : "+s"(w[0]), "+s"(w[1]));
    if constexpr (N == 3) asm("" : "+s"(w[0]), "+s"(w[1]), "+s"(w[2]));
    if constexpr (N == 4) asm("" : "+s"(w[0]), "+s"(w[1]), "+s"(w[2]), "+s"(w[3]));
    if constexpr (N == 5) asm("" : "+s"(w[0]), "+s"(w[1]), "+s"(w[2]), "+s"(w[3]), "+s"(w[4]));
    T out;
    __builtin_memcpy(&out, w, sizeof(T));
    return out;
}

// Exclusive scan of the bin histogram by one block of kScanThreads: tiles of
// 16 * kScanThreads counts, sixteen consecutive counts per lane (four 16-byte
// loads), a wave scan and a scan of the wave totals per tile.  The counts of
// up to four tiles are loaded in one round before any of them is scanned (a
// round per tile made the scan of a large grid a chain of dependent loads);
// the histogram is cleared behind the loads for the next step.
__device__ inline void block_scan_bins(const BinParams& b)
{
    constexpr int IPT = 16, TILES = 4, TILE = IPT * kScanThreads;
    __shared__ int wtot[kScanThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x >> 6;
    int carry = 0;     // bins before the current tile (uniform)
    for (int base = 0; base < b.nbins; base += TILES * TILE) {
        int v[TILES][IPT];
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int k0 = base + t * TILE + IPT * threadIdx.x;
            if (k0 + IPT <= b.nbins) {
#pragma unroll
                for (int q = 0; q < IPT / 4; ++q) {
                    const Int4 w = *(FPS_GLOBAL const Int4*)&b.bin_count[k0 + 4 * q];
                    v[t][4 * q] = w.x; v[t][4 * q + 1] = w.y; v[t][4 * q + 2] = w.z; v[t][4 * q + 3] = w.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < IPT; ++e) v[t][e] = k0 + e < b.nbins ? b.bin_count[k0 + e] : 0;
            }
        }
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int k0 = base + t * TILE + IPT * threadIdx.x;
            if (k0 + IPT <= b.nbins) {
#pragma unroll
                for (int q = 0; q < IPT / 4; ++q)
                    *(FPS_GLOBAL Int4*)&b.bin_count[k0 + 4 * q] = Int4{0, 0, 0, 0};
            } else {
                for (int e = 0; e < IPT; ++e)
                    if (k0 + e < b.nbins) b.bin_count[k0 + e] = 0;
            }
        }
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            if (base + t * TILE >= b.nbins) break;      // uniform
            const int k0 = base + t * TILE + IPT * threadIdx.x;
            int tsum = 0;
#pragma unroll
            for (int e = 0; e < IPT; ++e) tsum += v[t][e];
            const int incl = wave_inclusive_scan(tsum);
            if (lane == kWave - 1) wtot[wid] = incl;
            __syncthreads();
            int wbase = 0, total = 0;
            for (int w = 0; w < kScanThreads / kWave; ++w) {
                const int x = wtot[w];
                wbase += w < wid ? x : 0;
                total += x;
            }
            int run = carry + wbase + incl - tsum;
            if (k0 + IPT <= b.nbins) {
#pragma unroll
                for (int q = 0; q < IPT / 4; ++q) {
                    Int4 w;
                    w.x = run; run += v[t][4 * q];
                    w.y = run; run += v[t][4 * q + 1];
                    w.z = run; run += v[t][4 * q + 2];
                    w.w = run; run += v[t][4 * q + 3];
                    *(FPS_GLOBAL Int4*)&b.bin_start[k0 + 4 * q] = w;
                }
            } else {
                for (int e = 0; e < IPT; ++e) {
                    if (k0 + e < b.nbins) b.bin_start[k0 + e] = run;
                    run += v[t][e];
                }
            }
            carry += total;
            __syncthreads();      // wtot is rewritten by the next tile
        }
    }
    if (threadIdx.x == 0) b.bin_start[b.nbins] = carry;
    __syncthreads();
}

// The first half of the multi-block bin scan: the count of chunk c, by one wave
// (sixteen 16-byte loads a lane, all out before the first wait).  A block of the
// end of step counts sixteen chunks: few of them fit a CU beside its registers,
// and with a block a chunk the end of step of 32 grids of 2048^2 cells (2,048
// chunks) took 28.7 us, against 10 so.
constexpr int kChunkWaves = kScanThreads / kWave;
__device__ __forceinline__ void wave_chunk_sum(const BinParams b, int c)
{
    constexpr int kPer = kChunkBins / (4 * kWave);
    const int lane = threadIdx.x & (kWave - 1), k0 = c * kChunkBins + 4 * lane;
    int t = 0;
    if (b.nbins - c * kChunkBins >= kChunkBins) {
        Int4 w[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) w[u] = *(FPS_GLOBAL const Int4*)&b.bin_count[k0 + 4 * kWave * u];
#pragma unroll
        for (int u = 0; u < kPer; ++u) t += w[u].x + w[u].y + w[u].z + w[u].w;
    } else {
        // the last chunk: clamped loads, so that they too go out together
#pragma unroll 16
        for (int u = 0; u < 4 * kPer; ++u) {
            const int k = c * kChunkBins + kWave * u + lane, n = b.bin_count[min(k, b.nbins - 1)];
            t += k < b.nbins ? n : 0;
        }
    }
    const int incl = wave_inclusive_scan(t);
    if (lane == kWave - 1) b.csum[c] = incl;
}

// Placement of the agents into their bins by rank, then the stable order: an
// agent's final slot counts the smaller ids of its own bin.  Whole-grid
// version, in two kernels (one thread per agent).  An agent alone in its bin
// (most of them in a sparse crowd) takes the bin's first slot in the
// placement pass; the others are marked (slot -1) for the order pass, which
// passes over everyone else after reading their slot and key (both read in
// agent order, no bin bounds).
__device__ inline void place_agent(const BinParams& b, int a)
{
    const int k = b.key[a], r = b.rank[a];
    const float x = b.x[a], y = b.y[a];
    if (k < 0) return;
    const int s0 = b.bin_start[k], s1 = b.bin_start[k + 1];
    if (s1 - s0 > 1) {
        b.perm_u[s0 + r] = a;
        b.slot[a] = -1;
    } else {
        b.slot[a] = s0;
        *(FPS_GLOBAL Float2*)&b.xy[s0] = Float2{x, y};
    }
}
__device__ inline void sort_agent(const BinParams& b, int a)
{
    const int k = b.key[a], sl = b.slot[a];
    if (k < 0 || sl >= 0) return;
    const int s0 = b.bin_start[k], s1 = b.bin_start[k + 1];
    int below = 0;
    for (int s = s0; s < s1; ++s) below += b.perm_u[s] < a;
    const int f = s0 + below;
    b.slot[a] = f;
    *(FPS_GLOBAL Float2*)&b.xy[f] = Float2{b.x[a], b.y[a]};
}

// Binning in LDS (at most kLdsAgents agents and kLdsBins bins), run by blocks of
// their own beside the end-of-step state update, one for every kLdsTile bins.
// A block starts from the agents' bin keys alone: the agents in the bins before
// its own (counted from the keys: no block waits for another), a histogram by
// LDS atomics, the exclusive scan, the placement by LDS atomics and the stable
// order by id; only the results are stored.  Being a function of the keys, it
// gives the same bins however often it runs on them (a scenario that did not
// step keeps its bins).  Same results as the global binning.
// A count, a start and an agent's number here are at most kLdsAgents, so bins
// are held two to a word and agents in 16 bits: at most 48 KB.  Bound by the
// chain keys - histogram - scan - placement - order, in one launch that the
// state update needs anyway.  Measured, a step of one centre of 576^2 / 724^2 /
// 1024^2 / 1400^2 cells with 2,000 to 3,000 people: 21.5 / 23.5 / 28.0 / 33.4 us; with one
// block for all bins 21.6 / 24.5 / 31.8 (and four launches, 45.2, beyond 65,536 bins); with the global
// histogram scanned and placed by one block, or beyond 32,768 bins by four
// launches, 36.7 / 43.6 / 48.5 (about 2 of the difference are the flood march's).
__device__ __forceinline__ void lds_bins_build(const BinParams b, int tile)      // by value: not reloaded after the stores
{
    constexpr int APT = kLdsAgents / kScanThreads, W = kScanThreads / kWave;
    static_assert(kLdsTile == 16 * kScanThreads && W == 16, "sixteen bins a thread, a wave total a lane of a row");
    extern __shared__ uint4 fin_lds4[];
    const int base = tile * kLdsTile, nb = min(b.nbins - base, kLdsTile);      // the block's bins
    uint32_t* lb = reinterpret_cast<uint32_t*>(fin_lds4);      // halves [nb]: counts, then starts, then ends
    const int nw = lds_bin_words(nb);
    uint16_t* lp = reinterpret_cast<uint16_t*>(lb + nw);       // the block's agents by bin, unordered
    __shared__ int wtot[W], wbelow[W];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x >> 6;
    int key[APT];      // within the block's bins, or -1
    float ax[APT], ay[APT];
    int below = 0;     // agents of the wave in bins before the block's
#pragma unroll
    for (int q = 0; q < APT; ++q) {
        const int a = threadIdx.x + q * kScanThreads;
        key[q] = -1;
        if (a < b.na) {
            key[q] = b.key[a];
            ax[q] = b.x[a];
            ay[q] = b.y[a];
        }
    }
    for (int v = threadIdx.x; v < nw / 4; v += kScanThreads) fin_lds4[v] = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < APT; ++q) {
        below += __popcll(__ballot(key[q] >= 0 && key[q] < base));
        key[q] = key[q] >= base && key[q] - base < nb ? key[q] - base : -1;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < APT; ++q)
        if (key[q] >= 0) atomicAdd(&lb[key[q] >> 1], 1u << (key[q] & 1) * 16);
    __syncthreads();
    // sixteen bins a thread; vectors past the last bin count nothing
    const int k0 = 16 * (int)threadIdx.x, v0 = k0 / 8;
    uint32_t hist[8];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint4 w = v0 + q < nw / 4 ? fin_lds4[v0 + q] : make_uint4(0, 0, 0, 0);
        hist[4 * q] = w.x; hist[4 * q + 1] = w.y; hist[4 * q + 2] = w.z; hist[4 * q + 3] = w.w;
    }
    int own = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) own += (int)(hist[e] & 0xffffu) + (int)(hist[e] >> 16);
    const int incl = wave_inclusive_scan(own);
    if (lane == kWave - 1) {
        wtot[wid] = incl;
        wbelow[wid] = below;
    }
    __syncthreads();
    // the waves' totals: one a lane, scanned within the row of sixteen lanes
    const int tot = wave_inclusive_scan(wtot[lane & (W - 1)]);
    const int carry = __builtin_amdgcn_readlane(wave_inclusive_scan(wbelow[lane & (W - 1)]), W - 1);
    const int total = __builtin_amdgcn_readlane(tot, W - 1);
    int run = incl - own + (wid > 0 ? __builtin_amdgcn_readlane(tot, max(wid - 1, 0)) : 0);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t h = hist[4 * q + e];
            w[e] = (uint32_t)run;
            run += (int)(h & 0xffffu);
            w[e] |= (uint32_t)run << 16;
            run += (int)(h >> 16);
        }
        if (v0 + q < nw / 4) fin_lds4[v0 + q] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    if (threadIdx.x == 0 && base + nb == b.nbins) b.bin_start[b.nbins] = carry + total;
    __syncthreads();
    // unordered placement: each agent takes the next free slot of its bin;
    // afterwards half k is the end of bin k (= start of bin k + 1)
#pragma unroll
    for (int q = 0; q < APT; ++q) {
        if (key[q] < 0) continue;
        const int sh = (key[q] & 1) * 16;
        const uint32_t was = atomicAdd(&lb[key[q] >> 1], 1u << sh);
        lp[was >> sh & 0xffffu] = (uint16_t)(threadIdx.x + q * kScanThreads);
    }
    __syncthreads();
    // the starts, four bins a lane and whole lines a wave: stored by the thread
    // that scanned them, every lane's sixteen bytes are a request of their own
    // (65,536 bins by one block: 17.2 us a launch against 13.3)
    for (int v = threadIdx.x; v < (nb + 3) / 4; v += kScanThreads) {
        const uint32_t w0 = v > 0 ? lb[2 * v - 1] >> 16 : 0u, w1 = lb[2 * v], w2 = lb[2 * v + 1];
        const Int4 st = {carry + (int)w0, carry + (int)(w1 & 0xffffu), carry + (int)(w1 >> 16), carry + (int)(w2 & 0xffffu)};
        if (4 * v + 4 <= nb) {
            *(FPS_GLOBAL Int4*)&b.bin_start[base + 4 * v] = st;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (4 * v + e < nb) b.bin_start[base + 4 * v + e] = st[e];
        }
    }
    // stable order: an agent's slot counts the smaller ids of its bin
    auto end = [&](int k) { return (int)(lb[k >> 1] >> (k & 1) * 16 & 0xffffu); };
#pragma unroll
    for (int q = 0; q < APT; ++q) {
        const int k = key[q];
        if (k < 0) continue;
        const int a = threadIdx.x + q * kScanThreads;
        const int s0 = k > 0 ? end(k - 1) : 0, s1 = end(k);
        int smaller = 0;
        for (int s = s0; s < s1; ++s) smaller += lp[s] < a;
        const int f = carry + s0 + smaller;
        b.slot[a] = f;
        *(FPS_GLOBAL Float2*)&b.xy[f] = Float2{ax[q], ay[q]};
    }
}

}  // namespace fps

// Scan building blocks shared by the scan kernels: the tile layout, loading,
// scanning and storing a tile, and the look-back over other tiles' descriptors.
#pragma once

#include "kcommon.hpp"
#include "kepoch.hpp"

#ifndef SKEL_SCAN_WAVES
#define SKEL_SCAN_WAVES 16
#endif

namespace skel {
namespace dev {

constexpr uint32_t kSpinLimit = 1u << 22;
constexpr int kFlatPerLane = 8;  // S5: descriptors each lane reads per round
// polls (about 1 us each) before a flat tile computes the totals it still misses
// itself; a test build sets it to 1
#ifndef SKEL_FLAT_PATIENCE
#define SKEL_FLAT_PATIENCE 1024
#endif
constexpr uint32_t kFlatPatience = SKEL_FLAT_PATIENCE;

// ALIGNED: the data starts 16-byte aligned; otherwise (rows of a matrix) its
// vectors are accessed at element alignment, by the same instructions
template <int DIN, int DOUT, int OP, int WAVES = SKEL_SCAN_WAVES, bool ALIGNED = true>
struct SP {
    static constexpr bool kAligned = ALIGNED;
    using in_t = typename Stored<DIN>::type;
    using out_t = typename Stored<DOUT>::type;
    using acc_t = typename Acc<DIN, DOUT, OP>::type;
    using C = Comb<acc_t, OP>;
    static constexpr int E = 16 / sizeof(in_t);           // elements per lane per row
    static constexpr int R = sizeof(in_t) == 4 ? 8 : 16;  // rows per wavefront
    static constexpr int kWaveElems = kWave * E * R;      // 2048
    // wavefronts per workgroup: 16 for 4-byte inputs; 8 for 8-byte inputs,
    // whose raw rows need twice the registers
    static constexpr int NW = sizeof(in_t) == 4 ? WAVES : (WAVES > 1 ? WAVES / 2 : 1);
    static constexpr int kBlock = NW * kWave;
    static constexpr int64_t kTile = (int64_t)NW * kWaveElems;
};

// a 16-byte vector at element alignment
template <class T>
using VecAny = unsigned int __attribute__((ext_vector_type(4), aligned(sizeof(T))));

template <class T>
__device__ __forceinline__ void load16_any(const T* p, T (&v)[16 / sizeof(T)]) {
    u32x4 raw = __builtin_nontemporal_load(reinterpret_cast<const VecAny<T>*>(p));
    __builtin_memcpy(&v, &raw, 16);
}

template <class T, int E>
__device__ __forceinline__ void store_vecs_any(T* p, const T (&v)[E]) {
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) * E / 16); ++k) {
        u32x4 raw;
        __builtin_memcpy(&raw, reinterpret_cast<const char*>(&v) + 16 * k, 16);
        reinterpret_cast<VecAny<T>*>(p)[k] = raw;
    }
}

template <class P>
using Raw = typename P::in_t[P::R][P::E];

template <class P>
__device__ __forceinline__ int64_t lane_base(int64_t tile) {
    return tile * P::kTile + (int64_t)(threadIdx.x / kWave) * P::kWaveElems +
           (int64_t)lane() * P::E;
}

// Load the lane's share of `tile` (rows of 16-byte vectors); NT marks the
// loads non-temporal (input read once: measured a few percent faster for the
// single-pass scan).
template <class P, bool FULL, bool NT = false>
__device__ __forceinline__ void tile_load(const typename P::in_t* in, int64_t n, int64_t tile,
                                          Raw<P>& raw) {
    const int64_t b = lane_base<P>(tile);
#pragma unroll
    for (int r = 0; r < P::R; ++r) {
        const int64_t idx = b + (int64_t)r * kWave * P::E;
        if (FULL || idx + P::E <= n) {
            if constexpr (!P::kAligned) load16_any(in + idx, raw[r]);
            else if constexpr (NT) load16_nt(in + idx, raw[r]);
            else load16(in + idx, raw[r]);
        } else {
#pragma unroll
            for (int e = 0; e < P::E; ++e) raw[r][e] = idx + e < n ? in[idx + e] : 0;
        }
    }
}

// op over the lane's elements below n
template <class P, bool FULL>
__device__ __forceinline__ typename P::acc_t lane_total(int64_t n, int64_t tile,
                                                        const Raw<P>& raw) {
    using C = typename P::C;
    const int64_t b = lane_base<P>(tile);
    typename P::acc_t t = C::id();
#pragma unroll
    for (int r = 0; r < P::R; ++r)
#pragma unroll
        for (int e = 0; e < P::E; ++e)
            if (FULL || b + (int64_t)r * kWave * P::E + e < n)
                t = C::op(t, widen<typename P::acc_t>(raw[r][e]));
    return t;
}

// Compiler-only barrier on the raw inputs (emits no instruction): without it
// the compiler keeps the widened values of phase 1 alive across the tile wait
// to reuse them in the store phase, which doubles the live registers.
template <class P>
__device__ __forceinline__ void keep_raw_only(Raw<P>& raw) {
#pragma unroll
    for (int r = 0; r < P::R; ++r)
#pragma unroll
        for (int e = 0; e < P::E; ++e) asm volatile("" : "+v"(raw[r][e]));
}

// Scan the wavefront's slice given its exclusive prefix, and store it.  REV:
// the slice is combined from its last element down (the prefix then holds
// everything after the slice).
// Returns prefix op (the slice's elements below n).
template <class P, bool FULL, bool REV = false>
__device__ __forceinline__ typename P::acc_t tile_scan_store(typename P::out_t* out, int64_t n,
                                                             int64_t tile, const Raw<P>& raw,
                                                             typename P::acc_t prefix,
                                                             bool exclusive) {
    using acc_t = typename P::acc_t;
    using out_t = typename P::out_t;
    using C = typename P::C;
    constexpr int E = P::E;
    const int l = lane();
    const int64_t b = lane_base<P>(tile);
    acc_t running = prefix;
#pragma unroll
    for (int rr = 0; rr < P::R; ++rr) {
        const int r = REV ? P::R - 1 - rr : rr;
        const int64_t idx = b + (int64_t)r * kWave * E;
        acc_t loc[E];  // lane-local inclusive scan of the row vector (in scan order)
        acc_t t = C::id();
#pragma unroll
        for (int ee = 0; ee < E; ++ee) {
            const int e = REV ? E - 1 - ee : ee;
            const acc_t x = (FULL || idx + e < n) ? widen<acc_t>(raw[r][e]) : C::id();
            t = C::op(t, x);
            loc[e] = t;
        }
        const acc_t incl = REV ? wave_inclusive_suffix_scan<C>(t) : wave_inclusive_scan<C>(t);
        const acc_t tot = lane_value(incl, REV ? 0 : kWave - 1);
        const acc_t ex = REV ? wave_shift_down(incl, C::id()) : wave_shift_up(incl, C::id());
        const bool first = REV ? l == kWave - 1 : l == 0;
        const acc_t base = C::op(running, first ? C::id() : ex);
        out_t o[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int before = REV ? e + 1 : e - 1;  // previous element in scan order
            const bool none = REV ? e == E - 1 : e == 0;
            const acc_t v = exclusive ? (none ? base : C::op(base, loc[before]))
                                      : C::op(base, loc[e]);
            o[e] = (out_t)v;
        }
        if (FULL || idx + E <= n) {
            // plain stores: with a row's stores outstanding per lane they
            // stream faster than non-temporal ones (i32 -> i64 exclusive scan
            // of 2^27: 353 us against 417 us)
            if constexpr (P::kAligned) store_vecs<out_t, E>(out + idx, o);
            else store_vecs_any<out_t, E>(out + idx, o);
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (idx + e < n) out[idx + e] = o[e];
        }
        running = C::op(running, tot);
        // one row at a time: keeps the live registers to one row's temporaries
        // (interleaving rows would spill at 1024 lanes per workgroup)
        __builtin_amdgcn_sched_barrier(0);
    }
    return running;
}

// Wavefront totals -> LDS; returns (exclusive prefix of this wavefront within
// the tile, tile total) in every thread.  Contains one barrier.
template <class P, bool REV = false>
__device__ __forceinline__ void tile_totals(typename P::acc_t lane_t, typename P::acc_t* s_wtot,
                                            typename P::acc_t* wex, typename P::acc_t* agg) {
    using C = typename P::C;
    const int w = threadIdx.x / kWave;
    const typename P::acc_t wt = wave_reduce<C>(lane_t);
    if (lane() == 0) s_wtot[w] = wt;
    __syncthreads();
    *wex = C::id();
    *agg = C::id();
#pragma unroll
    for (int k = 0; k < P::NW; ++k) {
        const typename P::acc_t t = s_wtot[k];
        if (REV ? k > w : k < w) *wex = C::op(*wex, t);
        *agg = C::op(*agg, t);
    }
}

// --------------------------------------------------------- tile descriptors
// two self-validating words per tile (see tagged_put / tagged_get)
enum { ST_INVALID = 0, ST_AGG = 1, ST_PREFIX = 2 };

template <class A>
__device__ __forceinline__ void publish(u64* st, int64_t t, int state, A val, uint32_t epoch) {
    tagged_put(st + 2 * t, state, epoch, val);
}

// Run by one whole wavefront.  Publishes the tile total, finds the exclusive
// prefix of the tile from its predecessors' descriptors, publishes the
// inclusive prefix, and returns the exclusive prefix (in every lane).  Lane l
// inspects tile base - l; a descriptor once seen valid (AGG or PREFIX) is
// final for this call, so a retry re-reads only the lanes still invalid.
template <class P>
__device__ typename P::acc_t lookback(u64* status, int64_t tile, typename P::acc_t agg,
                                      uint32_t epoch, u64* err) {
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    const int l = lane();
    if (tile == 0) {
        if (l == 0) publish(status, 0, ST_PREFIX, agg, epoch);
        return C::id();
    }
    if (l == 0) publish(status, tile, ST_AGG, agg, epoch);
    acc_t excl = C::id();
    int64_t base = tile - 1;
    uint32_t spins = 0;
    int s = ST_INVALID;
    acc_t val = C::id();
    while (true) {
        if (s == ST_INVALID) {
            const int64_t j = base - l;
            s = j >= 0 ? tagged_get(status + 2 * j, epoch, val) : ST_PREFIX;
            if (j < 0) val = C::id();
        }
        const u64 pre = __ballot(s == ST_PREFIX);
        const u64 inv = __ballot(s == ST_INVALID);
        const int p = pre ? __ffsll((long long)pre) - 1 : kWave;
        const u64 need = p >= kWave - 1 ? ~0ull : ((2ull << p) - 1);
        if (inv & need) {
            if (++spins > kSpinLimit) {
                if (l == 0) atomicOr(err, 1ull);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        excl = C::op(excl, wave_reduce<C>(l <= p ? val : C::id()));
        if (p < kWave) break;
        base -= kWave;
        s = ST_INVALID;
    }
    if (l == 0) publish(status, tile, ST_PREFIX, C::op(excl, agg), epoch);
    return excl;
}

// Flat look-back (S5, S3's middle sizes, row scans).  The tile is the workgroup
// index.  Each tile publishes its total, then every lane of the workgroup reads
// its share of the totals of all preceding tiles -- one round of parallel loads,
// re-reading only those not yet valid -- and the workgroup combines them.  A tile
// so waits for one publish-to-read latency, not for a chain of prefixes, and takes
// no ticket from an atomic counter (device-scope atomics on one word serialise, 12 ns
// each: 5000003 floats, 611 tiles, 10.2 us, 18.5 with a ticket).
// Nothing orders the workgroups of one launch across XCDs when another stream's
// kernels hold part of the device, so a preceding tile may not start while this
// one waits.  A lane whose patience ends therefore computes the total it misses
// from the input (flat_total), and the tile finishes; only the tile that advances
// the epoch then waits for every tile to have started, and the slots that all
// others leave let them.  The input must still be there: calls whose output
// overlaps it take a form with tile ids from a counter, but for S5, which then (and
// for few tiles) keeps waiting, bounded.

// The total of tile `seq` by one lane, in the steps of lane_total, wave_reduce and
// tile_totals (the same bits): a few milliseconds, for a tile that does not start.
// Nothing is published: a valid descriptor says that its tile has started.
template <class P, bool REV>
__device__ __forceinline__ typename P::acc_t flat_total(const typename P::in_t* in, int64_t n,
                                                        int64_t seq, int64_t ntiles) {
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    const int64_t tile = REV ? ntiles - 1 - seq : seq;
    acc_t agg = C::id();
#pragma unroll 1
    for (int w = 0; w < P::NW; ++w) {
        acc_t level[6], t = C::id();  // pending halves of the butterfly's tree
#pragma unroll 1
        for (int i = 0; i < kWave; ++i) {
            const int l = (int)(__builtin_bitreverse32((uint32_t)i) >> 26);
            const int64_t b = tile * P::kTile + (int64_t)w * P::kWaveElems + (int64_t)l * P::E;
            t = C::id();
#pragma unroll 1
            for (int k = 0; k < P::R * P::E; ++k) {
                const int64_t idx = b + (int64_t)(k / P::E) * kWave * P::E + k % P::E;
                if (idx < n) t = C::op(t, widen<acc_t>(in[idx]));
            }
#pragma unroll
            for (int v = 0; v < 6; ++v) {
                if (!((i >> v) & 1)) {
                    level[v] = t;
                    break;
                }
                t = C::op(level[v], t);
            }
        }
        agg = C::op(agg, t);
    }
    return agg;
}

// This lane's share of the totals of tiles 0 .. seq - 1.  missing: one was not there
// after the last poll, and RESCUE: was computed from the n elements of in, else left out.
template <class P, bool REV, bool RESCUE>
__device__ __forceinline__ typename P::acc_t flat_prefix(u64* status, int64_t seq,
                                                         uint32_t epoch,
                                                         const typename P::in_t* in, int64_t n,
                                                         int64_t ntiles, bool* missing) {
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    acc_t a = C::id();
    for (int64_t base = 0; base < seq; base += (int64_t)kFlatPerLane * P::kBlock) {
        acc_t v[kFlatPerLane];
        bool ready[kFlatPerLane];
#pragma unroll
        for (int k = 0; k < kFlatPerLane; ++k) {
            v[k] = C::id();
            ready[k] = base + k * P::kBlock + (int64_t)threadIdx.x >= seq;
        }
        uint32_t spins = 0;
        while (true) {
            bool all = true;
#pragma unroll
            for (int k = 0; k < kFlatPerLane; ++k) {
                if (ready[k]) continue;
                const int64_t j = base + k * P::kBlock + threadIdx.x;
                ready[k] = tagged_get(status + 2 * j, epoch, v[k]) != ST_INVALID;
                all = all && ready[k];
            }
            if (all) break;
            if (++spins > (RESCUE ? kFlatPatience : kSpinLimit)) {  // bounded
                *missing = true;
                if constexpr (RESCUE) {
#pragma unroll 1
                    for (int k = 0; k < kFlatPerLane; ++k) {
                        bool want = false;
#pragma unroll
                        for (int q = 0; q < kFlatPerLane; ++q) want = want || (q == k && !ready[q]);
                        if (!want) continue;
                        const acc_t t = flat_total<P, REV>(
                            in, n, base + k * P::kBlock + threadIdx.x, ntiles);
#pragma unroll
                        for (int q = 0; q < kFlatPerLane; ++q) {
                            v[q] = q == k ? t : v[q];
                            ready[q] = ready[q] || q == k;
                        }
                    }
                }
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int k = 0; k < kFlatPerLane; ++k) a = C::op(a, ready[k] ? v[k] : C::id());
    }
    return a;
}

// wavefronts per SIMD of the flat forms with the rescue: as many as without it
template <class P, bool RESCUE>
constexpr int flat_waves() {
    return !RESCUE ? 1 : sizeof(typename P::in_t) == 4 ? 4 : P::NW <= 1 ? 3 : 2;
}

// A flat tile: seq of ntiles in scan order, covering data tile `tile` of n elements;
// descriptors at status.  last: this workgroup advances the epoch, once every one of
// the `all` descriptors of the call (at `first`) has been seen valid: by then every
// tile has read this call's epoch.
template <class P, bool FULL, bool REV, bool RESCUE, bool ROWS>
__device__ __forceinline__ void flat_tile(const typename P::in_t* in, typename P::out_t* out,
                                          int64_t n, int64_t seq, int64_t tile, int64_t ntiles,
                                          int exclusive, u64* status, u64* sync, bool last,
                                          u64* first, int64_t all) {
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    __shared__ acc_t s_wtot[P::NW];
    __shared__ acc_t s_red[P::NW];
    __shared__ acc_t s_prefix;
    __shared__ uint32_t s_epoch;
    __shared__ int s_missing;
    uint32_t ep = 0;
    if (threadIdx.x == 0) ep = epoch_of_call(sync);  // in flight with the tile's loads
    Raw<P> raw;
    tile_load<P, FULL, true>(in, n, tile, raw);
    acc_t wex, agg;
    tile_totals<P, REV>(lane_total<P, FULL>(n, tile, raw), s_wtot, &wex, &agg);
    if (threadIdx.x == 0) {
        s_epoch = ep;
        if (RESCUE) s_missing = 0;
        if (!last) publish(status, seq, ST_AGG, agg, ep);
    }
    __syncthreads();
    bool missing = false;
    const acc_t part =
        flat_prefix<P, REV, RESCUE>(status, seq, s_epoch, in, n, ntiles, &missing);
    if (missing) {
        if (RESCUE) s_missing = 1;
        else atomicOr(sync + SYNC_ERROR, 1ull);
    }
    const acc_t pre = block_reduce<C>(part, s_red);
    // (block_reduce's barrier orders s_missing) every tile seen, if the call's are
    // this one's predecessors and none was missing
    const bool seen = last && !(RESCUE && s_missing) && (!ROWS || (status == first && seq == all));
    if (threadIdx.x == 0) {
        s_prefix = pre;
        if (seen) epoch_advance(sync);
    }
    __syncthreads();
    keep_raw_only<P>(raw);
    tile_scan_store<P, FULL, REV>(out, n, tile, raw, C::op(s_prefix, wex), exclusive != 0);
    if ((ROWS || RESCUE) && last && !seen) {
        bool expired = false;
        if constexpr (ROWS) {
            flat_prefix<P, REV, false>(first, all, s_epoch, in, n, ntiles, &expired);
        } else {
            // (only after a rescue: one descriptor after another, in little code)
            acc_t v;
#pragma unroll 1
            for (int64_t j = threadIdx.x; j < all; j += P::kBlock)
#pragma unroll 1
                for (uint32_t spins = 0;
                     tagged_get(first + 2 * j, s_epoch, v) == ST_INVALID && !expired;) {
                    expired = ++spins > kSpinLimit;
                    __builtin_amdgcn_s_sleep(1);
                }
        }
        if (expired) atomicOr(sync + SYNC_ERROR, 1ull);
        __syncthreads();
        if (threadIdx.x == 0) epoch_advance(sync);
    }
}

}  // namespace dev
}  // namespace skel

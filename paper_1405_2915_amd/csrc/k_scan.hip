// Scan skeleton kernels (Section III, scan): inclusive out[i] = x[0] op ...
// op x[i]; exclusive out[0] = identity, out[i] = x[0] op ... op x[i-1].  The
// reverse kinds combine from the end (out[i] = x[i] op ... op x[n-1], and its
// exclusive form); they are the adjoints of the forward sum scans and run in
// the single-pass variant, which visits tiles, rows, lanes and vector
// elements in descending order while keeping the ascending 16-byte layout.
//
// Tile layout (all variants): a workgroup of NW wavefronts (16, or 8 for 8-byte
// inputs) owns a tile of NW * 2048 elements; each wavefront owns a contiguous
// slice of 2048 and walks
// it in rows of 64 lanes x one 16-byte vector, so every load and store
// instruction of a wavefront covers one contiguous 1 KiB span (no LDS
// transposition).  Only the raw inputs stay in registers across the
// inter-tile wait: phase 1 needs just each lane's sum and one wavefront
// reduction to produce the tile total, and the row scans (a lane scans its
// own vector serially, the wavefront scans the 64 lane totals with lane
// shifts, rows are chained by a running carry) run after the tile's prefix is
// known.
//
// Variants:
//   S0  one workgroup walks all tiles in order carrying the prefix (small n)
//   S1  reduce-then-scan: tile totals, one workgroup scans the totals, then
//       every tile rescans with its offset (three launches, input read twice)
//   S2  single pass with decoupled look-back: each tile publishes its total
//       as soon as it has it, then wavefront 0 inspects the 64 preceding tile
//       descriptors at once and combines back to the nearest finished prefix;
//       on a retry only the descriptors that were not yet valid are re-read.
//       Tiles are numbered by an atomic counter in start order, so every tile
//       waited on is already resident: the wait always ends.
//   S4  S2 with tiles of two wavefronts (4096 elements for 4-byte inputs,
//       2048 for 8-byte): for arrays of a few million elements, whose 32768-
//       element tiles would leave most CUs idle (2^20 elements: 256 tiles
//       instead of 32)
//   S5  flat look-back over S4's tiles for arrays of at most 1024 of them:
//       tiles numbered by workgroup index, and each tile reads the totals of
//       all its predecessors in one round of parallel loads (no prefix chain,
//       no atomic counter)
//   S3  (middle sizes: the flat look-back of S5 on tiles of four wavefronts,
//       while the device holds them all at once, up to 2^23 elements; the
//       32768-element tiles below would leave CUs idle there: 5000003 floats are
//       153 tiles for 256 CUs, 14.3 us per scan against 11.5 flat, and 2^23
//       floats 17.7 against 15.1)
//       S2's tile step run by persistent workgroups (one per resident slot)
//       that loop over tile ids; a workgroup takes its next id once its
//       stores are issued, so no workgroup launch sits between one tile's
//       stores and the next tile's loads, and the counter's round trip
//       overlaps the stores' drain (2^27 i32 -> i64 exclusive: 310 us against
//       337 us for S2 on MI355X).
//
// Tile descriptors are self-validating tagged words (two per tile), written
// and read with single-copy-atomic device-scope accesses, so no fences and no
// clearing pass are needed; the host gives every call a fresh epoch.  The
// look-back wait is bounded: on expiry the kernel raises a flag that
// skel_sync reports, and finishes (with wrong values) instead of hanging.
#include <mutex>

#include "kscan.hpp"
#include "dispatch.hpp"
#include "launch.hpp"

namespace skel {
namespace {

using namespace dev;

// ------------------------------------------------------------------ kernels
// `seq` is the tile's position in scan order (descriptor index), `tile` the
// data tile it covers (they differ for the reverse kinds)
// s_next (persistent form only): thread 0 takes the workgroup's next tile id
// after issuing this tile's stores, so the counter's round trip overlaps their
// drain
template <class P, bool FULL, bool REV>
__device__ __forceinline__ void lookback_tile(const typename P::in_t* in,
                                              typename P::out_t* out, int64_t n, int64_t seq,
                                              int64_t tile, int exclusive, u64* status,
                                              u64* sync, uint32_t epoch,
                                              int64_t* s_next = nullptr) {
    using acc_t = typename P::acc_t;
    __shared__ acc_t s_wtot[P::NW];
    __shared__ acc_t s_prefix;
    Raw<P> raw;
    tile_load<P, FULL, true>(in, n, tile, raw);
    acc_t wex, agg;
    tile_totals<P, REV>(lane_total<P, FULL>(n, tile, raw), s_wtot, &wex, &agg);
    if (threadIdx.x < kWave) {
        const acc_t e = lookback<P>(status, seq, agg, epoch, sync + SYNC_ERROR);
        if (threadIdx.x == 0) s_prefix = e;
    }
    __syncthreads();
    keep_raw_only<P>(raw);
    tile_scan_store<P, FULL, REV>(out, n, tile, raw, P::C::op(s_prefix, wex), exclusive != 0);
    // the next id is taken only once this tile's stores are issued: an id held
    // longer delays the tiles after it, which wait on its descriptor (taking
    // it before the stores measured 3% slower, a whole tile ahead 34%)
    if (s_next != nullptr && threadIdx.x == 0)
        *s_next = (int64_t)atomicAdd(&sync[SYNC_TILE_COUNTER], 1ull);
}

template <class P, bool REV>
__global__ __launch_bounds__(P::kBlock) void scan_lookback(const typename P::in_t* in,
                                                        typename P::out_t* out, int64_t n,
                                                        int64_t ntiles, int exclusive,
                                                        u64* status, u64* sync) {
    __shared__ int64_t s_tile;
    __shared__ uint32_t s_epoch;
    if (threadIdx.x == 0) {
        s_epoch = epoch_of_call(sync);  // before taking a tile id (see below)
        const u64 t = atomicAdd(&sync[SYNC_TILE_COUNTER], 1ull);
        if (t == (u64)ntiles - 1)  // every other tile id has been taken
            __hip_atomic_store(&sync[SYNC_TILE_COUNTER], 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        s_tile = (int64_t)t;
    }
    __syncthreads();
    const int64_t seq = s_tile;
    const int64_t tile = REV ? ntiles - 1 - seq : seq;  // data tile in scan order
    const uint32_t epoch = s_epoch;
    if ((tile + 1) * P::kTile <= n)
        lookback_tile<P, true, REV>(in, out, n, seq, tile, exclusive, status, sync, epoch);
    else
        lookback_tile<P, false, REV>(in, out, n, seq, tile, exclusive, status, sync, epoch);
    // The workgroup that finishes last (every other one has passed its last
    // descriptor access) resets the counter and advances the epoch for the
    // next call.
    if (threadIdx.x == 0) {
        const u64 d = atomicAdd(&sync[SYNC_DONE], 1ull);
        if (d == (u64)ntiles - 1) {
            __hip_atomic_store(&sync[SYNC_DONE], 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            epoch_advance(sync);
        }
    }
}

// Persistent form: one workgroup per resident slot loops over tile ids taken
// from the counter (ids >= ntiles end the loop).  A tile waits only on tiles
// with smaller ids, all held by running workgroups that never wait on larger
// ids, so every wait ends.  Every workgroup takes exactly one id >= ntiles;
// the last one to leave has seen every tile finish and every id taken, so it
// resets the counters and advances the epoch.
template <class P, bool REV>
__global__ __launch_bounds__(P::kBlock) void scan_lookback_persist(
    const typename P::in_t* in, typename P::out_t* out, int64_t n, int64_t ntiles,
    int exclusive, u64* status, u64* sync) {
    __shared__ int64_t s_tile;
    __shared__ uint32_t s_epoch;
    if (threadIdx.x == 0) {
        s_epoch = epoch_of_call(sync);
        s_tile = (int64_t)atomicAdd(&sync[SYNC_TILE_COUNTER], 1ull);
    }
    __syncthreads();
    const uint32_t epoch = s_epoch;
    int64_t seq = s_tile;
    while (seq < ntiles) {
        const int64_t tile = REV ? ntiles - 1 - seq : seq;
        if ((tile + 1) * P::kTile <= n)
            lookback_tile<P, true, REV>(in, out, n, seq, tile, exclusive, status, sync, epoch,
                                        &s_tile);
        else
            lookback_tile<P, false, REV>(in, out, n, seq, tile, exclusive, status, sync, epoch,
                                         &s_tile);
        __syncthreads();
        seq = s_tile;
        __syncthreads();  // s_tile is rewritten during the next tile
    }
    if (threadIdx.x == 0) {
        const u64 d = atomicAdd(&sync[SYNC_DONE], 1ull);
        if (d == (u64)gridDim.x - 1) {
            __hip_atomic_store(&sync[SYNC_TILE_COUNTER], 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&sync[SYNC_DONE], 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            epoch_advance(sync);
        }
    }
}

template <class P, bool REV, bool RESCUE>
__global__ __launch_bounds__(P::kBlock, (flat_waves<P, RESCUE>())) void scan_flat(
    const typename P::in_t* in, typename P::out_t* out, int64_t n, int64_t ntiles, int exclusive,
    u64* status, u64* sync) {
    const int64_t seq = blockIdx.x;
    const int64_t tile = REV ? ntiles - 1 - seq : seq;  // data tile in scan order
    const bool last = seq == ntiles - 1;
    if ((tile + 1) * P::kTile <= n)
        flat_tile<P, true, REV, RESCUE, false>(in, out, n, seq, tile, ntiles, exclusive, status,
                                               sync, last, status, ntiles - 1);
    else
        flat_tile<P, false, REV, RESCUE, false>(in, out, n, seq, tile, ntiles, exclusive, status,
                                                sync, last, status, ntiles - 1);
}

// S1 pass 1: tile totals
template <class P, bool FULL>
__device__ __forceinline__ typename P::acc_t tile_sum(const typename P::in_t* in, int64_t n,
                                                      int64_t tile) {
    Raw<P> raw;
    tile_load<P, FULL>(in, n, tile, raw);
    return lane_total<P, FULL>(n, tile, raw);
}

template <class P>
__global__ __launch_bounds__(P::kBlock) void scan_tile_totals(const typename P::in_t* in, int64_t n,
                                                           typename P::acc_t* sums) {
    __shared__ typename P::acc_t lds[P::NW];
    const int64_t tile = blockIdx.x;
    typename P::acc_t a = (tile + 1) * P::kTile <= n ? tile_sum<P, true>(in, n, tile)
                                                     : tile_sum<P, false>(in, n, tile);
    a = block_reduce<typename P::C>(a, lds);
    if (threadIdx.x == 0) sums[tile] = a;
}

// S1 pass 2: exclusive scan of the tile totals, in place, by one workgroup
template <class P>
__global__ __launch_bounds__(1024) void scan_tile_offsets(typename P::acc_t* sums,
                                                          int64_t ntiles) {
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    constexpr int NW = 1024 / kWave;
    __shared__ acc_t lds[NW];
    const int w = threadIdx.x / kWave, l = lane();
    acc_t carry = C::id();
    for (int64_t base = 0; base < ntiles; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const acc_t v = i < ntiles ? sums[i] : C::id();
        const acc_t incl = wave_inclusive_scan<C>(v);
        if (l == kWave - 1) lds[w] = incl;
        __syncthreads();
        acc_t wex = C::id(), total = C::id();
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            if (k < w) wex = C::op(wex, lds[k]);
            total = C::op(total, lds[k]);
        }
        const acc_t lex = wave_shift_up(incl, C::id());
        if (i < ntiles) sums[i] = C::op(carry, C::op(wex, lex));
        carry = C::op(carry, total);
        __syncthreads();
    }
}

// S1 pass 3: rescan every tile with its offset
template <class P, bool FULL>
__device__ __forceinline__ void apply_tile(const typename P::in_t* in, typename P::out_t* out,
                                           int64_t n, int64_t tile, typename P::acc_t offset,
                                           int exclusive) {
    __shared__ typename P::acc_t s_wtot[P::NW];
    Raw<P> raw;
    tile_load<P, FULL>(in, n, tile, raw);
    typename P::acc_t wex, agg;
    tile_totals<P>(lane_total<P, FULL>(n, tile, raw), s_wtot, &wex, &agg);
    keep_raw_only<P>(raw);
    tile_scan_store<P, FULL>(out, n, tile, raw, P::C::op(offset, wex), exclusive != 0);
}

template <class P>
__global__ __launch_bounds__(P::kBlock) void scan_tile_apply(const typename P::in_t* in,
                                                          typename P::out_t* out, int64_t n,
                                                          const typename P::acc_t* offs,
                                                          int exclusive) {
    const int64_t tile = blockIdx.x;
    if ((tile + 1) * P::kTile <= n)
        apply_tile<P, true>(in, out, n, tile, offs[tile], exclusive);
    else
        apply_tile<P, false>(in, out, n, tile, offs[tile], exclusive);
}

// S0: one workgroup, tiles in order; the carry is held identically by every
// thread (it is combined from the same LDS totals)
template <class P, bool FULL>
__device__ __forceinline__ typename P::acc_t single_tile(const typename P::in_t* in,
                                                         typename P::out_t* out, int64_t n,
                                                         int64_t tile, typename P::acc_t carry,
                                                         int exclusive) {
    __shared__ typename P::acc_t s_wtot[P::NW];
    Raw<P> raw;
    tile_load<P, FULL>(in, n, tile, raw);
    typename P::acc_t wex, agg;
    tile_totals<P>(lane_total<P, FULL>(n, tile, raw), s_wtot, &wex, &agg);
    keep_raw_only<P>(raw);
    tile_scan_store<P, FULL>(out, n, tile, raw, P::C::op(carry, wex), exclusive != 0);
    __syncthreads();  // s_wtot is rewritten by the next tile
    return P::C::op(carry, agg);
}

template <class P>
__global__ __launch_bounds__(P::kBlock) void scan_single(const typename P::in_t* in,
                                                      typename P::out_t* out, int64_t n,
                                                      int64_t ntiles, int exclusive) {
    typename P::acc_t carry = P::C::id();
    for (int64_t tile = 0; tile < ntiles; ++tile) {
        if ((tile + 1) * P::kTile <= n) carry = single_tile<P, true>(in, out, n, tile, carry, exclusive);
        else carry = single_tile<P, false>(in, out, n, tile, carry, exclusive);
    }
}

// --------------------------------------------------------------- launchers
// S1's three launches; `sums` holds one accumulator per tile (written by the
// first launch before the others read it, so it needs no clearing)
template <class P>
skel_status reduce_then_scan(const typename P::in_t* in, typename P::out_t* out, int64_t n,
                             int excl, typename P::acc_t* sums, hipStream_t st) {
    const int64_t ntiles = (n + P::kTile - 1) / P::kTile;
    skel_status e;
    scan_tile_totals<P><<<(unsigned)ntiles, P::kBlock, 0, st>>>(in, n, sums);
    if ((e = launch_check("scan_tile_totals")) != SKEL_OK) return e;
    scan_tile_offsets<P><<<1, 1024, 0, st>>>(sums, ntiles);
    if ((e = launch_check("scan_tile_offsets")) != SKEL_OK) return e;
    scan_tile_apply<P><<<(unsigned)ntiles, P::kBlock, 0, st>>>(in, out, n, sums, excl);
    return launch_check("scan_tile_apply");
}

template <int DIN, int DOUT, int OP>
skel_status scan_typed(int v, int kind, const void* x, void* y, int64_t n, LaunchCtx& lc) {
    using P = SP<DIN, DOUT, OP>;
    using in_t = typename P::in_t;
    using out_t = typename P::out_t;
    using acc_t = typename P::acc_t;
    const in_t* in = static_cast<const in_t*>(x);
    out_t* out = static_cast<out_t*>(y);
    const int64_t ntiles = (n + P::kTile - 1) / P::kTile;
    const bool rev = kind == SKEL_REVERSE_INCLUSIVE || kind == SKEL_REVERSE_EXCLUSIVE;
    const int excl = (kind == SKEL_EXCLUSIVE || kind == SKEL_REVERSE_EXCLUSIVE) ? 1 : 0;
    hipStream_t st = lc.stream;
    // the output leaves the input in place: a flat tile may read it again
    const uintptr_t x0 = reinterpret_cast<uintptr_t>(x), y0 = reinterpret_cast<uintptr_t>(y);
    const bool apart = x0 + (uintptr_t)n * sizeof(in_t) <= y0 ||
                       y0 + (uintptr_t)n * sizeof(out_t) <= x0;
    if (rev && v != S2_LOOKBACK && v != S3_PERSISTENT_LOOKBACK && v != S4_SMALL_TILE_LOOKBACK &&
        v != S5_FLAT_LOOKBACK)
        return fail(SKEL_E_UNSUPPORTED, "reverse scans run in the single-pass variants only");
    if (v == S5_FLAT_LOOKBACK) {
        using PS = SP<DIN, DOUT, OP, 2>;
        static_assert(PS::kTile == scan_flat_tile(DIN), "S5 tile size known to the plan");
        const int64_t nts = (n + PS::kTile - 1) / PS::kTile;
        if (nts > kFlatMaxTiles)
            return fail(SKEL_E_UNSUPPORTED, "S5 takes at most %lld elements of this type",
                        (long long)(kFlatMaxTiles * PS::kTile));
        void* status = nullptr;
        skel_status e = ws_status(lc, (size_t)nts * 16, &status);
        if (e != SKEL_OK) return e;
        // up to two tiles per CU, which holds eight or more, the tiles of four
        // launches on as many streams (HIP runs four queues at once) are resident
        // together, and every wait ends without the means to compute a missing total
        // (binary32 2^20 5.3 us with them, 5.2 without; 557293 int64 9.8, 9.4)
        const bool few = nts <= 2 * (int64_t)lc.dev->cus;
        const auto kern =
            few || !apart ? (rev ? scan_flat<PS, true, false> : scan_flat<PS, false, false>)
                          : (rev ? scan_flat<PS, true, true> : scan_flat<PS, false, true>);
        kern<<<(unsigned)nts, PS::kBlock, 0, st>>>(in, out, n, nts, excl,
                                                   static_cast<u64*>(status), lc.ws->sync);
        return launch_check("scan_flat");
    }
    if (v == S4_SMALL_TILE_LOOKBACK) {
        using PS = SP<DIN, DOUT, OP, 2>;
        const int64_t nts = (n + PS::kTile - 1) / PS::kTile;
        void* status = nullptr;
        skel_status e = ws_status(lc, (size_t)nts * 16, &status);
        if (e != SKEL_OK) return e;
        if (rev)
            scan_lookback<PS, true><<<(unsigned)nts, PS::kBlock, 0, st>>>(
                in, out, n, nts, excl, static_cast<u64*>(status), lc.ws->sync);
        else
            scan_lookback<PS, false><<<(unsigned)nts, PS::kBlock, 0, st>>>(
                in, out, n, nts, excl, static_cast<u64*>(status), lc.ws->sync);
        return launch_check("scan_lookback_small");
    }
    switch (v) {
    case S0_SINGLE_WG:
        scan_single<P><<<1, P::kBlock, 0, st>>>(in, out, n, ntiles, excl);
        return launch_check("scan_single");
    case S1_REDUCE_THEN_SCAN: {
        void* mem = nullptr;
        skel_status e = ws_scratch(lc, (size_t)ntiles * sizeof(acc_t), &mem);
        if (e != SKEL_OK) return e;
        return reduce_then_scan<P>(in, out, n, excl, static_cast<acc_t*>(mem), st);
    }
    case S3_PERSISTENT_LOOKBACK: {
        // middle sizes: flat, while the device holds every tile at once; 8192
        // elements per tile.  (In place the tiles below, whose ids from a counter
        // make every wait end without reading the input again.)
        using PM = SP<DIN, DOUT, OP, DIN == SKEL_I64 ? 8 : 4>;
        const auto flat = rev ? scan_flat<PM, true, true> : scan_flat<PM, false, true>;
        const int64_t ntm = (n + PM::kTile - 1) / PM::kTile;
        const bool mid = apart && ntm <= kFlatMaxTiles &&
                         ntm <= resident_slots(reinterpret_cast<const void*>(flat), PM::kBlock, lc);
        void* status = nullptr;
        skel_status e = ws_status(lc, (size_t)(mid ? ntm : ntiles) * 16, &status);
        if (e != SKEL_OK) return e;
        if (mid) {
            flat<<<(unsigned)ntm, PM::kBlock, 0, st>>>(in, out, n, ntm, excl,
                                                       static_cast<u64*>(status), lc.ws->sync);
            return launch_check("scan_flat_mid");
        }
        auto kern = rev ? scan_lookback_persist<P, true> : scan_lookback_persist<P, false>;
        const int64_t slots = resident_slots(reinterpret_cast<const void*>(kern), P::kBlock, lc);
        if (slots < 1) return fail(SKEL_E_HIP, "scan_lookback_persist does not fit a CU");
        kern<<<(unsigned)std::min<int64_t>(ntiles, slots), P::kBlock, 0, st>>>(
            in, out, n, ntiles, excl, static_cast<u64*>(status), lc.ws->sync);
        return launch_check("scan_lookback_persist");
    }
    default: {  // S2_LOOKBACK
        void* status = nullptr;
        skel_status e = ws_status(lc, (size_t)ntiles * 16, &status);
        if (e != SKEL_OK) return e;
        if (rev)
            scan_lookback<P, true><<<(unsigned)ntiles, P::kBlock, 0, st>>>(
                in, out, n, ntiles, excl, static_cast<u64*>(status), lc.ws->sync);
        else
            scan_lookback<P, false><<<(unsigned)ntiles, P::kBlock, 0, st>>>(
                in, out, n, ntiles, excl, static_cast<u64*>(status), lc.ws->sync);
        return launch_check("scan_lookback");
    }
    }
}

template <int DIN, int DOUT>
skel_status scan_op(int v, int kind, int op, const void* x, void* y, int64_t n,
                    LaunchCtx& lc) {
    switch (op) {
    case SKEL_SUM: return scan_typed<DIN, DOUT, SKEL_SUM>(v, kind, x, y, n, lc);
    case SKEL_MIN: return scan_typed<DIN, DOUT, SKEL_MIN>(v, kind, x, y, n, lc);
    default: return scan_typed<DIN, DOUT, SKEL_MAX>(v, kind, x, y, n, lc);
    }
}

}  // namespace

skel_status launch_scan(int v, int kind, int op, skel_dtype din, skel_dtype dout,
                        const void* x, void* y, int64_t n, LaunchCtx& lc) {
    if (din == SKEL_I32 && dout == SKEL_I32) return scan_op<SKEL_I32, SKEL_I32>(v, kind, op, x, y, n, lc);
    if (din == SKEL_I32) return scan_op<SKEL_I32, SKEL_I64>(v, kind, op, x, y, n, lc);
    if (din == SKEL_I64) return scan_op<SKEL_I64, SKEL_I64>(v, kind, op, x, y, n, lc);
    return scan_op<SKEL_F32, SKEL_F32>(v, kind, op, x, y, n, lc);
}

}  // namespace skel

// ------------------------------------------------- allocation-free Scan ----
// skel_scan_noalloc runs S1 with its tile totals in a file-scope device array
// instead of the stream's workspace, so a call allocates nothing.  Every GPU
// the library runs on holds its own copy of the array (until the process
// ends); host code reaches it only through the address hipGetSymbolAddress
// returns with that device current, never through the array's name.
namespace skel {

constexpr int64_t kNoAllocTiles = 32768;  // tile totals the array holds (8 bytes each)
static __device__ __align__(256) unsigned long long scratch[kNoAllocTiles];  // 256 KiB

namespace {

constexpr int kNoAllocMaxDevices = 64;
void* g_scratch_addr[kNoAllocMaxDevices];  // per device ordinal
std::mutex g_scratch_mu;

skel_status scratch_address(int device, void** out) {
    if (device < 0 || device >= kNoAllocMaxDevices)
        return fail(SKEL_E_INVAL, "device %d beyond the %d the allocation-free scan tracks",
                    device, kNoAllocMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return fail(SKEL_E_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", device,
                        hipGetErrorString(e));
        }
        g_scratch_addr[device] = p;
    }
    *out = g_scratch_addr[device];
    return SKEL_OK;
}

template <int DIN, int DOUT, int OP>
skel_status noalloc_typed(const void* x, void* y, int64_t n, int excl, void* sums,
                          hipStream_t st) {
    using P = SP<DIN, DOUT, OP>;
    static_assert(sizeof(typename P::acc_t) <= sizeof(scratch[0]), "one array word per tile");
    return reduce_then_scan<P>(static_cast<const typename P::in_t*>(x),
                               static_cast<typename P::out_t*>(y), n, excl,
                               static_cast<typename P::acc_t*>(sums), st);
}

template <int DIN, int DOUT>
skel_status noalloc_op(int op, const void* x, void* y, int64_t n, int excl, void* sums,
                       hipStream_t st) {
    switch (op) {
    case SKEL_SUM: return noalloc_typed<DIN, DOUT, SKEL_SUM>(x, y, n, excl, sums, st);
    case SKEL_MIN: return noalloc_typed<DIN, DOUT, SKEL_MIN>(x, y, n, excl, sums, st);
    default: return noalloc_typed<DIN, DOUT, SKEL_MAX>(x, y, n, excl, sums, st);
    }
}

// the scan tile of an input type: what bounds n for a given array size
int64_t noalloc_tile(skel_dtype din) {
    return din == SKEL_I64 ? SP<SKEL_I64, SKEL_I64, SKEL_SUM>::kTile
                           : SP<SKEL_I32, SKEL_I32, SKEL_SUM>::kTile;
}

}  // namespace

skel_status scan_noalloc_setup(int device) {
    void* p = nullptr;
    return scratch_address(device, &p);
}

}  // namespace skel

using namespace skel;

extern "C" skel_status skel_scan_noalloc(const void* in, skel_dtype din, void* out,
                                         skel_dtype dout, int64_t n, skel_scan_kind kind,
                                         skel_reduce_op op, void* stream) {
    if (!rt().initialized) return fail(SKEL_E_NOINIT, "skel_init has not been called");
    if (kind == SKEL_REVERSE_INCLUSIVE || kind == SKEL_REVERSE_EXCLUSIVE)
        return fail(SKEL_E_UNSUPPORTED, "the allocation-free scan runs the forward kinds only");
    if (kind != SKEL_INCLUSIVE && kind != SKEL_EXCLUSIVE)
        return fail(SKEL_E_INVAL, "unknown scan kind %d", (int)kind);
    if (op < SKEL_SUM || op > SKEL_MAX) return fail(SKEL_E_INVAL, "unknown scan op %d", (int)op);
    const bool types_ok = (din == SKEL_I32 && (dout == SKEL_I32 || dout == SKEL_I64)) ||
                          (din == SKEL_I64 && dout == SKEL_I64) ||
                          (din == SKEL_F32 && dout == SKEL_F32);
    if (!types_ok)
        return fail(SKEL_E_DTYPE, "Scan %s -> %s not supported",
                    dtype_valid(din) ? dtype_name(din) : "?",
                    dtype_valid(dout) ? dtype_name(dout) : "?");
    if (n < 0) return fail(SKEL_E_INVAL, "negative element count %lld", (long long)n);
    if (n == 0) return SKEL_OK;
    const int64_t tile = noalloc_tile(din);
    if ((n + tile - 1) / tile > kNoAllocTiles)
        return fail(SKEL_E_SHAPE,
                    "n = %lld exceeds the allocation-free maximum of %lld elements for %s "
                    "input (%lld tiles of %lld)", (long long)n,
                    (long long)(kNoAllocTiles * tile), dtype_name(din),
                    (long long)kNoAllocTiles, (long long)tile);
    if (!in || !out) return fail(SKEL_E_INVAL, "null data pointer");
    if (reinterpret_cast<uintptr_t>(in) % 16 != 0 || reinterpret_cast<uintptr_t>(out) % 16 != 0)
        return fail(SKEL_E_INVAL, "in and out must be 16-byte aligned");
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(in), b0 = reinterpret_cast<uintptr_t>(out);
    const uintptr_t a1 = a0 + (uintptr_t)n * dtype_size(din);
    const uintptr_t b1 = b0 + (uintptr_t)n * dtype_size(dout);
    if (a0 < b1 && b0 < a1 && !(a0 == b0 && din == dout))
        return fail(SKEL_E_INVAL, "out must equal in (same types) or not overlap it");
    int device = -1;
    skel_status st = hip_check(hipGetDevice(&device), "hipGetDevice");
    if (st != SKEL_OK) return st;
    void* sums = nullptr;
    st = scratch_address(device, &sums);
    if (st != SKEL_OK) return st;
    const int excl = kind == SKEL_EXCLUSIVE ? 1 : 0;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (din == SKEL_I32 && dout == SKEL_I32)
        return noalloc_op<SKEL_I32, SKEL_I32>(op, in, out, n, excl, sums, s);
    if (din == SKEL_I32) return noalloc_op<SKEL_I32, SKEL_I64>(op, in, out, n, excl, sums, s);
    if (din == SKEL_I64) return noalloc_op<SKEL_I64, SKEL_I64>(op, in, out, n, excl, sums, s);
    return noalloc_op<SKEL_F32, SKEL_F32>(op, in, out, n, excl, sums, s);
}

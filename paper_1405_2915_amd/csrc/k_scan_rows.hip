// Row-wise Scan: every row of a rows x cols matrix scanned on its own (a batch of
// Scan instances of one length, Section III), in one launch for all rows.  Vectors
// are accessed at element alignment, so ragged rows cost no more instructions
// than aligned ones.  Forms, by shape:
//   short rows   up to 32 vectors, or 64 of many rows: 8, 16, 32 or 64 lanes per row, so
//                that a wavefront scans several rows at once, and four wavefronts share
//                a workgroup
//                (8-byte outputs in unaligned rows of 129 to 256 elements: one element
//                per lane, 64 at a time)
//   a wavefront  per row, walking it in chunks of as many vectors per lane as the
//                row needs (1, 2, 4 or 8 rows of 64 vectors) with a running carry;
//                the form for many rows
//   few rows     (fewer than 1024) of more than 4096 elements: a workgroup of four
//                wavefronts per row that it holds (8192 elements, 4096 of 8 bytes); one
//                of 16 per row (32768 and 16384) for at most one row per CU; longer
//                rows, up to one and a half per CU, are cut: binary32 sums into the
//                wavefront form's chunks in three launches that keep its order of
//                additions, everything else into tiles, with up to 1024 tiles of two
//                wavefronts in all the flat look-back within each row, otherwise tiles
//                of 16 wavefronts with the decoupled look-back
// All are HBM-bound once enough rows or tiles are in flight.  Measured, forward
// and reverse together, against one wavefront per row in chunks of 2048 elements
// (64-element chunks of single accesses where rows are not 16-byte aligned),
// binary32: 65536 x 20 117 -> 7 us, 20000 x 100 43 -> 9.2, 3000 x 1001 18.2 -> 11.3,
// 65536 x 512 121 -> 89 (6 TB/s), 900 x 5001 64 -> 20; 16384 x 2048 92.6 both (5.8
// TB/s).  Longer rows, binary32 / int32 (one call, whose 64-element form took 562, 161
// and 5149 us): 300 x 100001 66 / 56, 40 x 50001 12.4 / 9.1, 3 x 1000003 31.5 / 10.1.
// Where the lines lie (one call): a wavefront per row against 16 wavefronts, 256 x
// 20000 17.2 / 10.0 us, 300 x 20000 18.1 / 15.6, 700 x 20000 22.5 / 26.7, 300 x 9001 9.7
// / 13.8; against cut rows, 300 x 50001 41 / 36, 384 x 50001 42 / 44, 512 x 50001 44 / 55;
// int64 300 x 50001 80 / 59, 512 x 50001 86 / 92, 1000 x 5001 (in tiles) 20 / 33.
#include "kscan.hpp"
#include "dispatch.hpp"
#include "launch.hpp"

namespace skel {
namespace {

using namespace dev;

// one wavefront, RV * 256 elements per chunk
template <int DIN, int DOUT, int OP, int RV>
struct SPW : SP<DIN, DOUT, OP, 1, false> {
    using Base = SP<DIN, DOUT, OP, 1, false>;
    static constexpr int NW = 1;
    static constexpr int kBlock = kWave;
    static constexpr int R = RV * 256 / (kWave * Base::E);
    static constexpr int kWaveElems = kWave * Base::E * R;
    static constexpr int64_t kTile = kWaveElems;
};

template <class P, bool REV>
__global__ __launch_bounds__(kWave) void scan_rows_wave(const typename P::in_t* in,
                                                        typename P::out_t* out, int64_t rows,
                                                        int64_t cols, int exclusive) {
    using acc_t = typename P::acc_t;
    const int64_t nch = (cols + P::kTile - 1) / P::kTile;
    for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
        const typename P::in_t* src = in + row * cols;
        typename P::out_t* dst = out + row * cols;
        acc_t carry = P::C::id();
        for (int64_t q = 0; q < nch; ++q) {
            const int64_t ch = REV ? nch - 1 - q : q;
            Raw<P> raw;
            if ((ch + 1) * P::kTile <= cols) {
                tile_load<P, true, true>(src, cols, ch, raw);
                keep_raw_only<P>(raw);
                carry = tile_scan_store<P, true, REV>(dst, cols, ch, raw, carry, exclusive != 0);
            } else {
                tile_load<P, false, true>(src, cols, ch, raw);
                keep_raw_only<P>(raw);
                carry = tile_scan_store<P, false, REV>(dst, cols, ch, raw, carry, exclusive != 0);
            }
        }
    }
}

// inclusive scan within groups of G = 8, 16, 32 or 64 lanes (REV: from the group's
// last lane down): row-of-16 steps that stay inside the group, then for 32 and 64
// the totals of the other half
template <class C, bool REV, class T>
__device__ __forceinline__ T group_scan(T v, int G) {
    const T id = C::id();
    const int l = lane(), p = REV ? G - 1 - (l & (G - 1)) : l & (G - 1);
    T u;
    u = REV ? dpp<kDppRowShl + 1>(id, v) : dpp<kDppRowShr + 1>(id, v);
    if (p >= 1) v = REV ? C::op(v, u) : C::op(u, v);
    u = REV ? dpp<kDppRowShl + 2>(id, v) : dpp<kDppRowShr + 2>(id, v);
    if (p >= 2) v = REV ? C::op(v, u) : C::op(u, v);
    u = REV ? dpp<kDppRowShl + 4>(id, v) : dpp<kDppRowShr + 4>(id, v);
    if (p >= 4) v = REV ? C::op(v, u) : C::op(u, v);
    if (G > 8) {
        // (lanes 16 .. 31 of a group of 32 take only their own half's here)
        const int h = p & 15;
        u = REV ? dpp<kDppRowShl + 8>(id, v) : dpp<kDppRowShr + 8>(id, v);
        if (h >= 8) v = REV ? C::op(v, u) : C::op(u, v);
    }
    if (G > 16) {
        const T a = lane_value(v, REV ? 16 : 15), b = lane_value(v, REV ? 48 : 47);
        const T t = l < 32 ? a : b;
        if ((p & 31) >= 16) v = REV ? C::op(v, t) : C::op(t, v);
    }
    if (G > 32) {
        const T t = lane_value(v, REV ? 32 : 31);
        if (p >= 32) v = REV ? C::op(v, t) : C::op(t, v);
    }
    return v;
}

constexpr int kShortBlock = 256;
// fewer rows than this, longer than that, may take more than a wavefront each (a row
// of up to 4096 elements is two chunks)
constexpr int64_t kFewRows = 1024, kLongRow = 4096;

template <class P, bool REV>
__global__ __launch_bounds__(kShortBlock) void scan_rows_short(const typename P::in_t* in,
                                                               typename P::out_t* out,
                                                               int64_t rows, int cols,
                                                               int exclusive, int G) {
    using in_t = typename P::in_t;
    using out_t = typename P::out_t;
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    constexpr int E = P::E;
    const int64_t row = ((int64_t)blockIdx.x * kShortBlock + threadIdx.x) / G;
    const int g = (int)threadIdx.x & (G - 1), c0 = g * E;
    const bool live = row < rows;  // (every lane takes part in the lane moves)
    const in_t* src = in + row * cols + c0;
    out_t* dst = out + row * cols + c0;
    in_t raw[E];
    if (live && c0 + E <= cols) {
        load16_any(src, raw);
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) raw[e] = live && c0 + e < cols ? src[e] : in_t(0);
    }
    acc_t loc[E];
    acc_t t = C::id();
#pragma unroll
    for (int ee = 0; ee < E; ++ee) {
        const int e = REV ? E - 1 - ee : ee;
        t = C::op(t, c0 + e < cols ? widen<acc_t>(raw[e]) : C::id());
        loc[e] = t;
    }
    const acc_t incl = group_scan<C, REV>(t, G);
    const acc_t nb = REV ? wave_shift_down(incl, C::id()) : wave_shift_up(incl, C::id());
    const acc_t base = C::op(C::id(), (REV ? g == G - 1 : g == 0) ? C::id() : nb);
    out_t o[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int before = REV ? e + 1 : e - 1;
        const bool none = REV ? e == E - 1 : e == 0;
        const acc_t v = exclusive ? (none ? base : C::op(base, loc[before])) : C::op(base, loc[e]);
        o[e] = (out_t)v;
    }
    if (live && c0 + E <= cols) {
        store_vecs_any<out_t, E>(dst, o);
    } else if (live) {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (c0 + e < cols) dst[e] = o[e];
    }
}

// Rows of up to 256 elements, 64 at a time, one element per lane: 8-byte outputs whose
// rows are not 16-byte aligned, whose vectors would each cross a line or fill half
// of one (37329 x 151 int64 22 us in vectors, 16 so; int32 -> int64 17.7, 16.6; up to
// 128 elements a row of vectors is level or better: 60000 x 65 int32 -> int64 13.3, 17.6)
template <class P, bool REV>
__global__ __launch_bounds__(kShortBlock) void scan_rows_single(const typename P::in_t* in,
                                                                typename P::out_t* out,
                                                                int64_t rows, int cols,
                                                                int exclusive, int) {
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    constexpr int K = 4;
    const int l = lane();
    const int64_t row = (int64_t)blockIdx.x * (kShortBlock / kWave) + threadIdx.x / kWave;
    if (row >= rows) return;  // whole wavefronts; no barrier follows
    const typename P::in_t* src = in + row * cols;
    typename P::out_t* dst = out + row * cols;
    typename P::in_t raw[K];
#pragma unroll
    for (int k = 0; k < K; ++k) raw[k] = k * kWave + l < cols ? src[k * kWave + l] : 0;
    acc_t carry = C::id();
#pragma unroll
    for (int kk = 0; kk < K; ++kk) {
        const int k = REV ? K - 1 - kk : kk, c = k * kWave + l;
        if (k * kWave >= cols) continue;
        const acc_t x = c < cols ? widen<acc_t>(raw[k]) : C::id();
        const acc_t incl = REV ? wave_inclusive_suffix_scan<C>(x) : wave_inclusive_scan<C>(x);
        const acc_t nb = REV ? wave_shift_down(incl, C::id()) : wave_shift_up(incl, C::id());
        const acc_t base = C::op(carry, l == (REV ? kWave - 1 : 0) ? C::id() : nb);
        if (c < cols) dst[c] = (typename P::out_t)(exclusive ? base : C::op(base, x));
        carry = C::op(carry, lane_value(incl, REV ? 0 : kWave - 1));
    }
}

// Flat look-back within each row: tile seq = row * tpr + t (t in scan order)
// publishes its total and reads those of the t tiles before it in its row.  The
// last workgroup, which advances the epoch, waits for every tile's total.
template <class P, bool REV>
__global__ __launch_bounds__(P::kBlock, (flat_waves<P, true>())) void scan_rows_flat(
    const typename P::in_t* in, typename P::out_t* out, int64_t cols, int64_t tpr, int exclusive,
    u64* status, u64* sync) {
    const int64_t row = (int64_t)blockIdx.x / tpr, t = (int64_t)blockIdx.x - row * tpr;
    const int64_t tile = REV ? tpr - 1 - t : t;
    const typename P::in_t* src = in + row * cols;
    typename P::out_t* dst = out + row * cols;
    const bool last = blockIdx.x == gridDim.x - 1;
    u64* const mine = status + 2 * row * tpr;
    const int64_t all = (int64_t)gridDim.x - 1;
    if ((tile + 1) * P::kTile <= cols)
        flat_tile<P, true, REV, true, true>(src, dst, cols, t, tile, tpr, exclusive, mine, sync,
                                            last, status, all);
    else
        flat_tile<P, false, REV, true, true>(src, dst, cols, t, tile, tpr, exclusive, mine, sync,
                                             last, status, all);
}

// Tiles with the decoupled look-back within each row (tpr > 1), numbered by an
// atomic counter in start order so that a tile waits only on tiles already
// running; tpr == 1: one workgroup per row, nothing to wait for.
template <class P, bool FULL, bool REV>
__device__ __forceinline__ void row_tile(const typename P::in_t* src, typename P::out_t* dst,
                                         int64_t cols, int64_t first, int64_t t, int64_t tile,
                                         bool alone, int exclusive, u64* status, u64* sync,
                                         uint32_t epoch) {
    using acc_t = typename P::acc_t;
    __shared__ acc_t s_wtot[P::NW];
    __shared__ acc_t s_prefix;
    Raw<P> raw;
    tile_load<P, FULL, true>(src, cols, tile, raw);
    acc_t wex, agg;
    tile_totals<P, REV>(lane_total<P, FULL>(cols, tile, raw), s_wtot, &wex, &agg);
    acc_t prefix = P::C::id();
    if (!alone) {
        if (threadIdx.x < kWave) {
            const acc_t e = lookback<P>(status + 2 * first, t, agg, epoch, sync + SYNC_ERROR);
            if (threadIdx.x == 0) s_prefix = e;
        }
        __syncthreads();
        prefix = s_prefix;
    }
    keep_raw_only<P>(raw);
    tile_scan_store<P, FULL, REV>(dst, cols, tile, raw, P::C::op(prefix, wex), exclusive != 0);
}

template <class P, bool REV>
__global__ __launch_bounds__(P::kBlock) void scan_rows_tiles(const typename P::in_t* in,
                                                             typename P::out_t* out, int64_t cols,
                                                             int64_t tpr, int exclusive,
                                                             u64* status, u64* sync) {
    __shared__ int64_t s_tile;
    __shared__ uint32_t s_epoch;
    const bool alone = tpr == 1;
    int64_t seq = blockIdx.x;
    uint32_t epoch = 0;
    if (!alone) {
        if (threadIdx.x == 0) {
            s_epoch = epoch_of_call(sync);
            const u64 k = atomicAdd(&sync[SYNC_TILE_COUNTER], 1ull);
            if (k == (u64)gridDim.x - 1)  // every other tile id has been taken
                __hip_atomic_store(&sync[SYNC_TILE_COUNTER], 0ull, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            s_tile = (int64_t)k;
        }
        __syncthreads();
        seq = s_tile;
        epoch = s_epoch;
    }
    const int64_t row = seq / tpr, t = seq - row * tpr;
    const int64_t tile = REV ? tpr - 1 - t : t;
    const typename P::in_t* src = in + row * cols;
    typename P::out_t* dst = out + row * cols;
    if ((tile + 1) * P::kTile <= cols)
        row_tile<P, true, REV>(src, dst, cols, row * tpr, t, tile, alone, exclusive, status, sync,
                               epoch);
    else
        row_tile<P, false, REV>(src, dst, cols, row * tpr, t, tile, alone, exclusive, status, sync,
                                epoch);
    if (!alone && threadIdx.x == 0) {
        const u64 d = atomicAdd(&sync[SYNC_DONE], 1ull);
        if (d == (u64)gridDim.x - 1) {
            __hip_atomic_store(&sync[SYNC_DONE], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            epoch_advance(sync);
        }
    }
}

// Long rows of binary32 sums: the wavefront form's arithmetic in three launches, so
// that the order of the additions, and with it every bit, depends on neither timing
// nor the form (a captured call takes the wavefront form).  A wavefront per chunk of
// P::kTile elements: the totals of its P::R vector rows; a wavefront per row: their
// sum so far at the start of every chunk, one addition after another as the carry of
// the wavefront form runs; a wavefront per chunk: the scan from there.  The input is
// read twice (mostly from cache for rows that fit it).
template <class P, bool REV>
__global__ __launch_bounds__(kWave) void scan_rows_totals(const typename P::in_t* in, int64_t cols,
                                                          int64_t nch, typename P::acc_t* tot) {
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    const int64_t row = (int64_t)blockIdx.x / nch, ch = (int64_t)blockIdx.x - row * nch;
    const int64_t b = lane_base<P>(ch);
    Raw<P> raw;
    if ((ch + 1) * P::kTile <= cols) tile_load<P, true, true>(in + row * cols, cols, ch, raw);
    else tile_load<P, false, true>(in + row * cols, cols, ch, raw);
    acc_t mine = C::id();
#pragma unroll
    for (int r = 0; r < P::R; ++r) {
        acc_t t = C::id();
#pragma unroll
        for (int ee = 0; ee < P::E; ++ee) {
            const int e = REV ? P::E - 1 - ee : ee;
            const bool in_row = b + (int64_t)r * kWave * P::E + e < cols;
            t = C::op(t, in_row ? widen<acc_t>(raw[r][e]) : C::id());
        }
        const acc_t incl = REV ? wave_inclusive_suffix_scan<C>(t) : wave_inclusive_scan<C>(t);
        const acc_t all = lane_value(incl, REV ? 0 : kWave - 1);
        if (lane() == r) mine = all;
    }
    if (lane() < P::R) tot[(int64_t)blockIdx.x * P::R + lane()] = mine;
}

// (A workgroup stages the totals in LDS, in scan order, and its first wavefront adds
// them up from broadcast reads of four: what bounds it is one dependent addition per
// 256 elements.  Loads into that wavefront and lane moves: 30 us for a row of 10^6
// elements; scalar loads, whose latency shows: 48.)
constexpr int kCarryBlock = 256, kCarryStage = 16 * kCarryBlock;

template <class P, bool REV>
__global__ __launch_bounds__(kCarryBlock) void scan_rows_carries(const typename P::acc_t* tot,
                                                                 int64_t nch,
                                                                 typename P::acc_t* carry) {
    using acc_t = typename P::acc_t;
    using C = typename P::C;
    constexpr int kTurn = 64, kChunks = kTurn / P::R;
    __shared__ __attribute__((aligned(16))) acc_t s[kCarryStage];
    const int64_t nb = nch * P::R;
    tot += blockIdx.x * nb;
    carry += blockIdx.x * nch;
    acc_t running = C::id();
    for (int64_t base = 0; base < nb; base += kCarryStage) {
        acc_t v[kCarryStage / kCarryBlock];
#pragma unroll
        for (int u = 0; u < kCarryStage / kCarryBlock; ++u) {
            const int64_t i = base + u * kCarryBlock + threadIdx.x;
            v[u] = i < nb ? tot[REV ? nb - 1 - i : i] : C::id();
        }
        __syncthreads();  // the last stage has been read
#pragma unroll
        for (int u = 0; u < kCarryStage / kCarryBlock; ++u)
            s[u * kCarryBlock + threadIdx.x] = v[u];
        __syncthreads();
        if (threadIdx.x >= kWave) continue;
        const int n = nb - base < kCarryStage ? (int)(nb - base) : kCarryStage;
        for (int t = 0; t < n; t += kTurn) {
            acc_t mine = C::id();
#pragma unroll
            for (int i = 0; i < kTurn; ++i) {
                if (i % P::R == 0 && lane() == i / P::R) mine = running;
                running = C::op(running, s[t + i]);
            }
            const int64_t c = (base + t) / P::R + lane();
            if (lane() < kChunks && c < nch) carry[REV ? nch - 1 - c : c] = mine;
        }
    }
}

template <class P, bool REV>
__global__ __launch_bounds__(kWave) void scan_rows_apply(const typename P::in_t* in,
                                                         typename P::out_t* out, int64_t cols,
                                                         int64_t nch,
                                                         const typename P::acc_t* carry,
                                                         int exclusive) {
    const int64_t row = (int64_t)blockIdx.x / nch, ch = (int64_t)blockIdx.x - row * nch;
    const typename P::in_t* src = in + row * cols;
    typename P::out_t* dst = out + row * cols;
    const typename P::acc_t c = carry[blockIdx.x];
    Raw<P> raw;
    if ((ch + 1) * P::kTile <= cols) {
        tile_load<P, true, true>(src, cols, ch, raw);
        keep_raw_only<P>(raw);
        tile_scan_store<P, true, REV>(dst, cols, ch, raw, c, exclusive != 0);
    } else {
        tile_load<P, false, true>(src, cols, ch, raw);
        keep_raw_only<P>(raw);
        tile_scan_store<P, false, REV>(dst, cols, ch, raw, c, exclusive != 0);
    }
}

// --------------------------------------------------------------- launchers
struct RowsCall {
    const void* x;
    void* y;
    int64_t rows, cols;
    bool rev;
    int excl;
};

template <int DIN, int DOUT, int OP, int RV>
skel_status run_wave(const RowsCall& c, LaunchCtx& lc) {
    using P = SPW<DIN, DOUT, OP, RV>;
    const auto kern = c.rev ? scan_rows_wave<P, true> : scan_rows_wave<P, false>;
    const unsigned grid = (unsigned)std::min<int64_t>(c.rows, INT64_C(1) << 20);
    kern<<<grid, kWave, 0, lc.stream>>>(static_cast<const typename P::in_t*>(c.x),
                                        static_cast<typename P::out_t*>(c.y), c.rows, c.cols,
                                        c.excl);
    return launch_check("scan_rows_wave");
}

// the descriptor array for a tiled form, or NULL (the form that needs none then
// serves the call) where it cannot be allocated, and inside a graph capture: the
// graph may be replayed beside other calls that use the stream's descriptors.  A
// row scan outside a capture uses none that a captured call does, either (the
// second workspace): a wavefront per row, which shares nothing, would serve it.
skel_status tile_status(LaunchCtx& lc, int64_t tiles, void** status) {
    *status = nullptr;
    if (capturing(lc)) return SKEL_OK;
    skel_status e = eager_workspace(lc);
    if (e == SKEL_OK) e = ws_status(lc, (size_t)tiles * 16, status);
    if (e != SKEL_E_NOMEM) return e;
    clear_error();
    return SKEL_OK;
}

template <class P>
skel_status run_tiles(const RowsCall& c, LaunchCtx& lc, bool* done) {
    const int64_t tpr = (c.cols + P::kTile - 1) / P::kTile;
    void* status = nullptr;
    if (tpr > 1) {
        const skel_status e = tile_status(lc, c.rows * tpr, &status);
        if (e != SKEL_OK || !status) return e;
    }
    const auto kern = c.rev ? scan_rows_tiles<P, true> : scan_rows_tiles<P, false>;
    kern<<<(unsigned)(c.rows * tpr), P::kBlock, 0, lc.stream>>>(
        static_cast<const typename P::in_t*>(c.x), static_cast<typename P::out_t*>(c.y), c.cols,
        tpr, c.excl, static_cast<u64*>(status), lc.ws->sync);
    *done = true;
    return launch_check("scan_rows_tiles");
}

template <int DIN, int DOUT, int OP>
skel_status run_ordered(const RowsCall& c, LaunchCtx& lc, bool* done) {
    using P = SPW<DIN, DOUT, OP, 8>;
    using acc_t = typename P::acc_t;
    const int64_t nch = (c.cols + P::kTile - 1) / P::kTile, chunks = c.rows * nch;
    if (capturing(lc) || chunks > max_groups(kWave)) return SKEL_OK;
    void* mem = nullptr;
    skel_status e = eager_workspace(lc);
    if (e == SKEL_OK) e = ws_scratch(lc, (size_t)chunks * (P::R + 1) * sizeof(acc_t), &mem);
    if (e == SKEL_E_NOMEM) {
        clear_error();
        return SKEL_OK;
    }
    if (e != SKEL_OK) return e;
    acc_t* tot = static_cast<acc_t*>(mem);
    acc_t* carry = tot + chunks * P::R;
    const auto* in = static_cast<const typename P::in_t*>(c.x);
    auto* out = static_cast<typename P::out_t*>(c.y);
    const auto totals = c.rev ? scan_rows_totals<P, true> : scan_rows_totals<P, false>;
    const auto carries = c.rev ? scan_rows_carries<P, true> : scan_rows_carries<P, false>;
    const auto apply = c.rev ? scan_rows_apply<P, true> : scan_rows_apply<P, false>;
    totals<<<(unsigned)chunks, kWave, 0, lc.stream>>>(in, c.cols, nch, tot);
    if ((e = launch_check("scan_rows_totals")) != SKEL_OK) return e;
    carries<<<(unsigned)c.rows, kCarryBlock, 0, lc.stream>>>(tot, nch, carry);
    if ((e = launch_check("scan_rows_carries")) != SKEL_OK) return e;
    apply<<<(unsigned)chunks, kWave, 0, lc.stream>>>(in, out, c.cols, nch, carry, c.excl);
    *done = true;
    return launch_check("scan_rows_apply");
}

// rows of several workgroups' tiles
template <int DIN, int DOUT, int OP>
skel_status run_long(const RowsCall& c, LaunchCtx& lc, bool* done) {
    using PS = SP<DIN, DOUT, OP, 2, false>;
    // sums of floating-point numbers keep one order of additions
    if constexpr (DOUT == SKEL_F32 && OP == SKEL_SUM) {
        return run_ordered<DIN, DOUT, OP>(c, lc, done);
    } else {
        const int64_t tpr = (c.cols + PS::kTile - 1) / PS::kTile;
        const auto flat = c.rev ? scan_rows_flat<PS, true> : scan_rows_flat<PS, false>;
        const char *x0 = static_cast<const char*>(c.x), *y0 = static_cast<const char*>(c.y);
        const int64_t n = c.rows * c.cols;
        const bool apart = x0 + n * sizeof(typename PS::in_t) <= y0 ||
                           y0 + n * sizeof(typename PS::out_t) <= x0;
        if (!apart || c.rows * tpr > kFlatMaxTiles ||
            c.rows * tpr > resident_slots(reinterpret_cast<const void*>(flat), PS::kBlock, lc))
            return run_tiles<SP<DIN, DOUT, OP, 16, false>>(c, lc, done);
        void* status = nullptr;
        const skel_status e = tile_status(lc, c.rows * tpr, &status);
        if (e != SKEL_OK || !status) return e;
        flat<<<(unsigned)(c.rows * tpr), PS::kBlock, 0, lc.stream>>>(
            static_cast<const typename PS::in_t*>(c.x), static_cast<typename PS::out_t*>(c.y),
            c.cols, tpr, c.excl, static_cast<u64*>(status), lc.ws->sync);
        *done = true;
        return launch_check("scan_rows_flat");
    }
}

template <int DIN, int DOUT, int OP>
skel_status scan_rows_typed(const RowsCall& c, LaunchCtx& lc) {
    using PS = SP<DIN, DOUT, OP, 2, false>;
    using PM = SP<DIN, DOUT, OP, 4, false>;
    using PL = SP<DIN, DOUT, OP, 16, false>;
    constexpr int E = PS::E;
    const bool single = sizeof(typename PS::out_t) == 8 && c.cols > 128 && c.cols <= 256 &&
                        (c.cols * sizeof(typename PS::in_t)) % 16 != 0;
    // 64 lanes per row: 20000 x 256 binary32 8.3 us against 9.2 for a wavefront per
    // workgroup, 60000 x 65 int64 17.9 against 23; but int32 -> int64 15.1 against 13.8,
    // and 200 x 200 2.92 against 2.81
    const int lanes = sizeof(typename PS::in_t) == sizeof(typename PS::out_t) &&
                      c.rows >= 4 * (int64_t)lc.dev->cus ? 64 : 32;
    if (c.cols <= lanes * E || single) {
        const int G = c.cols <= 8 * E ? 8 : c.cols <= 16 * E ? 16 : c.cols <= 32 * E ? 32 : 64;
        auto kern = c.rev ? scan_rows_short<PS, true> : scan_rows_short<PS, false>;
        if constexpr (sizeof(typename PS::out_t) == 8)
            if (single) kern = c.rev ? scan_rows_single<PS, true> : scan_rows_single<PS, false>;
        // (2^29 rows at 8 lanes are more work items than one launch numbers)
        const int64_t per_group = kShortBlock / G, most = max_groups(kShortBlock) * per_group;
        for (int64_t r = 0; r < c.rows; r += most) {
            const int64_t rows = std::min(c.rows - r, most);
            kern<<<(unsigned)((rows + per_group - 1) / per_group), kShortBlock, 0, lc.stream>>>(
                static_cast<const typename PS::in_t*>(c.x) + r * c.cols,
                static_cast<typename PS::out_t*>(c.y) + r * c.cols, rows, (int)c.cols, c.excl, G);
            const skel_status e = launch_check(single ? "scan_rows_single" : "scan_rows_short");
            if (e != SKEL_OK) return e;
        }
        return SKEL_OK;
    }
    if (c.rows < kFewRows && c.cols > kLongRow) {
        bool done = false;
        skel_status e = SKEL_OK;
        const bool one_each = c.rows <= lc.dev->cus;  // a workgroup of 16 wavefronts per row
        if (c.cols <= PM::kTile) e = run_tiles<PM>(c, lc, &done);
        else if (c.cols <= PL::kTile && one_each) e = run_tiles<PL>(c, lc, &done);
        else if (c.cols > PL::kTile && 2 * c.rows < 3 * lc.dev->cus)
            e = run_long<DIN, DOUT, OP>(c, lc, &done);
        if (e != SKEL_OK || done) return e;
    }
    if (c.cols <= 256) return run_wave<DIN, DOUT, OP, 1>(c, lc);
    if (c.cols <= 512) return run_wave<DIN, DOUT, OP, 2>(c, lc);
    if (c.cols <= 1024) return run_wave<DIN, DOUT, OP, 4>(c, lc);
    return run_wave<DIN, DOUT, OP, 8>(c, lc);
}

template <int DIN, int DOUT>
skel_status scan_rows_op(int op, const RowsCall& c, LaunchCtx& lc) {
    switch (op) {
    case SKEL_SUM: return scan_rows_typed<DIN, DOUT, SKEL_SUM>(c, lc);
    case SKEL_MIN: return scan_rows_typed<DIN, DOUT, SKEL_MIN>(c, lc);
    default: return scan_rows_typed<DIN, DOUT, SKEL_MAX>(c, lc);
    }
}

}  // namespace

skel_status launch_scan_rows(int kind, int op, skel_dtype din, skel_dtype dout, const void* x,
                             void* y, int64_t rows, int64_t cols, LaunchCtx& lc) {
    const RowsCall c{x, y, rows, cols,
                     kind == SKEL_REVERSE_INCLUSIVE || kind == SKEL_REVERSE_EXCLUSIVE,
                     kind == SKEL_EXCLUSIVE || kind == SKEL_REVERSE_EXCLUSIVE ? 1 : 0};
    if (din == SKEL_I32 && dout == SKEL_I32) return scan_rows_op<SKEL_I32, SKEL_I32>(op, c, lc);
    if (din == SKEL_I32) return scan_rows_op<SKEL_I32, SKEL_I64>(op, c, lc);
    if (din == SKEL_I64) return scan_rows_op<SKEL_I64, SKEL_I64>(op, c, lc);
    return scan_rows_op<SKEL_F32, SKEL_F32>(op, c, lc);
}

}  // namespace skel

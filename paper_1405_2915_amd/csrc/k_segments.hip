// Segmented Reduce: many vectors of uneven length, stored back to back in one
// container and delimited by an offsets container, reduced in one call:
//   out[s] = op over x[offsets[s]] .. x[offsets[s+1] - 1]
// This is the batched form of the Reduce skeleton (Section III): one skeleton
// instance applied to a set of operands of different sizes.
//
// Variants:
//   B0  per segment: one two-pass Reduce per segment (2 launches each); the
//       plain loop a caller would write
//   B1  whole batch: the work is divided over the elements, not over the
//       segments.  Every workgroup takes one chunk of kChunk consecutive
//       elements and reads which segments start in it from a table that the
//       check of the offsets writes, so many short segments and a few long
//       ones load the device alike.  A chunk inside one segment is a plain reduction; a
//       chunk with segment starts is scanned once (a segmented scan in
//       registers, its values in LDS) and every segment that ends in it reads
//       its total at its last element.  What a segment has in other chunks is
//       kept as partials, combined in chunk order by a last small launch
//       (deterministic; no workgroup waits on another).
//       Measured: 200003 segments of 1..256 elements (36 MB) 17.6 us, against
//       1058 us for one work item per segment (each item costs a workgroup a
//       search, two barriers and a ticket: 0.8 us of the 1024 resident
//       workgroups' time, and the item table took one workgroup 0.5 ms);
//       4096 log-uniform segments of 32..2^20 (1.65 GB) 249 us against 277;
//       20011 of 1000..9000 62 us against 162.
//       (Empty segments take no elements, so a run of them falls to one
//       workgroup: a million 2.4 ms, 5.0 with a work item each.)
// B1 checks the offsets first: if they decrease or leave [0, n] nothing is
// computed and error flag 4 is raised.
#include "kcommon.hpp"
#include "dispatch.hpp"
#include "launch.hpp"

namespace skel {
namespace {

using namespace dev;

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / kWave;
// 16-byte vectors per lane and chunk.  Measured (4096 long vectors / 200003
// short ones): 3 rows 300 / 21.6 us, 4 rows 251 / 20.6, 6 rows 259 / 20.7,
// 8 rows 266 / 21.6 (the chunk's scanned values in LDS then allow only four
// workgroups per CU).
constexpr int kRows = 4;
constexpr int kSlice = kWave * 4 * kRows;       // elements per wavefront: 1024
constexpr int kChunk = kWaves * kSlice;         // elements per workgroup: 4096
constexpr int kCheckBlocks = 64;                // workgroups of the offsets check
constexpr int kCheckWaves = kCheckBlocks * 1024 / kWave;
constexpr int kOwnChunks = 4;                   // first[] entries one lane writes alone
constexpr int kGroup = kWave;                   // chunks per group[] entry
constexpr int kSerialPieces = 16;               // partials one lane combines alone
constexpr int kWavePieces = 1024;               // and one wavefront, in one round of loads

template <int OP>
using CF = Comb<float, OP>;

// Running value of a segmented scan: v combines everything since the last
// segment start, f says whether there was one.
struct SegVal {
    float v;
    uint32_t f;
};
template <int OP>
struct SegComb {
    static __device__ __forceinline__ SegVal id() { return {CF<OP>::id(), 0u}; }
    static __device__ __forceinline__ SegVal op(SegVal a, SegVal b) {
        return {b.f ? b.v : CF<OP>::op(a.v, b.v), a.f | b.f};
    }
};

// op over x[a, b) by one workgroup: scalar head up to 16-byte alignment,
// 16-byte vectors, scalar tail
template <int OP>
__device__ __forceinline__ float range_reduce(const float* x, int64_t a, int64_t b,
                                              float* lds) {
    using C = CF<OP>;
    float acc = C::id();
    int64_t va = (a + 3) & ~int64_t(3);
    if (va > b) va = b;
    const int64_t vb = va + ((b - va) & ~int64_t(3));
    if (a + threadIdx.x < va) acc = C::op(acc, x[a + threadIdx.x]);
    const f32x4* xv = reinterpret_cast<const f32x4*>(x + va);
    const int64_t nv = (vb - va) >> 2;
    float acc2[4] = {C::id(), C::id(), C::id(), C::id()};
    int64_t i = threadIdx.x;
    for (; i + 3 * kBlock < nv; i += 4 * kBlock) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(&xv[i + u * kBlock]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            acc2[u] = C::op(acc2[u], v[u].x);
            acc2[u] = C::op(acc2[u], v[u].y);
            acc2[u] = C::op(acc2[u], v[u].z);
            acc2[u] = C::op(acc2[u], v[u].w);
        }
    }
    for (; i < nv; i += kBlock) {
        const f32x4 v = xv[i];
        acc2[0] = C::op(C::op(C::op(C::op(acc2[0], v.x), v.y), v.z), v.w);
    }
    if (vb + threadIdx.x < b) acc = C::op(acc, x[vb + threadIdx.x]);
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = C::op(acc, acc2[u]);
    return block_reduce<C>(acc, lds);  // valid in wavefront 0
}

// ------------------------------------------------------------------- B1 ----
// Scratch of one call.  Every chunk writes its own entries, so nothing needs
// clearing.
//   bad[b]   workgroup b of the check saw an offset out of order or range
//   group[g] the first s with off[s] >= the start of chunk c for every chunk c
//            of group g (kGroup chunks), if that is one s; -1: see
//   first[c] the same of chunk c alone
//            (both for the chunks that begin in [0, off[nseg]] and end beyond
//            off[0])
//   fin[c]   the segment that began before chunk c and ends in it, or -1
//   head[c]  op over chunk c's part of the segment that began before it
//   tail[c]  op over chunk c's part of the segment that begins in c and ends
//            after it
struct SegWork {
    uint32_t* bad;
    int64_t* group;
    int64_t* first;
    int64_t* fin;
    float* head;
    float* tail;
};

// Checks the offsets and finds each chunk's first segment from the other side:
// segment s (off[s] = lo, off[s + 1] = hi) is followed by s + 1 in the chunks
// that begin in (lo, hi].  A lane writes up to kOwnChunks of them itself; a
// wavefront writes a longer segment's together, one entry per whole group, so
// that a segment of 2^28 elements takes 1024 stores instead of 65536 (30 us by
// one wavefront).  Nothing is written for an offset that is out of order or
// range.  The table saves every chunk a search of the offsets, two or three rounds
// of dependent loads (200003 short segments 19.4 -> 17.1 us, 20011 of about 5000
// elements 77 -> 63).
__global__ __launch_bounds__(1024) void seg_check(const int64_t* off, int64_t nseg, int64_t n,
                                                  int64_t nchunks, SegWork wk, u64* err) {
    int b = 0;
    const int64_t wave = (int64_t)(threadIdx.x / kWave) * kCheckBlocks + blockIdx.x;
    // few segments are spread over the wavefronts, whose long ones go in turn
    // (4096 long segments 258.4 -> 254.3 us); fewer than four per wavefront cost
    // short ones more (900: 9.3 -> 9.5 us at one)
    const int64_t share = (nseg + kCheckWaves - 1) / kCheckWaves;
    const int64_t per = share < 4 ? 4 : share < kWave ? share : kWave;
    for (int64_t base = wave * per; base < nseg; base += kCheckWaves * per) {
        const int64_t s = lane() < per ? base + lane() : nseg;
        int64_t c = 0, count = 0;  // chunks c .. c + count - 1 follow segment s
        if (s < nseg) {
            const int64_t lo = off[s], hi = off[s + 1];
            if (lo < 0 || hi < lo || hi > n) {
                b = 1;
            } else {
                c = lo / kChunk + 1;
                const int64_t end = hi / kChunk;
                count = (end < nchunks ? end : nchunks - 1) - c + 1;
                if (s == 0) {  // the chunk that off[0] lies in
                    const int64_t c0 = c - 1 < nchunks ? c - 1 : nchunks - 1;
                    wk.first[c0] = 0;
                    wk.group[c0 / kGroup] = -1;
                }
            }
        }
        if (count <= kOwnChunks)
            for (int64_t k = c; k < c + count; ++k) {
                wk.first[k] = s + 1;
                if (k % kGroup == 0) wk.group[k / kGroup] = -1;
            }
        for (u64 many = __ballot(count > kOwnChunks); many; many &= many - 1) {
            const int l = __ffsll(many) - 1;
            const int64_t a = lane_value(c, l), end = a + lane_value(count, l) - 1;
            // groups that begin in a .. end; only the last may be cut short
            const int64_t g0 = (a + kGroup - 1) / kGroup, g1 = end / kGroup;
            for (int64_t g = g0 + lane(); g <= g1; g += kWave) {
                const int64_t ge = g * kGroup + kGroup - 1;
                wk.group[g] = end >= (ge < nchunks ? ge : nchunks - 1) ? base + l + 1 : -1;
            }
            // the chunks before the first group, and those of a last one cut short
            int64_t k = a + lane();
            if (k < g0 * kGroup && k <= end) wk.first[k] = base + l + 1;
            k = g1 * kGroup + lane();
            if (g1 >= g0 && k <= end) wk.first[k] = base + l + 1;
        }
    }
    b = __syncthreads_or(b);
    if (threadIdx.x == 0) {
        wk.bad[blockIdx.x] = (uint32_t)(b != 0);
        if (b) atomicOr(err, 4ull);
    }
}

// What bounds it: long segments, HBM (one 16 KiB chunk per workgroup, all of
// it in flight at once: 6.6 TB/s); short segments, the chain of dependent
// loads of a chunk (flags and table, offsets) and the segmented scan's latency
// (its arithmetic does not show: a scan that moves one word per step instead of
// two took as long).
template <int OP>
__global__ __launch_bounds__(kBlock) void seg_reduce_chunks(const float* x, int64_t n,
                                                            const int64_t* off, int64_t nseg,
                                                            SegWork wk, float* out) {
    using C = CF<OP>;
    using SC = SegComb<OP>;
    __shared__ __attribute__((aligned(16))) float scanned[kChunk];
    __shared__ uint32_t starts[kChunk / 32];  // bit e: a segment starts at element e
    __shared__ float slice_sum[kWaves];       // each slice's value since its last start
    __shared__ float lds[kWaves];
    const int l = lane(), w = threadIdx.x / kWave;
    const int64_t c = blockIdx.x, c0 = c * kChunk, c1 = c0 + kChunk;
    const bool last = c == (int64_t)gridDim.x - 1;
    // the loads that depend on nothing go first
    f32x4 v[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const int64_t i = c0 + w * kSlice + r * (kWave * 4) + 4 * l;
        if (i + 4 <= n) {
            v[r] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(x + i));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[r][e] = i + e < n ? x[i + e] : 0.0f;
        }
    }
    uint32_t bad = 0;
#pragma unroll
    for (int k = 0; k < kCheckBlocks; ++k) bad |= wk.bad[k];
    const int64_t off_end = off[nseg], off_begin = off[0];
    const int64_t d = last ? c : c + 1;
    const int64_t g0 = wk.group[c / kGroup], g1 = wk.group[d / kGroup];
    const int64_t f0 = wk.first[c], f1 = wk.first[d];
    // offsets out of order, or a chunk outside [off[0], off[nseg]] (the last
    // chunk also owns the empty segments at n)
    if (bad || c0 > off_end || (!last && c1 <= off_begin)) {
        if (threadIdx.x == 0) wk.fin[c] = -1;
        return;
    }
    // segments s0 .. s1 - 1 start in this chunk; segment s0 - 1 covers its
    // first element if it ends beyond c0
    const int64_t s0 = g0 >= 0 ? g0 : f0;
    const int64_t s1 = last || c1 > off_end ? nseg : g1 >= 0 ? g1 : f1;
    const int64_t he = off[s0];
    const bool has_head = s0 > 0 && he > c0;
    if (s0 == s1) {
        // no start: the chunk (up to its end or the last segment's) is part of
        // one segment
        float a[4] = {C::id(), C::id(), C::id(), C::id()};
        if (has_head) {
            const int64_t e1 = he < c1 ? he : c1;
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const int64_t i = c0 + w * kSlice + r * (kWave * 4) + 4 * l;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < e1) a[e] = C::op(a[e], v[r][e]);
            }
        }
        const float part = block_reduce<C>(C::op(C::op(a[0], a[1]), C::op(a[2], a[3])), lds);
        if (threadIdx.x == 0) {
            wk.head[c] = part;
            wk.fin[c] = has_head && he <= c1 ? s0 - 1 : -1;
        }
        return;
    }
    if (threadIdx.x < kChunk / 32) starts[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t s = s0 + threadIdx.x; s < s1; s += kBlock) {
        const uint64_t p = (uint64_t)(off[s] - c0);  // (a start at n may equal kChunk)
        if (p < kChunk) atomicOr(&starts[p >> 5], 1u << (p & 31));
    }
    __syncthreads();
    // segmented scan of the wavefront's slice, row by row
    SegVal running = SC::id();
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const int p = w * kSlice + r * (kWave * 4) + 4 * l;
        const uint32_t nib = (starts[p >> 5] >> (p & 31)) & 15u;
        float loc[4];
        float t = C::id();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            t = C::op((nib >> e) & 1u ? C::id() : t, v[r][e]);
            loc[e] = t;
        }
        const SegVal incl = wave_inclusive_scan<SC>(SegVal{t, nib});
        SegVal ex = wave_shift_up(incl, SC::id());
        if (l == 0) ex = SC::id();
        const float in = SC::op(running, ex).v;
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = nib & ((2u << e) - 1u) ? loc[e] : C::op(in, loc[e]);
        *reinterpret_cast<f32x4*>(&scanned[p]) = o;
        running = SC::op(running, lane_value(incl, kWave - 1));
    }
    if (l == 0) slice_sum[w] = running.v;
    __syncthreads();
    // op over elements [a, b) of the chunk, 0 <= a < b <= kChunk, where a is a
    // segment's start or 0 and no other segment with elements starts in (a, b):
    // its last element's scanned value, preceded by what the slices before it hold
    const auto piece = [&](int a, int b) {
        const int wa = a / kSlice, wb = (b - 1) / kSlice;
        float t = scanned[b - 1];
        if (wa < wb) {
            float h = slice_sum[wa];
            for (int q = wa + 1; q < wb; ++q) h = C::op(h, slice_sum[q]);
            t = C::op(h, t);
        }
        return t;
    };
    for (int64_t s = s0 + threadIdx.x; s < s1; s += kBlock) {
        const int64_t a = off[s], b = off[s + 1];
        if (a == b) out[s] = C::id();
        else if (b <= c1) out[s] = piece((int)(a - c0), (int)(b - c0));
        else wk.tail[c] = piece((int)(a - c0), kChunk);
    }
    if (threadIdx.x == 0) {
        if (has_head) wk.head[c] = piece(0, (int)(he - c0));
        wk.fin[c] = has_head ? s0 - 1 : -1;
    }
}

// the segments that span chunks: lane t looks at one chunk and, if such a
// segment ends in it, combines its partials in chunk order -- alone for a few
// pieces, by a wavefront (one round of loads) for more, by the whole workgroup
// for many (4096 long segments: 4 us less than the workgroup for all but a few
// pieces, one segment after another)
template <int OP>
__global__ __launch_bounds__(kBlock) void seg_finish(const int64_t* off, int64_t nchunks,
                                                     SegWork wk, float* out) {
    using C = CF<OP>;
    struct Span {
        int64_t seg, a, e;  // the pieces: tail[a], head[a + 1 .. e]
    };
    __shared__ float lds[kWaves];
    __shared__ Span todo[kBlock];  // a wavefront's from the front, the workgroup's from the back
    __shared__ int ntodo, nlarge;
    if (threadIdx.x == 0) ntodo = nlarge = 0;
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t seg = c < nchunks ? wk.fin[c] : -1;
    if (seg >= 0) {
        const int64_t a = off[seg] / kChunk;
        if (c - a <= kSerialPieces) {
            // every load issued before the first is used
            const float t0 = wk.tail[a];
            float h[kSerialPieces];
#pragma unroll
            for (int u = 0; u < kSerialPieces; ++u)
                h[u] = a + 1 + u <= c ? wk.head[a + 1 + u] : C::id();
            float t = t0;
#pragma unroll
            for (int u = 0; u < kSerialPieces; ++u) t = C::op(t, h[u]);
            out[seg] = t;
        } else if (c - a <= kWavePieces) {
            todo[atomicAdd(&ntodo, 1)] = {seg, a, c};  // (any order: each is one segment)
        } else {
            todo[kBlock - 1 - atomicAdd(&nlarge, 1)] = {seg, a, c};
        }
    }
    __syncthreads();
    const int m = ntodo;
    for (int k = threadIdx.x / kWave; k < m; k += kWaves) {
        const Span sp = todo[k];
        float t = lane() == 0 ? wk.tail[sp.a] : C::id();
        const int64_t q = sp.a + 1 + lane();
        float h[kWavePieces / kWave];
#pragma unroll
        for (int u = 0; u < kWavePieces / kWave; ++u)
            h[u] = q + u * kWave <= sp.e ? wk.head[q + u * kWave] : C::id();
#pragma unroll
        for (int u = 0; u < kWavePieces / kWave; ++u) t = C::op(t, h[u]);
        t = wave_reduce<C>(t);
        if (lane() == 0) out[sp.seg] = t;
    }
    const int big = nlarge;
    for (int k = 0; k < big; ++k) {
        const Span sp = todo[kBlock - 1 - k];
        float t = threadIdx.x == 0 ? wk.tail[sp.a] : C::id();
        int64_t q = sp.a + 1 + threadIdx.x;
        for (; q + 15 * kBlock <= sp.e; q += 16 * kBlock) {
            float h[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) h[u] = wk.head[q + u * kBlock];
#pragma unroll
            for (int u = 0; u < 16; ++u) t = C::op(t, h[u]);
        }
        for (; q <= sp.e; q += kBlock) t = C::op(t, wk.head[q]);
        t = block_reduce<C>(t, lds);
        if (threadIdx.x == 0) out[sp.seg] = t;
        __syncthreads();  // lds is reused by the next segment
    }
}

// B0: one segment per launch pair (partials, then finish)
template <int OP>
__global__ __launch_bounds__(kBlock) void seg_one_partials(const float* x, int64_t a, int64_t b,
                                                           float* part) {
    __shared__ float lds[kBlock / kWave];
    using C = CF<OP>;
    // grid-stride over this segment with the workgroup's range share
    const int64_t len = b - a;
    const int64_t per = (len + gridDim.x - 1) / gridDim.x;
    const int64_t ca = a + (int64_t)blockIdx.x * per;
    int64_t cb = ca + per;
    if (cb > b) cb = b;
    const float v = range_reduce<OP>(x, ca < b ? ca : b, cb, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = v;
    (void)sizeof(C);
}

template <int OP>
__global__ __launch_bounds__(1024) void seg_one_finish(const float* part, int g, float* out) {
    __shared__ float lds[1024 / kWave];
    using C = CF<OP>;
    float a = C::id();
    for (int i = threadIdx.x; i < g; i += 1024) a = C::op(a, part[i]);
    a = block_reduce<C>(a, lds);
    if (threadIdx.x == 0) *out = a;
}

template <int OP>
skel_status run_segments(int v, const float* x, int64_t n, const int64_t* off_dev,
                         const int64_t* off_host, int64_t nseg, float* out, LaunchCtx& lc) {
    hipStream_t st = lc.stream;
    if (v == B0_PER_SEGMENT) {
        const int gmax = lc.dev->cus * 4;
        void* part = nullptr;
        skel_status e = ws_scratch(lc, (size_t)gmax * sizeof(float), &part);
        if (e != SKEL_OK) return e;
        for (int64_t s = 0; s < nseg; ++s) {
            int64_t a = off_host[s], b = off_host[s + 1];
            a = a < 0 ? 0 : (a > n ? n : a);
            b = b < a ? a : (b > n ? n : b);
            int64_t g = (b - a + 2047) / 2048;
            if (g < 1) g = 1;
            if (g > gmax) g = gmax;
            seg_one_partials<OP><<<(unsigned)g, kBlock, 0, st>>>(x, a, b,
                                                                 static_cast<float*>(part));
            seg_one_finish<OP><<<1, 1024, 0, st>>>(static_cast<float*>(part), (int)g, out + s);
        }
        return launch_check("reduce_segments_per_segment");
    }
    // B1: check, chunks, then the segments that span chunks
    const int64_t nchunks = n > 0 ? (n + kChunk - 1) / kChunk : 1;
    const auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
    const size_t bad_b = up(kCheckBlocks * sizeof(uint32_t)),
                 group_b = up((size_t)((nchunks + kGroup - 1) / kGroup) * 8),
                 first_b = up((size_t)nchunks * 8), fin_b = first_b,
                 part_b = up((size_t)nchunks * 4);
    void* mem = nullptr;
    skel_status e = ws_scratch(lc, bad_b + group_b + first_b + fin_b + 2 * part_b, &mem);
    if (e != SKEL_OK) return e;
    char* p = static_cast<char*>(mem);
    SegWork wk;
    wk.bad = reinterpret_cast<uint32_t*>(p);
    wk.group = reinterpret_cast<int64_t*>(p += bad_b);
    wk.first = reinterpret_cast<int64_t*>(p += group_b);
    wk.fin = reinterpret_cast<int64_t*>(p += first_b);
    wk.head = reinterpret_cast<float*>(p += fin_b);
    wk.tail = reinterpret_cast<float*>(p += part_b);
    seg_check<<<kCheckBlocks, 1024, 0, st>>>(off_dev, nseg, n, nchunks, wk,
                                             lc.ws->sync + SYNC_ERROR);
    if ((e = launch_check("reduce_segments_check")) != SKEL_OK) return e;
    seg_reduce_chunks<OP><<<(unsigned)nchunks, kBlock, 0, st>>>(x, n, off_dev, nseg, wk, out);
    if ((e = launch_check("reduce_segments_chunks")) != SKEL_OK || nchunks == 1) return e;
    seg_finish<OP><<<(unsigned)((nchunks + kBlock - 1) / kBlock), kBlock, 0, st>>>(off_dev, nchunks,
                                                                                   wk, out);
    return launch_check("reduce_segments_finish");
}

}  // namespace

skel_status launch_reduce_segments(int v, int op, const float* x, int64_t n,
                                   const int64_t* off_dev, const int64_t* off_host,
                                   int64_t nseg, float* out, LaunchCtx& lc) {
    switch (op) {
    case SKEL_SUM: return run_segments<SKEL_SUM>(v, x, n, off_dev, off_host, nseg, out, lc);
    case SKEL_MIN: return run_segments<SKEL_MIN>(v, x, n, off_dev, off_host, nseg, out, lc);
    default: return run_segments<SKEL_MAX>(v, x, n, off_dev, off_host, nseg, out, lc);
    }
}

}  // namespace skel

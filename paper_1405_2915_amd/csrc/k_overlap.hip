// MapOverlap skeleton kernels: a map whose element function sees a
// neighbourhood (Section III lists mapoverlap among the data-parallel
// skeletons).  Here the neighbourhood function is a linear weighting in
// correlation orientation:
//   1D  out[i]    = sum_k w[k] * x[e(i + k - r)]
//   2D  out[i][j] = sum_a sum_b W[a][b] * x[e(i + a - ry)][e(j + b - rx)]
// with e() the border rule (clamp, constant pad, cyclic).
//
// Variants:
//   O1a  1D direct: one output per lane, taps read through the caches
//   O1b  1D LDS tile: a workgroup stages its outputs' inputs once; each lane
//        slides a register window over them, four taps per 16-byte LDS read
//   O1c  1D cross-lane: r <= 4 neighbours come from adjacent lanes by
//        shuffles; no LDS, no barrier
//   O2a  2D direct: one output per lane, (2ry+1)(2rx+1) taps from global
//   O2b  2D LDS tile: a 64-column output tile of 16 or 32 rows plus halo staged
//        in LDS with 16-byte loads; each lane computes four columns of one or
//        two rows
//   O2c  2D separable (W = wy (x) wx): the staged tile is filtered along rows
//        into a second LDS buffer, then along columns; 2(2r+1) instead of
//        (2r+1)^2 multiply-adds per output
//   O2d  2D separable with the row pass read from global memory through L1
//        and only its result staged in LDS
//   O2e  2D marching window (ry, rx <= 4): each wavefront walks down a strip
//        of 256 columns, loading every input row once; horizontal neighbours
//        come from the adjacent lanes by DPP moves and the 2ry+1 output rows
//        a loaded row feeds are kept in a ring of registers.  No LDS, no
//        barrier.
// 2D tiles are visited in an XCD-aware order: consecutive workgroups go to
// different XCDs round-robin, so tile ids are remapped to give each XCD a
// contiguous band of tiles whose shared halo rows stay in that XCD's L2.
#include <type_traits>

#include "kcommon.hpp"
#include "dispatch.hpp"
#include "launch.hpp"

namespace skel {
namespace {

using dev::f32x4;
// a 16-byte vector at any float's address: one global access, as for an
// aligned one (a line boundary inside it costs a second line)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

struct W1 {
    float w[2 * SKEL_MAX_RADIUS_1D + 1];
};
struct W2 {
    float w[(2 * SKEL_MAX_RADIUS_2D + 1) * (2 * SKEL_MAX_RADIUS_2D + 1)];
    float wy[2 * SKEL_MAX_RADIUS_2D + 1];
    float wx[2 * SKEL_MAX_RADIUS_2D + 1];
};

// border rule: true and the index to read, or false for the constant pad
__device__ __forceinline__ bool border(int64_t j, int64_t n, int edge, int64_t& k) {
    if (j >= 0 && j < n) {
        k = j;
        return true;
    }
    if (edge == SKEL_EDGE_CLAMP) {
        k = j < 0 ? 0 : n - 1;
        return true;
    }
    if (edge == SKEL_EDGE_CYCLIC) {
        int64_t m = j % n;
        k = m < 0 ? m + n : m;
        return true;
    }
    return false;
}

// the same for j at most a tile and its halo past either end: CYCLIC without the
// 64-bit remainder (3895 images of 12 x 64, 5-point: 26 us against 13 for CLAMP
// with it)
__device__ __forceinline__ bool border_near(int64_t j, int64_t n, int edge, int64_t& k) {
    if (edge != SKEL_EDGE_CYCLIC) return border(j, n, edge, k);
    const int64_t past = j < 0 ? -1 - j : j - n;  // < 0: inside
    const int64_t in = past < n ? past : (int64_t)((uint32_t)past % (uint32_t)n);
    k = past < 0 ? j : j < 0 ? n - 1 - in : in;
    return true;
}

__device__ __forceinline__ float fetch1(const float* x, int64_t n, int64_t j, int edge,
                                        float pad) {
    int64_t k;
    return border(j, n, edge, k) ? x[k] : pad;
}

__device__ __forceinline__ float fetch2(const float* x, int64_t rows, int64_t cols, int64_t i,
                                        int64_t j, int edge, float pad) {
    int64_t a, b;
    if (!border(i, rows, edge, a) || !border(j, cols, edge, b)) return pad;
    return x[a * cols + b];
}

constexpr int kBlock = 256;

// ------------------------------------------------------------------- 1D
template <int RT>
__global__ __launch_bounds__(kBlock) void ov1_direct(const float* x, float* out, int64_t n,
                                                     W1 w, int r_, int edge, float pad) {
    const int r = RT >= 0 ? RT : r_;
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    float acc = 0.0f;
    if (i - r >= 0 && i + r < n) {
#pragma unroll
        for (int k = 0; k <= 2 * (RT >= 0 ? RT : SKEL_MAX_RADIUS_1D); ++k) {
            if (k > 2 * r) break;
            acc = __builtin_fmaf(w.w[k], x[i + k - r], acc);
        }
    } else {
        for (int k = 0; k <= 2 * r; ++k)
            acc = __builtin_fmaf(w.w[k], fetch1(x, n, i + k - r, edge, pad), acc);
    }
    out[i] = acc;
}

// The transpose of a clamped 1D map (adjoint of MapOverlap 1D, CLAMP) is the
// zero-padded correlation with reversed weights except at the two end
// elements, which also collect every read past them:
//     out[0]   = sum_i lo[i] x[i],         lo[i] = w'[0] + ... of tap i outward
//     out[n-1] = sum_m hi[m] x[n - 1 - m]
// with the prefix sums of the forward weights as coefficients
// (launch_overlap1d_transposed).
struct Ends1 {
    float lo[SKEL_MAX_RADIUS_1D + 1], hi[SKEL_MAX_RADIUS_1D + 1];
};

// The same element by element: first + step * lane of 0 or, HI, n - 1, from x
// as x(i).  The prefix sums give the same result up to rounding, but for infinite
// and NaN inputs, which must meet each weight (a sum of weights may be zero or
// have another sign): a non-finite result is computed again from these terms.
template <bool HI, class X>
__device__ __forceinline__ float end_terms(const W1& w, int r, int64_t n, X x, int first, int step) {
    float p = 0.0f;
    for (int k = first; k <= 2 * r; k += step) {
        // w is reversed: the forward tap 2r - k reads element i + r - k
        const int reach = HI ? r - k : k - r;  // farthest output that reads the end through it
        for (int64_t m = 0; m <= reach && m < n; ++m)
            p = __builtin_fmaf(w.w[k], x(HI ? n - 1 - m : m), p);
        if (n == 1 && reach < 0) p = __builtin_fmaf(w.w[k], x(0), p);
    }
    return p;
}

// O1b.  A workgroup of NT lanes stages the inputs of its 4 * NT outputs in LDS;
// a lane owns four consecutive outputs and slides a window of eight inputs
// along the taps: per four taps one 16-byte LDS read feeds sixteen
// multiply-adds, the weights come from scalar registers, and the loop runs over
// the actual radius.  The additions of an output run in tap order, as in O1a.
// What bounds it is HBM up to a radius of about 16, then the vector ALU (2r + 1
// unpacked multiply-adds per output).  Measured on 2^24 floats, the map and its
// transpose together: radius 5 51 us (4.9 TB/s), 16 62 us, 64 158 us, against
// 267, 519 and 1780 us for a fully unrolled window of the largest radius (its
// 129 guarded taps and 132 window registers).  Eight or sixteen outputs per
// lane measured slower (radius 16: 65 and 84 us).
template <int NT, bool ENDS>
__global__ __launch_bounds__(NT) void ov1_window(const float* x, float* out, int64_t n, W1 w,
                                                 int r, int edge, float pad, Ends1 ends) {
    constexpr int T = NT * 4;  // outputs per workgroup
    // (the last window read may reach past the taps by up to five floats)
    __shared__ __attribute__((aligned(16))) float s[T + 2 * SKEL_MAX_RADIUS_1D + 8];
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * T;
    const int staged = T + 2 * r;
    if (base - r >= 0 && base + T + r + 4 <= n) {
        // whole vectors at any alignment; the last may pass the halo by three
        const float* src = x + (base - r);
        constexpr int V = 1 + (2 * SKEL_MAX_RADIUS_1D + T - 1) / T;
        f32x4 v[V];
#pragma unroll
        for (int u = 0; u < V; ++u)
            if (4 * (tid + u * NT) < staged)
                v[u] = *reinterpret_cast<const f32x4u*>(src + 4 * (tid + u * NT));
#pragma unroll
        for (int u = 0; u < V; ++u)
            if (4 * (tid + u * NT) < staged) *reinterpret_cast<f32x4*>(s + 4 * (tid + u * NT)) = v[u];
    } else {
        for (int k = tid; k < staged; k += NT) s[k] = fetch1(x, n, base - r + k, edge, pad);
    }
    __syncthreads();
    const f32x4* win = reinterpret_cast<const f32x4*>(s) + tid;
    f32x4 lo = win[0];
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const auto taps = [&](int k, auto count) {
        const f32x4 hi = win[k / 4 + 1];
        const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
        for (int t = 0; t < decltype(count)::value; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = __builtin_fmaf(w.w[k + t], v[c + t], acc[c]);
        lo = hi;
    };
    int k = 0;
#pragma unroll 2
    for (; k + 4 <= 2 * r + 1; k += 4) taps(k, std::integral_constant<int, 4>());
    if (r & 1) taps(k, std::integral_constant<int, 3>());  // 2r + 1 is odd: 3 or 1 remain
    else taps(k, std::integral_constant<int, 1>());
    if constexpr (ENDS) {
        const int l = dev::lane(), mine = tid - l;  // first lane of this wavefront
        const int reach = n - 1 < r ? (int)(n - 1) : r;
        if (base == 0 && mine == 0) {
            float p = 0.0f;
            for (int i = l; i <= reach; i += dev::kWave) p = __builtin_fmaf(ends.lo[i], s[r + i], p);
            p = dev::wave_reduce<dev::Comb<float, SKEL_SUM>>(p);
            if (!__builtin_isfinite(p))
                p = dev::wave_reduce<dev::Comb<float, SKEL_SUM>>(end_terms<false>(
                    w, r, n, [&](int64_t i) { return s[r + (int)i]; }, l, dev::kWave));
            if (l == 0) acc[0] = p;
        }
        const int64_t e = n - 1 - base;  // the last element, if this tile holds it
        if (e < T && e / 4 / dev::kWave == mine / dev::kWave) {
            float p = 0.0f;
            for (int m = l; m <= reach; m += dev::kWave)
                p = __builtin_fmaf(ends.hi[m], s[(int)e + r - m], p);
            p = dev::wave_reduce<dev::Comb<float, SKEL_SUM>>(p);
            if (!__builtin_isfinite(p))
                p = dev::wave_reduce<dev::Comb<float, SKEL_SUM>>(end_terms<true>(
                    w, r, n, [&](int64_t i) { return s[(int)(i - base) + r]; }, l, dev::kWave));
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (4 * tid + c == (int)e) acc[c] = p;
        }
    }
    const int64_t i = base + 4 * tid;
    if (i + 4 <= n) {
        *reinterpret_cast<f32x4*>(out + i) = f32x4{acc[0], acc[1], acc[2], acc[3]};
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (i + c < n) out[i + c] = acc[c];
    }
}

// O1c: no LDS and no barrier.  Each wavefront owns kShflRows consecutive rows
// of 256 outputs (one 16-byte vector per lane per row, every row's load
// issued before any arithmetic); the r <= 4 neighbours on either side of a
// lane's vector come from the adjacent lanes by cross-lane shuffles, a row's
// end lanes take theirs from the adjacent row's end lane, and the first and
// last lanes of the group read one extra vector each (from cache).  Groups
// that touch the array ends take the scalar path.
// rows of 64 vectors per wavefront: one measured fastest in the bench step
// (5-point stencil on 2^26 floats: 103 us with one row, 112 with two or four,
// 123 with eight); more rows mean fewer, longer-lived wavefronts
#ifndef SKEL_O1C_ROWS
#define SKEL_O1C_ROWS 1
#endif
constexpr int kShflRows = SKEL_O1C_ROWS;

template <int RT, bool ENDS>
__global__ __launch_bounds__(kBlock) void ov1_shfl(const float* x, float* out, int64_t n, W1 w,
                                                   int r_, int edge, float pad, Ends1 ends) {
    constexpr int MR = RT >= 0 ? RT : 4;
    constexpr int U = kShflRows;
    const int r = RT >= 0 ? RT : r_;
    const int l = dev::lane();
    // this wavefront's U consecutive rows of 64 x 4 elements
    const int64_t wb0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x - l) * 4 * U;
    if (wb0 >= n) return;
    const bool interior = wb0 - 4 >= 0 && wb0 + 4 * dev::kWave * U + 4 <= n;
    if (interior) {
        const f32x4* xv = reinterpret_cast<const f32x4*>(x + wb0);
        f32x4 c[U];
#pragma unroll
        for (int k = 0; k < U; ++k) c[k] = xv[k * dev::kWave + l];  // all loads in flight
        f32x4 edge_l = {0.f, 0.f, 0.f, 0.f}, edge_r = {0.f, 0.f, 0.f, 0.f};
        if (l == 0) edge_l = xv[-1];
        if (l == dev::kWave - 1) edge_r = xv[U * dev::kWave];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            // neighbours: adjacent lanes of the same row; at the row ends, the
            // adjacent row's end lane (or the extra halo vectors)
            const f32x4 prev = k > 0 ? c[k - 1] : edge_l;
            const f32x4 next = k + 1 < U ? c[k + 1] : edge_r;
            // register-only moves: lane 0 takes the previous row's last vector
            // (or the halo), lane 63 the next row's first (or the halo)
            const f32x4 lt = dev::wave_shift_up(
                c[k], k > 0 ? dev::lane_value(prev, dev::kWave - 1) : edge_l);
            const f32x4 rt = dev::wave_shift_down(c[k], k + 1 < U ? dev::lane_value(next, 0)
                                                                  : edge_r);
            const float v[12] = {lt.x, lt.y, lt.z, lt.w, c[k].x, c[k].y, c[k].z, c[k].w,
                                 rt.x, rt.y, rt.z, rt.w};
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk <= 2 * MR; ++kk) {
                if (kk > 2 * r) break;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[q] = __builtin_fmaf(w.w[kk], v[4 + q + kk - r], acc[q]);
            }
            // plain store: measured faster than non-temporal here (5-point
            // stencil on 2^26 floats: 96 us against 103 us)
            reinterpret_cast<f32x4*>(out + wb0)[k * dev::kWave + l] =
                f32x4{acc[0], acc[1], acc[2], acc[3]};
        }
    } else {
        for (int k = 0; k < U; ++k) {
            const int64_t wb = wb0 + (int64_t)k * 4 * dev::kWave;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = wb + 4 * l + q;
                if (i >= n) break;
                float acc = 0.0f;
                for (int kk = 0; kk <= 2 * r; ++kk)
                    acc = __builtin_fmaf(w.w[kk], fetch1(x, n, i + kk - r, edge, pad), acc);
                if constexpr (ENDS) {
                    if (i == 0 || i == n - 1) {
                        acc = 0.0f;
                        for (int m = 0; m <= r && m < n; ++m)
                            acc = i == 0 ? __builtin_fmaf(ends.lo[m], x[m], acc)
                                         : __builtin_fmaf(ends.hi[m], x[n - 1 - m], acc);
                        if (!__builtin_isfinite(acc)) {
                            const auto at = [&](int64_t e) { return x[e]; };
                            acc = i == 0 ? end_terms<false>(w, r, n, at, 0, 1)
                                         : end_terms<true>(w, r, n, at, 0, 1);
                        }
                    }
                }
                out[i] = acc;
            }
        }
    }
}

// ------------------------------------------------------------------- 2D
constexpr int kTX = 64;  // columns of an output tile (LDS variants)

// compile-time radii of the direct form, or (-1, -1) for any radius
template <int RY, int RX>
struct Rad {
    static constexpr bool dyn = RY < 0;
    static constexpr int MY = dyn ? SKEL_MAX_RADIUS_2D : RY;
    static constexpr int MX = dyn ? SKEL_MAX_RADIUS_2D : RX;
};

// The LDS variants know the column radius at compile time (their inner loops
// run along a row) and take the row radius at run time (their outer loops run
// down the rows), so every pair of radii has straight-line inner loops.
template <int RX>
struct Cols {
    static constexpr int HX = (RX + 3) / 4 * 4;  // column halo rounded to 16 bytes
    static constexpr int LW = kTX + 2 * HX;      // LDS row width of the input tile
    static constexpr int NV = (4 + 2 * HX) / 4;  // 16-byte vectors a lane's 4 outputs read
};
constexpr int kHW = kTX + 4;  // LDS row width of a row-filtered tile (padded)

// workgroup b of the nb that take tiles t0 .. t0 + nb - 1 -> (tile x, tile y), in
// an XCD-contiguous order: the first nb % 8 XCDs take one tile more than the
// others.  (A grid rounded up to whole turns of the XCDs launches up to seven
// idle workgroups per image: 16384 images of 16 x 16, 5-point, 270 us against 37.)
__device__ __forceinline__ void tile_coords(uint32_t b, int64_t nbx, uint32_t nb, int64_t t0,
                                            int64_t& bx, int64_t& by) {
    const uint32_t xcd = b & 7, more = nb & 7;
    const uint32_t L = xcd * (nb >> 3) + (xcd < more ? xcd : more) + (b >> 3);
    if (t0 == 0) {  // (a 64-bit division would cost every workgroup its start)
        by = L / (uint32_t)nbx;
        bx = L - (uint32_t)by * (uint32_t)nbx;
    } else {
        by = (t0 + L) / nbx;
        bx = t0 + L - by * nbx;
    }
}

// four consecutive columns starting at j of row rp, through the column rule
__device__ __forceinline__ f32x4 fetch_row4(const float* rp, int64_t cols, int64_t j, int edge,
                                            float pad) {
    if (j >= 0 && j + 4 <= cols) return *reinterpret_cast<const f32x4u*>(rp + j);
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int64_t c;
        v[q] = border_near(j + q, cols, edge, c) ? rp[c] : pad;
    }
    return f32x4{v[0], v[1], v[2], v[3]};
}

// the same of row i, through the row rule too
__device__ __forceinline__ f32x4 fetch4(const float* x, int64_t rows, int64_t cols, int64_t i,
                                        int64_t j, int edge, float pad) {
    int64_t a;
    if (!border_near(i, rows, edge, a)) return f32x4{pad, pad, pad, pad};
    return fetch_row4(x + a * cols, cols, j, edge, pad);
}

// Stage nrows rows from y0 - ry and columns [x0 - HX, x0 + kTX + HX) of the
// input into LDS (row stride Cols::LW), as 16-byte vectors at any alignment of
// the rows; four loads in flight per lane.  Vectors that no output reads (past
// a ragged last column or row and its halo) are left alone.
template <int RX>
__device__ __forceinline__ void stage_tile(const float* x, int64_t rows, int64_t cols, int64_t y0,
                                           int64_t x0, int nrows, int ry, int edge, float pad,
                                           float* tin) {
    using CL = Cols<RX>;
    constexpr int V = CL::LW / 4;
    const bool interior = y0 - ry >= 0 && y0 - ry + nrows <= rows && x0 - CL::HX >= 0 &&
                          x0 + kTX + CL::HX <= cols;
    const auto batch = [&](auto load) {
        for (int k0 = threadIdx.x; k0 < nrows * V; k0 += 4 * kBlock) {
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + u * kBlock, rr = k / V;
                if (k < nrows * V) v[u] = load(rr, 4 * (k - rr * V));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k0 + u * kBlock < nrows * V)
                    *reinterpret_cast<f32x4*>(tin + 4 * (k0 + u * kBlock)) = v[u];
        }
    };
    if (interior) {
        const float* src = x + (y0 - ry) * cols + (x0 - CL::HX);
        batch([&](int rr, int cc) {
            return *reinterpret_cast<const f32x4u*>(src + (int64_t)rr * cols + cc);
        });
    } else {
        batch([&](int rr, int cc) {
            const int64_t i = y0 - ry + rr, j = x0 - CL::HX + cc;
            if (i >= rows + ry || j >= cols + RX) return f32x4{0.f, 0.f, 0.f, 0.f};
            return fetch4(x, rows, cols, i, j, edge, pad);
        });
    }
}

// The transpose of a clamped 2D map is the zero-padded correlation with
// reversed weights except on the first and last rows and columns, which also
// collect the reads past them.  Workgroups 0 .. nbb - 1 of a transposed launch
// of the tile forms compute those pixels (and the tiles leave them out), so
// that they run beside the tiles; the marching form, whose registers have no
// room for either, is followed by a launch of its own (ov2_border).  A border pixel of row 0 weighs row i by the
// sum of the weight rows a <= ry - i, one of the last row by the sum of a >= ry
// + m (i = rows - 1 - m), and likewise along the columns; the row sums are
// tabulated in LDS, the column sums of the corner columns run along.  kBorderG
// lanes share a pixel's row terms, combined by a fixed butterfly.
// Measured on CLAMP transposes against a gather of every border pixel's taps in
// a second launch: that launch took 11.6 us of the 9 x 9 transpose on 4096^2, 4.7
// on 24 fields of 121 x 163 and 30 on 64 of 2048^2 (5-point); beside the tiles
// the first two cost nothing measurable, the last (own launch) 12 us.
constexpr int kBorderG = 4;
constexpr int64_t kMaxBorderGroups = 1 << 20;  // (they take further pixels in turns)
constexpr int kBorderTab = (2 * SKEL_MAX_RADIUS_2D + 1) * (2 * SKEL_MAX_RADIUS_2D + 1) +
                           2 * (SKEL_MAX_RADIUS_2D + 1) * (2 * SKEL_MAX_RADIUS_2D + 1);

__device__ __forceinline__ int64_t border_pixels(int64_t rows, int64_t cols) {
    return (rows > 1 ? 2 : 1) * cols + (cols > 1 ? 2 : 1) * (rows > 2 ? rows - 2 : 0);
}

// outputs along an axis of len elements whose tap a (radius r) reads element s
// under CLAMP: lo .. hi
__device__ __forceinline__ void clamped_reads(int64_t s, int a, int r, int64_t len, int64_t& lo,
                                              int64_t& hi) {
    const int64_t i = s - a + r;
    lo = s == 0 || i < 0 ? 0 : i;
    hi = s == len - 1 || i > len - 1 ? len - 1 : i;
}

__device__ __forceinline__ void border_transposed(const float* g, float* dx, int64_t rows,
                                                  int64_t cols, const W2& w, int ry, int rx,
                                                  int groups, float* tab) {
    const int nx = 2 * rx + 1, ny = 2 * ry + 1;
    float* lo = tab + ny * nx;
    float* hi = lo + (ry + 1) * nx;
    // w holds the reversed weights: W[a][b] = w.w[last - (a * nx + b)]
    const int lastw = ny * nx - 1;
    for (int q = threadIdx.x; q <= lastw; q += kBlock) tab[q] = w.w[lastw - q];
    for (int q = threadIdx.x; q < (ry + 1) * nx; q += kBlock) {
        const int i = q / nx, b = q - i * nx;
        float sl = 0.0f, sh = 0.0f;
        for (int a = 0; a < ny; ++a) {
            const float wab = w.w[lastw - (a * nx + b)];
            if (rows == 1 || a <= ry - i) sl += wab;
            if (a >= ry + i) sh += wab;
        }
        lo[q] = sl;
        hi[q] = sh;
    }
    __syncthreads();
    const int lg = threadIdx.x % kBorderG;
    const int64_t pixels = border_pixels(rows, cols), nrow = rows > 1 ? 2 : 1;
    constexpr int64_t kPer = kBlock / kBorderG;  // pixels per workgroup and turn
    for (int64_t p0 = blockIdx.x * kPer; p0 < pixels; p0 += groups * kPer) {
        const int64_t p = p0 + threadIdx.x / kBorderG;
        const bool live = p < pixels;  // (the butterfly needs every lane)
        int64_t s = 0, t = 0;
        if (live && p < nrow * cols) {
            s = p < cols ? 0 : rows - 1;
            t = p < cols ? p : p - cols;
        } else if (live) {
            const int64_t q = p - nrow * cols;
            s = 1 + (cols > 1 ? q >> 1 : q);
            t = cols > 1 && (q & 1) ? cols - 1 : 0;
        }
        // row terms: table row k weighs input row i0 + di * k
        const float* tr = s == 0 ? lo : s == rows - 1 ? hi : tab;
        const int64_t i0 = s == 0 ? 0 : s == rows - 1 ? rows - 1 : s + ry;
        const int di = s == 0 ? 1 : -1, terms = s == 0 || s == rows - 1 ? ry + 1 : ny;
        float acc = 0.0f;
        for (int k = live ? lg : terms; k < terms; k += kBorderG) {
            const int64_t i = i0 + di * k;
            if (i < 0 || i >= rows) continue;
            const float* rk = tr + k * nx;
            const float* gi = g + i * cols;
            if (cols == 1) {
                float c = 0.0f;
                for (int b = 0; b < nx; ++b) c += rk[b];
                acc = __builtin_fmaf(c, gi[0], acc);
            } else if (t == 0 || t == cols - 1) {
                // input column m from the edge, farthest first: the weights that
                // reach the edge from it add up
                const int dir = t == 0 ? 1 : -1;
                const float* wm = t == 0 ? rk : rk + 2 * rx;  // weight of column m: wm[dir * (rx - m)]
                const float* gm = gi + t;                     // column m: gm[dir * m]
                float c = 0.0f;
                int m = rx;
                for (; m >= cols; --m) c += wm[dir * (rx - m)];
#pragma unroll 4
                for (; m >= 0; --m) {
                    c += wm[dir * (rx - m)];
                    acc = __builtin_fmaf(c, gm[dir * m], acc);
                }
            } else if (t >= rx && t + rx < cols) {
                const float* gj = gi + t + rx;
#pragma unroll 4
                for (int b = 0; b < nx; ++b) acc = __builtin_fmaf(rk[b], gj[-b], acc);
            } else {
                for (int b = 0; b < nx; ++b) {
                    const int64_t j = t + rx - b;
                    if (j >= 0 && j < cols) acc = __builtin_fmaf(rk[b], gi[j], acc);
                }
            }
        }
#pragma unroll
        for (int o = kBorderG >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        // an infinity or a NaN must meet each weight, not their sums (which may be
        // zero or of another sign): such a pixel is gathered tap by tap
        if (live && lg == 0 && !__builtin_isfinite(acc)) {
            acc = 0.0f;
            for (int q = 0; q <= lastw; ++q) {
                const int a = q / nx, b = q - a * nx;
                int64_t ilo, ihi, jlo, jhi;
                clamped_reads(s, a, ry, rows, ilo, ihi);
                clamped_reads(t, b, rx, cols, jlo, jhi);
                for (int64_t i = ilo; i <= ihi; ++i)
                    for (int64_t j = jlo; j <= jhi; ++j)
                        acc = __builtin_fmaf(tab[q], g[i * cols + j], acc);
            }
        }
        if (live && lg == 0) dx[s * cols + t] = acc;
    }
}

template <int RY, int RX>
__global__ __launch_bounds__(kBlock) void ov2_direct(const float* x, float* out, int64_t rows,
                                                     int64_t cols, W2 w, int ry_, int rx_,
                                                     int edge, float pad, int64_t nbx) {
    // blockIdx.y: one of several equally shaped images stored back to back
    x += (int64_t)blockIdx.y * rows * cols;
    out += (int64_t)blockIdx.y * rows * cols;
    using RD = Rad<RY, RX>;
    const int ry = RD::dyn ? ry_ : RY, rx = RD::dyn ? rx_ : RX;
    const int wx = 2 * rx + 1;
    const int64_t j = (blockIdx.x % nbx) * 64 + threadIdx.x % 64;
    const int64_t i = (blockIdx.x / nbx) * 4 + threadIdx.x / 64;
    if (i >= rows || j >= cols) return;
    float acc = 0.0f;
    const bool interior = i - ry >= 0 && i + ry < rows && j - rx >= 0 && j + rx < cols;
#pragma unroll
    for (int a = 0; a <= 2 * RD::MY; ++a) {
        if (a > 2 * ry) break;
#pragma unroll
        for (int b = 0; b <= 2 * RD::MX; ++b) {
            if (b > 2 * rx) break;
            const float v = interior ? x[(i + a - ry) * cols + (j + b - rx)]
                                     : fetch2(x, rows, cols, i + a - ry, j + b - rx, edge, pad);
            acc = __builtin_fmaf(w.w[a * wx + b], v, acc);
        }
    }
    out[i * cols + j] = acc;
}

__global__ __launch_bounds__(kBlock) void ov2_border(const float* g, float* dx, int64_t rows,
                                                     int64_t cols, W2 w, int ry, int rx) {
    __shared__ float tab[kBorderTab];
    border_transposed(g + (int64_t)blockIdx.y * rows * cols, dx + (int64_t)blockIdx.y * rows * cols,
                      rows, cols, w, ry, rx, (int)gridDim.x, tab);
}

// store one 4-wide output segment of row i starting at column j (inner: leave
// out the first and last rows and columns, see border_transposed)
__device__ __forceinline__ void store4(float* out, int64_t rows, int64_t cols, int64_t i,
                                       int64_t j, const float (&v)[4], bool inner) {
    if (i >= rows || (inner && (i == 0 || i == rows - 1))) return;
    const bool whole = j + 4 <= cols && !(inner && (j == 0 || j + 4 == cols));
    if (whole && (cols & 3) == 0) {
        // non-temporal: measured faster than plain stores for the 2D tiles
        // (9x9 separable on 4096^2: 42 us against 46 us)
        dev::store_vec_nt(f32x4{v[0], v[1], v[2], v[3]},
                          reinterpret_cast<f32x4*>(out + i * cols + j));
    } else if (whole) {
        // (plain: neighbouring lanes share the lines of an unaligned row)
        *reinterpret_cast<f32x4u*>(out + i * cols + j) = f32x4{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (j + c < cols && !(inner && (j + c == 0 || j + c == cols - 1)))
                out[i * cols + j + c] = v[c];
    }
}

// O2b.  What bounds it from radius 2 on is the vector ALU: one multiply-add per
// tap and output (unpacked), the weights in scalar registers, 4 x RO outputs
// per lane so that a row read from LDS feeds RO output rows.  RO: rows per lane
// (a tile has 16 * RO rows).  Measured, map and clamped transpose together,
// against 64-row tiles with run-time column radii, element-wise staging of
// unaligned rows and border tiles, and a second launch for the border pixels:
// dense 7 x 7 on 1501 x 1999 83 -> 24 us, on 4096^2 242 -> 84; 17 x 17 on 4096^2
// 720 -> 295 (its multiply-adds alone: 247); 5-point on 24 fields of 121 x 163
// 21.5 -> 9.1.
template <int RX, int RO>
__global__ __launch_bounds__(kBlock) void ov2_lds(const float* x, float* out, int64_t rows,
                                                  int64_t cols, W2 w, int ry, int edge, float pad,
                                                  int64_t nbx, int64_t nb, int64_t t0, int nbb) {
    // blockIdx.y: one of several equally shaped images stored back to back
    x += (int64_t)blockIdx.y * rows * cols;
    out += (int64_t)blockIdx.y * rows * cols;
    static_assert(RO == 1 || RO == 2, "the row loop below");
    using CL = Cols<RX>;
    constexpr int NX = 2 * RX + 1, LW = CL::LW;
    extern __shared__ __attribute__((aligned(16))) float tin[];
    const int nbl = t0 == 0 ? nbb : 0;  // border workgroups of this launch
    if ((int)blockIdx.x < nbl) {
        border_transposed(x, out, rows, cols, w, ry, RX, nbl, tin);
        return;
    }
    int64_t bx, by;
    tile_coords(blockIdx.x - nbl, nbx, (uint32_t)nb, t0, bx, by);
    const int64_t y0 = by * (16 * RO), x0 = bx * kTX;
    stage_tile<RX>(x, rows, cols, y0, x0, 16 * RO + 2 * ry, ry, edge, pad, tin);
    __syncthreads();
    const int cg = threadIdx.x % 16, rg = threadIdx.x / 16;
    float acc[RO][4];
#pragma unroll
    for (int o = 0; o < RO; ++o)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[o][c] = 0.0f;
    // input row k of the lane's window contributes to output row o with weight
    // row k - o: to both rows of a pair but for the first and last k
    const float* win = tin + RO * rg * LW + 4 * cg;
    const auto row_of = [&](int k, float (&seg)[4 * CL::NV]) {
#pragma unroll
        for (int v = 0; v < CL::NV; ++v) {
            const f32x4 q = *reinterpret_cast<const f32x4*>(win + k * LW + 4 * v);
            seg[4 * v] = q.x;
            seg[4 * v + 1] = q.y;
            seg[4 * v + 2] = q.z;
            seg[4 * v + 3] = q.w;
        }
    };
    const auto add = [&](float (&o)[4], const float* wr, const float (&seg)[4 * CL::NV]) {
#pragma unroll
        for (int b = 0; b < NX; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) o[c] = __builtin_fmaf(wr[b], seg[CL::HX - RX + b + c], o[c]);
    };
    float seg[4 * CL::NV];
    row_of(0, seg);
    add(acc[0], w.w, seg);
    for (int k = 1; k <= 2 * ry; ++k) {
        row_of(k, seg);
        add(acc[0], w.w + k * NX, seg);
        if constexpr (RO == 2) add(acc[1], w.w + (k - 1) * NX, seg);
    }
    if constexpr (RO == 2) {
        row_of(2 * ry + 1, seg);
        add(acc[1], w.w + 2 * ry * NX, seg);
    }
#pragma unroll
    for (int o = 0; o < RO; ++o)
        store4(out, rows, cols, y0 + RO * rg + o, x0 + 4 * cg, acc[o], nbb > 0);
}

// the column pass of the separable tiles: RO output rows per lane from the
// row-filtered tile th (row stride kHW)
template <int RO>
__device__ __forceinline__ void column_pass(const float* th, const W2& w, int ry, int rg, int cg,
                                            float (&acc)[RO][4]) {
#pragma unroll
    for (int o = 0; o < RO; ++o)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[o][c] = 0.0f;
    // filtered row k contributes to output row o with weight k - o
    const float* win = th + RO * rg * kHW + 4 * cg;
    const auto add = [&](float (&o)[4], float wa, f32x4 v) {
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = __builtin_fmaf(wa, v[c], o[c]);
    };
    add(acc[0], w.wy[0], *reinterpret_cast<const f32x4*>(win));
#pragma unroll 4
    for (int k = 1; k <= 2 * ry; ++k) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(win + k * kHW);
        add(acc[0], w.wy[k], v);
        if constexpr (RO == 2) add(acc[1], w.wy[k - 1], v);
    }
    if constexpr (RO == 2)
        add(acc[1], w.wy[2 * ry], *reinterpret_cast<const f32x4*>(win + (2 * ry + 1) * kHW));
}

// O2c: the staged tile filtered along its rows into a second LDS buffer
template <int RX, int RO>
__global__ __launch_bounds__(kBlock) void ov2_sep(const float* x, float* out, int64_t rows,
                                                  int64_t cols, W2 w, int ry, int edge, float pad,
                                                  int64_t nbx, int64_t nb, int64_t t0, int nbb) {
    // blockIdx.y: one of several equally shaped images stored back to back
    x += (int64_t)blockIdx.y * rows * cols;
    out += (int64_t)blockIdx.y * rows * cols;
    using CL = Cols<RX>;
    constexpr int LW = CL::LW;
    extern __shared__ __attribute__((aligned(16))) float tin[];
    const int nbl = t0 == 0 ? nbb : 0;  // border workgroups of this launch
    if ((int)blockIdx.x < nbl) {
        border_transposed(x, out, rows, cols, w, ry, RX, nbl, tin);
        return;
    }
    const int nrows = 16 * RO + 2 * ry;
    float* th = tin + nrows * LW;
    int64_t bx, by;
    tile_coords(blockIdx.x - nbl, nbx, (uint32_t)nb, t0, bx, by);
    const int64_t y0 = by * (16 * RO), x0 = bx * kTX;
    stage_tile<RX>(x, rows, cols, y0, x0, nrows, ry, edge, pad, tin);
    __syncthreads();
    const int cg = threadIdx.x % 16, rg = threadIdx.x / 16;
    // row pass: th[y][x] = sum_b wx[b] * in[y][x + b - rx] for all staged rows
    for (int y = rg; y < nrows; y += 16) {
        const float* row = tin + y * LW + 4 * cg;
        float seg[4 * CL::NV];
#pragma unroll
        for (int v = 0; v < CL::NV; ++v) {
            const f32x4 q = *reinterpret_cast<const f32x4*>(row + 4 * v);
            seg[4 * v] = q.x;
            seg[4 * v + 1] = q.y;
            seg[4 * v + 2] = q.z;
            seg[4 * v + 3] = q.w;
        }
        f32x4 h = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b <= 2 * RX; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                h[c] = __builtin_fmaf(w.wx[b], seg[CL::HX - RX + b + c], h[c]);
        *reinterpret_cast<f32x4*>(th + y * kHW + 4 * cg) = h;
    }
    __syncthreads();
    float acc[RO][4];
    column_pass<RO>(th, w, ry, rg, cg, acc);
#pragma unroll
    for (int o = 0; o < RO; ++o)
        store4(out, rows, cols, y0 + RO * rg + o, x0 + 4 * cg, acc[o], nbb > 0);
}

// O2d: separable, with the row pass read straight from global memory through
// the L1 cache (each lane loads its 4 + 2*HX inputs as 16-byte vectors;
// neighbouring lanes' overlaps hit L1), so LDS holds only the row-pass result
// of a 64 x 16*RO tile.  The small LDS footprint allows full occupancy, and the
// low tiles keep many workgroups in flight.  Measured as O2b: 7 x 7 on 1501 x 1999
// 97 -> 25 us, on 4096^2 440 -> 68; 9 x 9 on 4096^2 80 -> 73 (the map 36, the
// transpose 36 + 12 for its border before).
template <int RX, int RO>
// (eight wavefronts per SIMD for radii up to 4: 64 registers where 66 would
// leave seven; 8192^2 9 x 9, map and transpose, 230 -> 225 us)
__global__ __launch_bounds__(kBlock, RX <= 4 ? 8 : 1) void ov2_sep_l1(const float* x, float* out, int64_t rows,
                                                     int64_t cols, W2 w, int ry, int edge,
                                                     float pad, int64_t nbx, int64_t nb, int64_t t0, int nbb) {
    // blockIdx.y: one of several equally shaped images stored back to back
    x += (int64_t)blockIdx.y * rows * cols;
    out += (int64_t)blockIdx.y * rows * cols;
    using CL = Cols<RX>;
    constexpr int HX = CL::HX, NV = CL::NV;
    extern __shared__ __attribute__((aligned(16))) float th[];
    const int nbl = t0 == 0 ? nbb : 0;  // border workgroups of this launch
    if ((int)blockIdx.x < nbl) {
        border_transposed(x, out, rows, cols, w, ry, RX, nbl, th);
        return;
    }
    int64_t bx, by;
    tile_coords(blockIdx.x - nbl, nbx, (uint32_t)nb, t0, bx, by);
    const int64_t y0 = by * (16 * RO), x0 = bx * kTX;
    const int nrows = 16 * RO + 2 * ry;
    const bool interior = y0 - ry >= 0 && y0 - ry + nrows <= rows && x0 - HX >= 0 &&
                          x0 + kTX + HX <= cols;
    const int cg = threadIdx.x % 16, rg = threadIdx.x / 16;
    // row pass: every row this lane handles is loaded before any arithmetic
    // (kIt rows of NV 16-byte vectors in flight per lane)
    constexpr int kIt = RO + 1;  // covers 16 * RO + 2 * ry rows, 2 * ry <= 16
    static_assert(2 * SKEL_MAX_RADIUS_2D <= 16, "rows of the row pass");
    f32x4 seg[kIt][NV];
    if (interior) {
        const float* src = x + (y0 - ry + rg) * cols + (x0 - HX + 4 * cg);
#pragma unroll
        for (int it = 0; it < kIt; ++it)
            if (rg + 16 * it < nrows)
#pragma unroll
                for (int v = 0; v < NV; ++v)
                    seg[it][v] = *reinterpret_cast<const f32x4u*>(src + 16 * it * cols + 4 * v);
    } else {
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int64_t i = y0 - ry + rg + 16 * it;
            if (rg + 16 * it >= nrows) continue;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int64_t j = x0 - HX + 4 * (cg + v);
                seg[it][v] = i >= rows + ry || j >= cols + RX
                                 ? f32x4{0.f, 0.f, 0.f, 0.f}
                                 : fetch4(x, rows, cols, i, j, edge, pad);
            }
        }
    }
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        const int y = rg + 16 * it;
        if (y >= nrows) continue;
        f32x4 h = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b <= 2 * RX; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int e = HX - RX + b + c;
                h[c] = __builtin_fmaf(w.wx[b], seg[it][e / 4][e % 4], h[c]);
            }
        *reinterpret_cast<f32x4*>(th + y * kHW + 4 * cg) = h;
    }
    __syncthreads();
    float acc[RO][4];
    column_pass<RO>(th, w, ry, rg, cg, acc);
#pragma unroll
    for (int o = 0; o < RO; ++o)
        store4(out, rows, cols, y0 + RO * rg + o, x0 + 4 * cg, acc[o], nbb > 0);
}

// O2e.  A workgroup's four wavefronts take four vertically stacked strips,
// so the ry halo rows that one strip shares with the next are read from
// cache.  Input row m of a strip (row i0 - ry + m of the image) feeds output
// rows m - a of the strip with weight row a; output row o accumulates in ring
// slot o mod (2ry+1), which is stored and cleared once row o + 2ry is in.
// What bounds it is how many rows a wavefront has in flight: all rows of a
// chunk are loaded before the first is used.  Measured (5-point stencil on
// 64 fields of 2048^2; strip rows / chunk rows): 32/9 394 us, 16/9 378,
// 64/9 397, 32/18 433, 16/18 (the whole strip) 358, O2b 428.  A dense 9 x 9
// needs 24 rows for a 16-row strip, more than the registers hold: 64-row
// strips in chunks of 18 rows are used there (on 4096^2, back to back with
// the image in the Infinity Cache: 67 us, 16-row strips 90; evicted, all of
// them lose to O2b, which the plan therefore keeps for radii above 2).
constexpr int kMarchCols = 4 * dev::kWave;    // columns per strip
constexpr int kMarchMaxR = 4;                 // radius reach of one neighbour lane
// With a run-time column radius (radii other than 1, 2 or 4 in both
// directions) the tap loop is longer, and whole-strip chunks spill; those
// instances load about eight rows at a time (one ring of 7 for radius 3,
// where two rings spill).
template <int RY, bool DYN>
struct March {
    static constexpr int NW = 2 * RY + 1;                       // ring slots
    static constexpr int rows = RY <= 2 ? 16 : 64;              // output rows per strip
    static constexpr int chunk = DYN ? (RY == 3 ? NW : NW * ((8 + NW - 1) / NW))
                               : RY <= 2 ? rows + 2 * RY : 2 * NW;  // rows loaded at once
    static_assert(chunk % NW == 0 && (rows + 2 * RY) % chunk == 0, "whole chunks per strip");
};

// four consecutive columns starting at j of row rp, through the column rule
__device__ __forceinline__ f32x4 march_chunk(const float* rp, int64_t cols, int64_t j,
                                             bool aligned, int edge, float pad) {
    if (aligned && j >= 0 && j + 4 <= cols) return *reinterpret_cast<const f32x4*>(rp + j);
    float v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int64_t c;
        v[q] = border(j + q, cols, edge, c) ? rp[c] : pad;
    }
    return f32x4{v[0], v[1], v[2], v[3]};
}

// Add loaded row m of a strip (held in ring position t = m mod (2ry+1)) into
// the output rows it feeds, then store output row m - 2ry, now complete, and
// clear its slot for row m + 1.  c: this lane's four columns; e: the chunk
// beyond the strip's end read by lanes 0 (left) and 63 (right).  SEP: the
// weights are factors, so the row is filtered once with wx and the result
// added with wy[a] (the LDS separable variants' order of operations).
// vec_store: the lane's four columns are inside the row and 16-byte aligned.
template <int RY, int MX, bool SEP>
__device__ __forceinline__ void march_row(float (&acc)[2 * RY + 1][4], int t, int m, f32x4 c,
                                          f32x4 e, const W2& w, int rx, float* out,
                                          int64_t i0, int64_t j, int64_t cols, bool vec_store) {
    constexpr int NW = 2 * RY + 1;
    const int nx = 2 * rx + 1;
    const f32x4 lt = dev::wave_shift_up(c, e), rt = dev::wave_shift_down(c, e);
    const float v[12] = {lt.x, lt.y, lt.z, lt.w, c.x, c.y, c.z, c.w, rt.x, rt.y, rt.z, rt.w};
    if constexpr (SEP) {
        float h[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int d = -MX; d <= MX; ++d) {
            if (d < -rx || d > rx) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) h[q] = __builtin_fmaf(w.wx[d + rx], v[4 + q + d], h[q]);
        }
#pragma unroll
        for (int a = 0; a < NW; ++a) {
            const int s = ((t - a) % NW + NW) % NW;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[s][q] = __builtin_fmaf(w.wy[a], h[q], acc[s][q]);
        }
    } else {
#pragma unroll
        for (int a = 0; a < NW; ++a) {
            const int s = ((t - a) % NW + NW) % NW;
#pragma unroll
            for (int d = -MX; d <= MX; ++d) {
                if (d < -rx || d > rx) continue;
                const float wab = w.w[a * nx + d + rx];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[s][q] = __builtin_fmaf(wab, v[4 + q + d], acc[s][q]);
            }
        }
    }
    const int sd = (t + 1) % NW;
    if (m >= 2 * RY) {
        float* op = out + (i0 + m - 2 * RY) * cols;
        if (vec_store) {
            dev::store_vec_nt(f32x4{acc[sd][0], acc[sd][1], acc[sd][2], acc[sd][3]},
                              reinterpret_cast<f32x4*>(op + j));
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (j + q < cols) op[j + q] = acc[sd][q];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[sd][q] = 0.0f;
}

template <int RY, int RX, bool SEP>
__global__ __launch_bounds__(kBlock) void ov2_march(const float* x, float* out, int64_t rows,
                                                    int64_t cols, W2 w, int rx_, int edge,
                                                    float pad, int64_t nbx) {
    // blockIdx.y: one of several equally shaped images stored back to back
    x += (int64_t)blockIdx.y * rows * cols;
    out += (int64_t)blockIdx.y * rows * cols;
    using M = March<RY, (RX < 0)>;
    constexpr int NW = M::NW, CH = M::chunk, kMarchRows = M::rows;
    constexpr int MX = RX >= 0 ? RX : kMarchMaxR;
    const int rx = RX >= 0 ? RX : rx_;
    const int l = dev::lane();
    const int64_t bx = (int64_t)blockIdx.x % nbx, by = (int64_t)blockIdx.x / nbx;
    const int64_t j0 = bx * kMarchCols;
    const int64_t i0 = (by * (kBlock / dev::kWave) + threadIdx.x / dev::kWave) * kMarchRows;
    if (i0 >= rows) return;  // whole wavefronts; no barrier follows
    const int64_t j = j0 + 4 * l;
    const bool aligned = (cols & 3) == 0;
    const int nout = (int)(rows - i0 < kMarchRows ? rows - i0 : kMarchRows);
    const int nin = nout + 2 * RY;
    // the chunk the edge lanes read beyond the strip: left of it for lane 0,
    // right of it for lane 63 (other lanes re-read their own chunk)
    const int64_t je = l == 0 ? j0 - 4 : l == dev::kWave - 1 ? j0 + kMarchCols : j;
    float acc[NW][4];
#pragma unroll
    for (int s = 0; s < NW; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[s][q] = 0.0f;
    int m0 = 0;
    // fast path: the strip lies inside the row, so every row is two
    // unconditional 16-byte loads per lane.  Rows beyond the image ends (at
    // most ry <= rows away) and the edge chunks beyond the row ends map by the
    // edge rule without branches: cyclic reads the chunk at the other end,
    // clamp repeats the row's end value, const takes the pad.
    if (aligned && j0 + kMarchCols <= cols && rows >= kMarchMaxR) {
        const bool lo = l == 0 && j0 == 0, hi = l == dev::kWave - 1 && j0 + kMarchCols == cols;
        const bool efix = (lo || hi) && edge != SKEL_EDGE_CYCLIC;
        const int64_t jf = lo ? cols - 4 : hi ? 0 : je;
        const int64_t jr = efix ? j : jf;
        for (; m0 + CH <= nin; m0 += CH) {
            f32x4 c[CH], e[CH];
            bool in[CH];
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const int64_t k = i0 - RY + m0 + t;
                in[t] = k >= 0 && k < rows;
                const int64_t kk = in[t] ? k
                                 : edge == SKEL_EDGE_CYCLIC ? (k < 0 ? k + rows : k - rows)
                                 : (k < 0 ? 0 : rows - 1);
                c[t] = *reinterpret_cast<const f32x4*>(x + kk * cols + j);
                e[t] = *reinterpret_cast<const f32x4*>(x + kk * cols + jr);
            }
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                if (edge == SKEL_EDGE_CONST && !in[t]) {
                    c[t] = f32x4{pad, pad, pad, pad};
                    e[t] = c[t];
                }
                if (efix) {
                    const float b = edge == SKEL_EDGE_CONST ? pad : lo ? c[t].x : c[t].w;
                    e[t] = f32x4{b, b, b, b};
                }
                march_row<RY, MX, SEP>(acc, t % NW, m0 + t, c[t], e[t], w, rx, out, i0, j, cols,
                                       true);
            }
        }
    } else if (rows >= kMarchMaxR) {
        // a strip past a ragged row end, or rows not 16-byte aligned: the
        // column rule is the same for every row, so each lane maps its four
        // columns and the edge chunk once; rows are then straight-line element
        // loads from valid addresses, with the pad selected afterwards
        int64_t ci[4], ei[4];
        bool cp[4], ep[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int64_t cc;
            cp[q] = !border(j + q, cols, edge, cc);
            ci[q] = cp[q] ? 0 : cc;
            ep[q] = !border(je + q, cols, edge, cc);
            ei[q] = ep[q] ? 0 : cc;
        }
        const bool vec_store = aligned && j + 4 <= cols;
        for (; m0 + CH <= nin; m0 += CH) {
            float cv[CH][4], ev[CH][4];
            bool in[CH];
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const int64_t k = i0 - RY + m0 + t;
                in[t] = k >= 0 && k < rows;
                const int64_t kk = in[t] ? k
                                 : edge == SKEL_EDGE_CYCLIC ? (k < 0 ? k + rows : k - rows)
                                 : (k < 0 ? 0 : rows - 1);
                const float* rp = x + kk * cols;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    cv[t][q] = rp[ci[q]];
                    ev[t][q] = rp[ei[q]];
                }
            }
#pragma unroll
            for (int t = 0; t < CH; ++t) {
                const bool padrow = edge == SKEL_EDGE_CONST && !in[t];
                float c[4], e[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    c[q] = padrow || cp[q] ? pad : cv[t][q];
                    e[q] = padrow || ep[q] ? pad : ev[t][q];
                }
                march_row<RY, MX, SEP>(acc, t % NW, m0 + t, f32x4{c[0], c[1], c[2], c[3]},
                                       f32x4{e[0], e[1], e[2], e[3]}, w, rx, out, i0, j, cols,
                                       vec_store);
            }
        }
    }
    // general path: the last strip of an image whose height is not a whole
    // number of strips, and images of fewer than four rows
    for (; m0 < nin; m0 += NW) {
#pragma unroll
        for (int t = 0; t < NW; ++t) {
            const int m = m0 + t;
            if (m >= nin) break;
            int64_t kk;
            f32x4 c = {pad, pad, pad, pad}, e = {pad, pad, pad, pad};
            if (border(i0 - RY + m, rows, edge, kk)) {
                const float* rp = x + kk * cols;
                c = march_chunk(rp, cols, j, aligned, edge, pad);
                if (l == 0 || l == dev::kWave - 1)
                    e = march_chunk(rp, cols, je, aligned, edge, pad);
            }
            march_row<RY, MX, SEP>(acc, t, m, c, e, w, rx, out, i0, j, cols,
                                   aligned && j + 4 <= cols);
        }
    }
}

// --------------------------------------------------------------- launchers
int64_t div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <int NT>
void run1d_window(const float* x, float* out, int64_t n, const W1& w, int r, int edge, float pad,
                  const Ends1* ends, hipStream_t st) {
    const unsigned grid = (unsigned)div_up(n, NT * 4);
    if (ends) ov1_window<NT, true><<<grid, NT, 0, st>>>(x, out, n, w, r, edge, pad, *ends);
    else ov1_window<NT, false><<<grid, NT, 0, st>>>(x, out, n, w, r, edge, pad, Ends1());
}

template <int RT>
skel_status run1d(int v, const float* x, float* out, int64_t n, const W1& w, int r, int edge,
                  float pad, const Ends1* ends, hipStream_t st) {
    if (v == O1A_DIRECT) {
        ov1_direct<RT><<<(unsigned)div_up(n, kBlock), kBlock, 0, st>>>(x, out, n, w, r, edge, pad);
        return launch_check("overlap1d_direct");
    }
    // selectable for r <= 4 only
    const unsigned grid = (unsigned)div_up(n, 4 * kBlock * kShflRows);
    if (ends) ov1_shfl<RT, true><<<grid, kBlock, 0, st>>>(x, out, n, w, r, edge, pad, *ends);
    else ov1_shfl<RT, false><<<grid, kBlock, 0, st>>>(x, out, n, w, r, edge, pad, Ends1());
    return launch_check("overlap1d_shuffle");
}

// One launch over `fields` images.  nbb: workgroups per image for the border
// pixels of a clamped transpose (0: the plain map).
struct Call2 {
    const float* x;
    float* out;
    int64_t rows, cols;
    unsigned fields;
    const W2& w;
    bool sep;
    int ry, rx, edge;
    float pad;
    int nbb;
    int cus;
    hipStream_t st;
};

template <int RY, int RX, bool SEP>
void march_launch(const Call2& c) {
    const int64_t nbx = div_up(c.cols, kMarchCols);
    const int64_t nb = nbx * div_up(c.rows, March<RY, (RX < 0)>::rows * (kBlock / dev::kWave));
    ov2_march<RY, RX, SEP><<<dim3((unsigned)nb, c.fields), kBlock, 0, c.st>>>(
        c.x, c.out, c.rows, c.cols, c.w, c.rx, c.edge, c.pad, nbx);
}

template <int RY, int RX>
void march_form(const Call2& c) {
    if (c.sep) march_launch<RY, RX, true>(c);
    else march_launch<RY, RX, false>(c);
}

// selectable for ry, rx <= 4 only
skel_status run2d_march(const Call2& c) {
    if (c.ry == c.rx && (c.ry == 1 || c.ry == 2 || c.ry == 4)) {
        if (c.ry == 1) march_form<1, 1>(c);
        else if (c.ry == 2) march_form<2, 2>(c);
        else march_form<4, 4>(c);
        return launch_check("overlap2d_march");
    }
    switch (c.ry) {
    case 0: march_form<0, -1>(c); break;
    case 1: march_form<1, -1>(c); break;
    case 2: march_form<2, -1>(c); break;
    case 3: march_form<3, -1>(c); break;
    case 4: march_form<4, -1>(c); break;
    default: return SKEL_E_UNSUPPORTED;
    }
    return launch_check("overlap2d_march");
}

template <int RY, int RX>
skel_status run2d_direct(const Call2& c) {
    const int64_t nbx = div_up(c.cols, 64), nby = div_up(c.rows, 4);
    ov2_direct<RY, RX><<<dim3((unsigned)(nbx * nby), c.fields), kBlock, 0, c.st>>>(
        c.x, c.out, c.rows, c.cols, c.w, c.ry, c.rx, c.edge, c.pad, nbx);
    return launch_check("overlap2d_direct");
}

// grid and LDS of one tile launch; bytes_per_row: LDS per row of the tile
template <class K>
void tile_launch(K kern, int ro, size_t bytes_per_row, const Call2& c) {
    const int64_t nbx = div_up(c.cols, kTX), nb = nbx * div_up(c.rows, 16 * ro);
    size_t lds = (16 * ro + 2 * c.ry) * bytes_per_row;
    if (c.nbb) lds = std::max(lds, kBorderTab * sizeof(float));
    // (one launch, but for an image of more tiles than a launch has workgroups)
    const int64_t most = (max_groups(kBlock) - c.nbb) / 8 * 8;
    for (int64_t t0 = 0; t0 < nb; t0 += most) {
        const int64_t here = std::min(nb - t0, most);
        kern<<<dim3((unsigned)(here + (t0 == 0 ? c.nbb : 0)), c.fields), kBlock, lds, c.st>>>(
            c.x, c.out, c.rows, c.cols, c.w, c.ry, c.edge, c.pad, nbx, here, t0, c.nbb);
    }
}

// Rows per lane (a tile has 16 times as many).  One row per lane keeps more
// workgroups in flight, whose loads overlap other workgroups' arithmetic; two
// share a row's LDS reads and halo.  With 16 workgroups per CU left at two rows
// (2^23 pixels) the second is level or better, below it the first (map and
// transpose, one / two rows per lane: 200 x 300 5-point 8.4 / 10.6 us, dense
// 17 x 17 21.6 / 27.2; 1501 x 1999 dense 9 x 9 30.4 / 34.1, separable 25.9 /
// 32.7; 4096^2 5-point 63.5 / 58.6, dense 9 x 9 116 / 112).  Four and eight
// rows per lane and tiles of 128 and 256 columns measured slower (4096^2 dense
// 9 x 9: 115-153 us).
template <int RX>
skel_status tile_form(int v, const Call2& c) {
    const int64_t tiles = div_up(c.cols, kTX) * div_up(c.rows, 16) * c.fields;
    const bool two = tiles >= 32 * (int64_t)c.cus;
    constexpr size_t in_row = Cols<RX>::LW * sizeof(float), th_row = kHW * sizeof(float);
    if (v == O2B_LDS_TILE) {
        if (two) tile_launch(ov2_lds<RX, 2>, 2, in_row, c);
        else tile_launch(ov2_lds<RX, 1>, 1, in_row, c);
        return launch_check("overlap2d_lds");
    }
    if (v == O2C_LDS_SEPARABLE) {
        if (two) tile_launch(ov2_sep<RX, 2>, 2, in_row + th_row, c);
        else tile_launch(ov2_sep<RX, 1>, 1, in_row + th_row, c);
        return launch_check("overlap2d_separable");
    }
    if (two) tile_launch(ov2_sep_l1<RX, 2>, 2, th_row, c);
    else tile_launch(ov2_sep_l1<RX, 1>, 1, th_row, c);
    return launch_check("overlap2d_separable_l1");
}

skel_status run2d_tile(int v, const Call2& c) {
    switch (c.rx) {
    case 0: return tile_form<0>(v, c);
    case 1: return tile_form<1>(v, c);
    case 2: return tile_form<2>(v, c);
    case 3: return tile_form<3>(v, c);
    case 4: return tile_form<4>(v, c);
    case 5: return tile_form<5>(v, c);
    case 6: return tile_form<6>(v, c);
    case 7: return tile_form<7>(v, c);
    case 8: return tile_form<8>(v, c);
    default: return SKEL_E_UNSUPPORTED;
    }
}

skel_status run2d(int v, const Call2& c) {
    if (v == O2E_MARCH) {
        const skel_status e = run2d_march(c);
        if (e != SKEL_OK || !c.nbb) return e;
        ov2_border<<<dim3(c.nbb, c.fields), kBlock, 0, c.st>>>(c.x, c.out, c.rows, c.cols, c.w,
                                                               c.ry, c.rx);
        return launch_check("overlap2d_border");
    }
    if (v != O2A_DIRECT) return run2d_tile(v, c);
    if (c.ry == 4 && c.rx == 4) return run2d_direct<4, 4>(c);
    if (c.ry == 1 && c.rx == 1) return run2d_direct<1, 1>(c);
    if (c.ry == 2 && c.rx == 2) return run2d_direct<2, 2>(c);
    return run2d_direct<-1, -1>(c);
}

skel_status run2d_fields(int v, Call2 c, int64_t fields) {
    const int64_t img = c.rows * c.cols;
    for (int64_t f0 = 0; f0 < fields; f0 += kMaxFieldsPerLaunch) {
        c.fields = (unsigned)std::min<int64_t>(fields - f0, kMaxFieldsPerLaunch);
        const skel_status e = run2d(v, c);
        if (e != SKEL_OK) return e;
        c.x += kMaxFieldsPerLaunch * img;
        c.out += kMaxFieldsPerLaunch * img;
    }
    return SKEL_OK;
}

}  // namespace

static skel_status launch_1d(int v, const float* x, float* out, int64_t n, const W1& wk, int r,
                             int edge, float pad, const Ends1* ends, LaunchCtx& lc) {
    if (v == O1B_LDS_TILE) {
        // short arrays: one wavefront per workgroup, which spreads them over more
        // CUs (2^12 floats, radius 16, map and transpose: 6.3 us against 7.3; 2^16:
        // 6.2 / 6.5; from 2^18 on the smaller halo share of 256 lanes is level or
        // better, 2^20 radius 64: 17.2 against 17.9)
        if (n <= (INT64_C(1) << 17)) run1d_window<64>(x, out, n, wk, r, edge, pad, ends, lc.stream);
        else run1d_window<256>(x, out, n, wk, r, edge, pad, ends, lc.stream);
        return launch_check("overlap1d_window");
    }
    switch (r) {
    case 1: return run1d<1>(v, x, out, n, wk, r, edge, pad, ends, lc.stream);
    case 2: return run1d<2>(v, x, out, n, wk, r, edge, pad, ends, lc.stream);
    case 3: return run1d<3>(v, x, out, n, wk, r, edge, pad, ends, lc.stream);
    case 4: return run1d<4>(v, x, out, n, wk, r, edge, pad, ends, lc.stream);
    default: return run1d<-1>(v, x, out, n, wk, r, edge, pad, ends, lc.stream);
    }
}

skel_status launch_overlap1d(int v, const float* x, float* out, int64_t n, const float* w,
                             int r, int edge, float pad, LaunchCtx& lc) {
    W1 wk{};
    for (int k = 0; k <= 2 * r; ++k) wk.w[k] = w[k];
    return launch_1d(v, x, out, n, wk, r, edge, pad, nullptr, lc);
}

skel_status launch_overlap1d_transposed(const float* g, float* dx, int64_t n, const float* w,
                                        int r, int edge, LaunchCtx& lc) {
    W1 wk{};
    for (int k = 0; k <= 2 * r; ++k) wk.w[k] = w[2 * r - k];
    const int v = r <= 4 ? O1C_SHUFFLE : O1B_LDS_TILE;
    if (edge != SKEL_EDGE_CLAMP)
        return launch_1d(v, g, dx, n, wk, r, edge, 0.0f, nullptr, lc);
    // tap k of output i reads element i + k - r: element 0 collects the taps
    // k <= r - i of output i, element n - 1 the taps k >= r + m of output
    // n - 1 - m (a single element: every tap)
    Ends1 ends{};
    double lo = 0.0, hi = 0.0;
    for (int i = r; i >= 0; --i) {
        lo += w[r - i];
        hi += w[r + i];
        ends.lo[i] = (float)lo;
        ends.hi[i] = (float)hi;
    }
    if (n == 1) ends.lo[0] = ends.hi[0] = (float)(lo + hi - w[r]);
    return launch_1d(v, g, dx, n, wk, r, SKEL_EDGE_CONST, 0.0f, &ends, lc);
}

skel_status launch_overlap2d(int v, const float* x, float* out, int64_t rows, int64_t cols,
                             int64_t fields, const float* w2d, const float* wy, const float* wx,
                             int ry, int rx, int edge, float pad, LaunchCtx& lc) {
    W2 wk{};
    const int ny = 2 * ry + 1, nx = 2 * rx + 1;
    for (int a = 0; a < ny; ++a)
        for (int b = 0; b < nx; ++b)
            wk.w[a * nx + b] = w2d ? w2d[a * nx + b] : wy[a] * wx[b];
    if (!w2d) {
        for (int a = 0; a < ny; ++a) wk.wy[a] = wy[a];
        for (int b = 0; b < nx; ++b) wk.wx[b] = wx[b];
    }
    const Call2 c{x, out, rows, cols, 0, wk, !w2d, ry, rx, edge, pad, 0, lc.dev->cus, lc.stream};
    return run2d_fields(v, c, fields);
}

skel_status launch_overlap2d_transposed(const float* g, float* dx, int64_t rows, int64_t cols,
                                        int64_t fields, const float* w2d, const float* wy,
                                        const float* wx, int ry, int rx, int edge, LaunchCtx& lc) {
    W2 wk{};
    const int ny = 2 * ry + 1, nx = 2 * rx + 1;
    for (int a = 0; a < ny; ++a)
        for (int b = 0; b < nx; ++b)
            wk.w[(ny - 1 - a) * nx + (nx - 1 - b)] = w2d ? w2d[a * nx + b] : wy[a] * wx[b];
    if (!w2d) {
        for (int a = 0; a < ny; ++a) wk.wy[a] = wy[ny - 1 - a];
        for (int b = 0; b < nx; ++b) wk.wx[b] = wx[nx - 1 - b];
    }
    const int64_t n = fields * rows * cols;
    const int r = ry > rx ? ry : rx;
    const int v = w2d ? overlap2d_dense_variant(n, rows, cols, r)
                      : overlap2d_separable_variant(n, rows, cols, r);
    // A clamped map of radii up to 1 whose weights mirror along both axes is its
    // own transpose: along an axis it is w1 I + w0 (down + up), and the shifts
    // down and up, each with its clamped end, add up to a symmetric matrix (the
    // diagonal entries of the two ends, the off-diagonals 1).  Every output is a
    // sum of the same products, and no border has to be gathered (64 images of
    // 2048^2, 5-point: a launch of 23 us in the kernel trace; a training pass
    // over them 2117 -> 2077 us).  At radius 2 the clamped shifts are not
    // symmetric (row 1 reads element 0 at distance 2, row 0 never reads row 1
    // at that distance).
    const auto mirrored = [](const float* w, int n, int step) {
        return w[0] == w[(n - 1) * step];
    };
    bool self = edge == SKEL_EDGE_CLAMP && ry <= 1 && rx <= 1;
    if (w2d) {
        for (int a = 0; self && a < ny; ++a) self = mirrored(w2d + a * nx, nx, 1);
        for (int b = 0; self && b < nx; ++b) self = mirrored(w2d + b, ny, nx);
    } else if (self) {
        self = mirrored(wy, ny, 1) && mirrored(wx, nx, 1);
    }
    int nbb = 0;
    if (edge == SKEL_EDGE_CLAMP && !self)
        nbb = (int)std::min(div_up(((rows > 1 ? 2 : 1) * cols +
                                    (cols > 1 ? 2 : 1) * (rows > 2 ? rows - 2 : 0)) * kBorderG,
                                   kBlock),
                            kMaxBorderGroups);
    const Call2 c{g, dx, rows, cols, 0, wk, !w2d, ry, rx,
                  edge == SKEL_EDGE_CYCLIC || self ? edge : SKEL_EDGE_CONST, 0.0f, nbb,
                  lc.dev->cus, lc.stream};
    return run2d_fields(v, c, fields);
}

}  // namespace skel

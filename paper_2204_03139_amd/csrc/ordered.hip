// Exact nearest neighbours of Sec. III-A (Eq. 1/2) over spatially ordered clouds: the result of the
// exhaustive fp32 search (the smallest canonical distance, the smallest index among its ties) with
// most pairs ruled out by bounding boxes instead of evaluated.
//
// k_order puts each cloud of each frame into the order of a space-filling curve and bounds it: 32
// consecutive points form a block with a box, 64 blocks a super-block with a box.  k_near gives
// each wave 64 consecutive (so nearby) ordered queries, one per lane.  The wave visits the
// super-blocks, and in them the blocks, whose boxes lie no further from its queries' box than the
// worst lane's best distance so far; a block that at least one lane cannot rule out by its own
// distance to the box is screened on the matrix cores (two instructions for its 32 points and all 64
// queries), and the 16 points (sub-tile) that may hold a query's smallest distance are evaluated at
// the end.  k_near_shared, for calls with too few query waves for the chip, evaluates the blocks
// themselves, the points read through the scalar cache.
//
// Exactness.  Subtraction, multiplication and fma round monotonically, and the distance to a box
// uses the operations of the canonical distance on the gaps between the query and the box, which
// are no larger in magnitude than the differences to any point in the box.  So the float distance
// to a box is never above the canonical float distance to any of its points, and a box is skipped
// only when it is strictly above the best: no minimum and no tie is lost.  A screened value has a
// bound on its error, and every sub-tile within it of the least is kept.  The kept sub-tiles are read
// again for the smallest canonical distance and its smallest original index; a lane that has more of
// them than it remembers, or in k_near_shared met its minimum in two sub-tiles, is searched again.  A
// box of zero size holds one point repeated: its distance and least index stand for the whole block.
// Points with a NaN coordinate are in no box: they are no targets, and queries of their own kind.
//
// What it costs and what bounds it (100 frames of 65,536 x 65,536, both directions).  k_near: 1.20 ms.  A
// wave screens 20 of 2,048 blocks (640 of 65,536 pairs per query; the least possible for these blocks
// is 17 to 21) in 3,390 vector instructions; the waits of six waves per SIMD bound it as much as
// their issue.  With the blocks evaluated, at 6.5 instructions per pair and 6,500 per wave, it took
// 1.72 ms, bound by vector issue; the exhaustive searches of the same frames 53.9 ms (fp32) and
// 25.2 ms (bf16 screen and its refine).  Targets on a sphere about all queries, where no box rules
// anything out and the screen settles nothing, are the exhaustive fp32 search's to win (20 frames: 20.7 ms
// against 10.9; the bf16 screen took 37 to 69).  Ordering: 0.28 ms, of which 0.17 ms deals out the points, 13 million 16-byte stores
// at random inside a cloud's megabyte.  On one frame a wave's chain of dependent loads bounds it: 106
// us, 56 us with four waves to a query wave.
#include <algorithm>

#include "batch.h"

namespace dc {
namespace {

constexpr int OB = 32;                 // points of a block
constexpr int OSUB = 16;               // points of a sub-tile, half a block
// points in scalar registers at once: with 8 the 100-frame search by evaluated blocks takes 1.75 ms,
// with 4 (which the compiler chooses by itself) or 16 (registers spill) about 0.2 ms more
constexpr int OLOAD = 8;
constexpr int OSUPER = 64;             // blocks of a super-block
constexpr int OSUPER_PTS = OB * OSUPER;
constexpr int OBOX = 7 * OSUPER;        // words of a super-block's boxes
constexpr int ORD_THREADS = 1024;
constexpr int ORD_WAVES = ORD_THREADS / 64;
constexpr int ORD_SMALL = 16384;       // points that one workgroup orders by itself
constexpr int ORD_SMALL_BITS = 13;
constexpr int ORD_BITS = 15;           // most bits of a curve position
constexpr int ORD_PART = 32768;        // most points of a part: its counts fit 16 bits
constexpr int ORD_AXIS_BITS = 8;       // most bits of one axis (the spread tables' 256 entries)
constexpr float ORD_FINITE = 1e15f;    // coordinates beyond this don't take part in the range

typedef float nfloat4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) nfloat4 *scalar_f4;
typedef const __attribute__((address_space(4))) float *scalar_f;

__device__ __forceinline__ float canon_gap(float dx, float dy, float dz) {
    return __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
}

// largest value over the 64 lanes (in every lane)
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_f(float v) {
    const int i = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, ROWS, 0xF, false));
}

__device__ __forceinline__ float lane63(float v) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// the same value in every lane, kept in a scalar register
__device__ __forceinline__ float uniform_float(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_f<0x111, 0xF>(v));  // row_shr:1
    v = fmaxf(v, dpp_f<0x112, 0xF>(v));  // row_shr:2
    v = fmaxf(v, dpp_f<0x114, 0xF>(v));  // row_shr:4
    v = fmaxf(v, dpp_f<0x118, 0xF>(v));  // row_shr:8
    v = fmaxf(v, dpp_f<0x142, 0xA>(v));  // row_bcast:15
    v = fmaxf(v, dpp_f<0x143, 0xC>(v));  // row_bcast:31
    return lane63(v);
}

__device__ __forceinline__ float wave_min(float v) { return -wave_max(-v); }


// The cells of a cloud: a coordinate's cell along its axis, and the cells' bits at their places in
// the curve position.
struct OrderCells {
    float lo[3], scale[3], top[3];
    unsigned spread[3][1 << ORD_AXIS_BITS];
};

// One cloud of every frame: its points, and where its order and boxes go.
struct OrderCloud {
    const float *src;  // [T,N,3]
    nfloat4 *pts;      // [T,npad]: (x, y, z, original index bits), padding NaN with index -1
    float *box;        // [T][supers][7][64]: min x, y, z, max x, y, z and the least index (bits)
                       // of the super's blocks
    float *sbox;       // [T][super chunks][6][64]: the same of 64 super-blocks
    // larger clouds only
    unsigned *cnt;     // [T][parts][2^bits] points per part and cell, 16 bits each
    unsigned *start;   // [T][parts][2^bits] the first position of a part's points of a cell; then
                       // [T] OrderCells; then [T][parts][OC_CHUNKS] points per chunk of cells
    unsigned short *rank;  // [T][N] a point's place among its part's points of its cell
    int n, part;       // points; points per part
    int bits, parts;   // of a curve position; of the cloud
};

struct OrderParams {
    OrderCloud c[2];
};

__device__ __forceinline__ OrderCells *cells_of(const OrderCloud &c, int T, int t) {
    return reinterpret_cast<OrderCells *>(c.start + ((size_t)T * c.parts << c.bits)) + t;
}

// points padded to whole query waves
__host__ __device__ __forceinline__ int order_npad(int n) { return (n + 63) & ~63; }
__host__ __device__ __forceinline__ int order_blocks(int n) { return order_npad(n) / OB; }
__host__ __device__ __forceinline__ int order_supers(int n) {
    return (order_npad(n) + OSUPER_PTS - 1) / OSUPER_PTS;
}

// sum over the 64 lanes (in every lane)
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_or_zero(float v) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
}

__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_or_zero<0x111, 0xF>(v);  // row_shr:1
    v += dpp_or_zero<0x112, 0xF>(v);  // row_shr:2
    v += dpp_or_zero<0x114, 0xF>(v);  // row_shr:4
    v += dpp_or_zero<0x118, 0xF>(v);  // row_shr:8
    v += dpp_or_zero<0x142, 0xA>(v);  // row_bcast:15
    v += dpp_or_zero<0x143, 0xC>(v);  // row_bcast:31
    return lane63(v);
}

// The cells of one cloud, worked out by one wave (the result in every lane's registers).
//
// The range comes from 256 of the points, spread over the cloud, after three rounds of dropping
// points more than 5 standard deviations out: a few stray points must not stretch the cells of all
// others (they fall into the outermost cells).  The bits of a curve position are dealt to the axis
// whose cells are longest at the time, most significant bit first, so cells stay as near to cubes
// as halving allows whatever the cloud's proportions.
struct CellPlan {
    float lo[3], scale[3];
    int ab[3];                 // bits of each axis
    int axis[ORD_BITS];        // the axis of each bit, most significant first
};

__device__ __forceinline__ CellPlan plan_cells(const float *src, int n, int bits, int lane) {
    constexpr int S = 4;  // samples per lane
    const float inf = __builtin_inff();
    float s[S][3];
    bool keep[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int k = u * 64 + lane;
        const int i = n <= 64 * S ? min(k, n - 1) : (int)((long)k * n / (64 * S));
        const float *p = src + 3 * (size_t)i;
        s[u][0] = p[0];
        s[u][1] = p[1];
        s[u][2] = p[2];
        keep[u] = fabsf(s[u][0]) < ORD_FINITE && fabsf(s[u][1]) < ORD_FINITE &&
                  fabsf(s[u][2]) < ORD_FINITE;
    }
    float piv[3] = {0.f, 0.f, 0.f};
    for (int round = 0; round < 4; ++round) {
        float d[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < S; ++u) {
            d[6] += keep[u] ? 1.f : 0.f;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float v = keep[u] ? s[u][k] - piv[k] : 0.f;
                d[k] += v;
                d[3 + k] += v * v;
            }
        }
#pragma unroll
        for (int k = 0; k < 7; ++k) d[k] = wave_sum(d[k]);
        const float inv = 1.f / fmaxf(d[6], 1.f);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float m = d[k] * inv;
            const float var = fmaxf(d[3 + k] * inv - m * m, 0.f);
            piv[k] += m;
            // the first round only finds a pivot, for accurate variances
            if (round > 0)
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    const float off = s[u][k] - piv[k];
                    if (off * off > 25.f * var) keep[u] = false;
                }
        }
    }
    CellPlan c;
    float e[3], ext[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        float l = inf, h = -inf;
#pragma unroll
        for (int u = 0; u < S; ++u) {
            l = fminf(l, keep[u] ? s[u][k] : inf);
            h = fmaxf(h, keep[u] ? s[u][k] : -inf);
        }
        l = wave_min(l);
        h = wave_max(h);
        if (!(l <= h)) l = h = 0.f;  // nothing kept: one cell
        c.lo[k] = l;
        e[k] = ext[k] = h - l;
        c.ab[k] = 0;
    }
#pragma unroll
    for (int b = 0; b < ORD_BITS; ++b) {
        int a = 0;
        float w = c.ab[0] < ORD_AXIS_BITS ? e[0] : -1.f;
        if (c.ab[1] < ORD_AXIS_BITS && e[1] > w) {
            a = 1;
            w = e[1];
        }
        if (c.ab[2] < ORD_AXIS_BITS && e[2] > w) a = 2;
        c.axis[b] = a;
        if (b < bits) {
            c.ab[0] += a == 0;
            c.ab[1] += a == 1;
            c.ab[2] += a == 2;
        }
        e[0] = a == 0 ? 0.5f * e[0] : e[0];
        e[1] = a == 1 ? 0.5f * e[1] : e[1];
        e[2] = a == 2 ? 0.5f * e[2] : e[2];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        c.scale[k] = ext[k] > 0.f ? (float)(1 << c.ab[k]) / ext[k] : 0.f;
        if (!(c.scale[k] < inf)) c.scale[k] = 0.f;
    }
    return c;
}

// the bits of axis k's cell v at their places in the curve position
__device__ __forceinline__ unsigned spread_bits(const CellPlan &c, int bits, int k, int v) {
    int used = 0;
    unsigned out = 0;
    for (int b = 0; b < bits; ++b)
        if (c.axis[b] == k) {
            ++used;
            out |= ((unsigned)(v >> (c.ab[k] - used)) & 1u) << (bits - 1 - b);
        }
    return out;
}

// The cells of a cloud into LDS, by a whole workgroup (ends in a barrier).
__device__ __forceinline__ void put_cells(const float *src, int n, int bits, OrderCells &o,
                                          CellPlan &plan) {
    if (threadIdx.x < 64) {
        const CellPlan c = plan_cells(src, n, bits, threadIdx.x);
        if (threadIdx.x == 0) {
            plan = c;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                o.lo[k] = c.lo[k];
                o.scale[k] = c.scale[k];
                o.top[k] = (float)((1 << c.ab[k]) - 1);
            }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 3 << ORD_AXIS_BITS; e += blockDim.x) {
        const int k = e >> ORD_AXIS_BITS;
        o.spread[k][e & ((1 << ORD_AXIS_BITS) - 1)] =
            spread_bits(plan, bits, k, e & ((1 << ORD_AXIS_BITS) - 1));
    }
    __syncthreads();
}

// A point's place on the curve: the interleaved bits taken as a Gray code, so that consecutive
// cells are neighbours (12% fewer pairs evaluated than in the plain interleaved order).
// A NaN coordinate falls into cell 0 of its axis.
__device__ __forceinline__ unsigned cell_of(const OrderCells &c, float x, float y, float z) {
    const float fx = fminf(fmaxf((x - c.lo[0]) * c.scale[0], 0.f), c.top[0]);
    const float fy = fminf(fmaxf((y - c.lo[1]) * c.scale[1], 0.f), c.top[1]);
    const float fz = fminf(fmaxf((z - c.lo[2]) * c.scale[2], 0.f), c.top[2]);
    unsigned g = c.spread[0][(int)fx] | c.spread[1][(int)fy] | c.spread[2][(int)fz];
    g ^= g >> 1;  // Gray code to rank
    g ^= g >> 2;
    g ^= g >> 4;
    g ^= g >> 8;
    return g;
}

__device__ __forceinline__ nfloat4 ordered_point(float x, float y, float z, int i) {
    nfloat4 v;
    v.x = x;
    v.y = y;
    v.z = z;
    v.w = __int_as_float(i);
    return v;
}

__device__ __forceinline__ nfloat4 padding_point() {
    const float nan = __builtin_nanf("");
    return ordered_point(nan, nan, nan, -1);
}

// the box of block `b` (of `nblk`) by four lanes, eight points each.  A point with a NaN coordinate is
// left out on every axis: its distances are NaN and never win, and a box that it stretched on its other
// axes might hold no point at all.
__device__ __forceinline__ void block_box(const nfloat4 *pts, int b, int nblk, int tid, float *box) {
    const float inf = __builtin_inff();
    float l[3] = {inf, inf, inf}, h[3] = {-inf, -inf, -inf};
    int least = 0x7fffffff;
    if (b < nblk) {
        nfloat4 v[OB / 4];
#pragma unroll
        for (int k = 0; k < OB / 4; ++k) v[k] = pts[(size_t)b * OB + 4 * k + (tid & 3)];
#pragma unroll
        for (int k = 0; k < OB / 4; ++k) {
            const bool whole = v[k].x == v[k].x && v[k].y == v[k].y && v[k].z == v[k].z;
            l[0] = fminf(l[0], whole ? v[k].x : inf);
            l[1] = fminf(l[1], whole ? v[k].y : inf);
            l[2] = fminf(l[2], whole ? v[k].z : inf);
            h[0] = fmaxf(h[0], whole ? v[k].x : -inf);
            h[1] = fmaxf(h[1], whole ? v[k].y : -inf);
            h[2] = fmaxf(h[2], whole ? v[k].z : -inf);
            if (whole) least = min(least, __float_as_int(v[k].w));
        }
    }
    least = min(least, __builtin_amdgcn_update_dpp(least, least, 0xB1, 0xF, 0xF, false));
    least = min(least, __builtin_amdgcn_update_dpp(least, least, 0x4E, 0xF, 0xF, false));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        l[k] = fminf(l[k], dpp_f<0xB1, 0xF>(l[k]));  // quad_perm [1,0,3,2]
        l[k] = fminf(l[k], dpp_f<0x4E, 0xF>(l[k]));  // quad_perm [2,3,0,1]
        h[k] = fmaxf(h[k], dpp_f<0xB1, 0xF>(h[k]));
        h[k] = fmaxf(h[k], dpp_f<0x4E, 0xF>(h[k]));
    }
    {
        const int k = tid & 3;
        float *o = box + (size_t)(b / OSUPER) * OBOX + b % OSUPER;
        if (k < 3) {
            o[k * OSUPER] = k == 0 ? l[0] : (k == 1 ? l[1] : l[2]);
            o[(3 + k) * OSUPER] = k == 0 ? h[0] : (k == 1 ? h[1] : h[2]);
        } else {
            o[6 * OSUPER] = __int_as_float(least);
        }
    }
}

// the box of super-block g by one wave
__device__ __forceinline__ void super_box(const float *box, int g, int lane, float *sbox) {
    float *o = sbox + (size_t)(g / 64) * 6 * 64 + g % 64;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const float v = box[(size_t)g * OBOX + k * OSUPER + lane];
        const float r = k < 3 ? wave_min(v) : wave_max(v);
        if (lane == 0) o[k * 64] = r;
    }
}

// the exclusive prefix of v over the wave's lanes, and (in `total`) the sum
__device__ __forceinline__ unsigned wave_prefix(unsigned v, int lane, unsigned &total) {
    unsigned incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    total = (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
    return incl - v;
}

constexpr int OC_CELLS = 4 * ORD_THREADS;  // cells of a scanning workgroup: a chunk
constexpr int OC_CHUNKS = (1 << ORD_BITS) / OC_CELLS;
__device__ __forceinline__ unsigned *totals_of(const OrderCloud &c, int T, int t) {
    return reinterpret_cast<unsigned *>(cells_of(c, T, T)) + (size_t)t * c.parts * OC_CHUNKS;
}

// A cloud of at most ORD_SMALL points (80 clouds of 8,192: 24 us, a chain of seven phases between
// barriers; the four launches of the larger clouds' path would take as long each): one workgroup counts its points by cell in LDS and deals
// them out.  Within a cell the order is whatever the atomics give: no result depends on it.
// Logical workgroup: x = cloud, y = frame.
__device__ __forceinline__ void order_small_body(const OrderParams &pr, const Blk &blk) {
    __shared__ unsigned cnt[1 << ORD_SMALL_BITS];
    __shared__ OrderCells cells;
    __shared__ CellPlan plan;
    __shared__ unsigned wsum[ORD_WAVES];
    const OrderCloud c = blk.x ? pr.c[1] : pr.c[0];
    const int t = blk.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = c.n, bits = c.bits;
    const float *src = c.src + (size_t)t * n * 3;
    nfloat4 *dst = c.pts + (size_t)t * order_npad(c.n);
    const int ncell = 1 << bits;
    constexpr int U = 4;  // points per thread in flight
    float p[U][3];
    auto load = [&](int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float *q = src + 3 * (size_t)min(i0 + u * ORD_THREADS, n - 1);
            p[u][0] = q[0];
            p[u][1] = q[1];
            p[u][2] = q[2];
        }
    };
    load(tid);
    for (int k = tid; k < ncell; k += ORD_THREADS) cnt[k] = 0;
    put_cells(src, n, bits, cells, plan);
    for (int i0 = tid; i0 < n; i0 += U * ORD_THREADS) {
        if (i0 != tid) load(i0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * ORD_THREADS < n)
                atomicAdd(&cnt[cell_of(cells, p[u][0], p[u][1], p[u][2])], 1u);
    }
    __syncthreads();
    {  // counts to starts: each wave scans a run of cells, 64 at a time
        const int per = max(ncell / ORD_WAVES, 64);
        const int c0 = wave * per;
        unsigned sum = 0;
        if (c0 < ncell)
            for (int k = lane; k < per; k += 64) sum += cnt[c0 + k];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (lane == 0) wsum[wave] = sum;
        __syncthreads();
        unsigned before = 0;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (c0 < ncell)
            for (int k = lane; k < per; k += 64) {
                unsigned total;
                const unsigned e = wave_prefix(cnt[c0 + k], lane, total);
                cnt[c0 + k] = before + e;
                before += total;
            }
        __syncthreads();
    }
    for (int i0 = tid; i0 < n; i0 += U * ORD_THREADS) {
        if (n > U * ORD_THREADS) load(i0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * ORD_THREADS;
            if (i < n)
                dst[atomicAdd(&cnt[cell_of(cells, p[u][0], p[u][1], p[u][2])], 1u)] =
                    ordered_point(p[u][0], p[u][1], p[u][2], i);
        }
    }
    for (int i = n + tid; i < order_npad(c.n); i += ORD_THREADS) dst[i] = padding_point();
    __syncthreads();  // the points are in place (this workgroup wrote them all)
    const int supers = order_supers(c.n);
    float *box = c.box + (size_t)t * supers * OBOX;
    for (int b = tid >> 2; b < supers * OSUPER; b += ORD_THREADS / 4)
        block_box(dst, b, order_blocks(c.n), tid, box);
    __syncthreads();
    float *sbox = c.sbox + (size_t)t * ((supers + 63) / 64) * 6 * 64;
    for (int g = wave; g < supers; g += ORD_WAVES) super_box(box, g, lane, sbox);
}

__global__ __launch_bounds__(ORD_THREADS) void k_order_small(OrderParams p) {
    order_small_body(p, grid_blk());
}

// Larger clouds, in four steps over parts of a cloud: counts per part and cell (and each point's
// place among its part's points of its cell), counts to starts, points dealt out, boxes.  Counting
// in LDS and not in memory: 13 million atomics on 200 clouds' counters in memory took 600 us.
constexpr int OC_THREADS = 256;
constexpr int OC_PER = 8;                       // points per thread
constexpr int OC_POINTS = OC_THREADS * OC_PER;  // points of a workgroup

// x = part, y = frame, z = cloud
__device__ __forceinline__ void order_count_body(const OrderParams &pr, const Blk &blk) {
    __shared__ unsigned cnt[1 << (ORD_BITS - 1)];  // two cells a word
    __shared__ unsigned chunk[OC_CHUNKS + 1];
    __shared__ OrderCells cells;
    __shared__ CellPlan plan;
    const OrderCloud c = blk.z ? pr.c[1] : pr.c[0];
    const int t = blk.y, tid = threadIdx.x;
    if (blk.x >= c.parts) return;
    const int base = blk.x * c.part;
    const int n = min(c.part, c.n - base);
    const int words = 1 << (c.bits - 1);
    for (int k = tid; k < words; k += ORD_THREADS) cnt[k] = 0;
    if (tid < OC_CHUNKS) chunk[tid] = 0;
    const float *cloud = c.src + (size_t)t * c.n * 3;
    put_cells(cloud, c.n, c.bits, cells, plan);
    if (blk.x == 0)
        for (int k = tid; k < (int)(sizeof(OrderCells) / 4); k += ORD_THREADS)
            reinterpret_cast<unsigned *>(cells_of(c, blk.gy, t))[k] = reinterpret_cast<const unsigned *>(&cells)[k];
    const float *src = cloud + 3 * (size_t)base;
    unsigned short *rank = c.rank + (size_t)t * c.n + base;
    constexpr int U = 8;  // points per thread in flight
    for (int i0 = tid; i0 < n; i0 += U * ORD_THREADS) {
        float p[U][3];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float *q = src + 3 * (size_t)min(i0 + u * ORD_THREADS, n - 1);
            p[u][0] = q[0];
            p[u][1] = q[1];
            p[u][2] = q[2];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * ORD_THREADS;
            if (i < n) {
                const unsigned g = cell_of(cells, p[u][0], p[u][1], p[u][2]);
                const unsigned sh = (g & 1u) * 16u;
                rank[i] = (unsigned short)(atomicAdd(&cnt[g >> 1], 1u << sh) >> sh);
            }
        }
    }
    __syncthreads();
    unsigned *out = c.cnt + ((size_t)t * c.parts + blk.x) * words;
    for (int k0 = 0; k0 < words; k0 += ORD_THREADS) {  // (a whole wave has words, or none)
        const int k = k0 + tid;
        unsigned sum = 0;
        if (k < words) {
            const unsigned w = cnt[k];
            out[k] = w;
            sum = (w & 0xFFFFu) + (w >> 16);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if ((tid & 63) == 0) atomicAdd(&chunk[k / (OC_CELLS / 2)], sum);
    }
    __syncthreads();
    if (tid < OC_CHUNKS) totals_of(c, blk.gy, t)[blk.x * OC_CHUNKS + tid] = chunk[tid];
}

__global__ __launch_bounds__(ORD_THREADS) void k_order_count(OrderParams p) {
    order_count_body(p, grid_blk_xcd());
}

// x = chunk of cells, y = frame, z = cloud: the starts of the chunk's cells in every part
__device__ __forceinline__ void order_scan_body(const OrderParams &pr, const Blk &blk) {
    __shared__ unsigned wsum[ORD_WAVES];
    __shared__ unsigned wpre[ORD_WAVES];
    const OrderCloud c = blk.z ? pr.c[1] : pr.c[0];
    const int t = blk.y;
    const int ncell = 1 << c.bits;
    if (blk.x * OC_CELLS >= ncell) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const size_t quads = (size_t)ncell / 4;  // four cells: two words of counts
    const uint2 *cnt = reinterpret_cast<const uint2 *>(c.cnt) + (size_t)t * c.parts * quads;
    const int at = blk.x * ORD_THREADS + tid;
    const bool ok = at < (int)quads;
    unsigned v[4] = {0, 0, 0, 0};
    auto add4 = [&](const uint2 &w, unsigned (&d)[4]) {
        d[0] += w.x & 0xFFFFu;
        d[1] += w.x >> 16;
        d[2] += w.y & 0xFFFFu;
        d[3] += w.y >> 16;
    };
    constexpr int U = 8;  // loads in flight
    if (ok)
        for (int k0 = 0; k0 < c.parts; k0 += U) {
            uint2 w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = cnt[min(k0 + u, c.parts - 1) * quads + at];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + u < c.parts) add4(w[u], v);
        }
    // the points in the cells before the chunk, over all parts
    unsigned sum = 0;
    const unsigned *tot = totals_of(c, blk.gy, t);
    for (int k = tid; k < c.parts * OC_CHUNKS; k += ORD_THREADS)
        if (k % OC_CHUNKS < blk.x) sum += tot[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    unsigned total;
    unsigned e = wave_prefix(v[0] + v[1] + v[2] + v[3], lane, total);
    if (lane == 0) {
        wsum[wave] = total;
        wpre[wave] = sum;
    }
    __syncthreads();
    for (int w = 0; w < ORD_WAVES; ++w) {
        e += wpre[w];
        if (w < wave) e += wsum[w];
    }
    if (!ok) return;
    uint4 s = make_uint4(e, e + v[0], e + v[0] + v[1], e + v[0] + v[1] + v[2]);
    uint4 *out = reinterpret_cast<uint4 *>(c.start) + (size_t)t * c.parts * quads;
    for (int k0 = 0; k0 < c.parts; k0 += U) {
        uint2 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = cnt[min(k0 + u, c.parts - 1) * quads + at];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + u < c.parts) {
                out[(k0 + u) * quads + at] = s;
                s.x += w[u].x & 0xFFFFu;
                s.y += w[u].x >> 16;
                s.z += w[u].y & 0xFFFFu;
                s.w += w[u].y >> 16;
            }
    }
}

__global__ __launch_bounds__(ORD_THREADS) void k_order_scan(OrderParams p) {
    order_scan_body(p, grid_blk_xcd());
}

__device__ __forceinline__ void stage_cells(const OrderCells *src, OrderCells &dst) {
    static_assert(sizeof(OrderCells) % 4 == 0, "whole words");
    for (int k = threadIdx.x; k < (int)(sizeof(OrderCells) / 4); k += OC_THREADS)
        reinterpret_cast<unsigned *>(&dst)[k] = reinterpret_cast<const unsigned *>(src)[k];
    __syncthreads();
}

// x = chunk of points, y = frame, z = cloud
__device__ __forceinline__ void order_deal_body(const OrderParams &pr, const Blk &blk) {
    __shared__ OrderCells cells;
    const OrderCloud c = blk.z ? pr.c[1] : pr.c[0];
    const int t = blk.y;
    const int i0 = blk.x * OC_POINTS + (int)threadIdx.x;
    if (blk.x * OC_POINTS >= order_npad(c.n)) return;
    const float *src = c.src + (size_t)t * c.n * 3;
    float p[OC_PER][3];
    unsigned r[OC_PER];
#pragma unroll
    for (int u = 0; u < OC_PER; ++u) {
        const int i = min(i0 + u * OC_THREADS, c.n - 1);
        const float *q = src + 3 * (size_t)i;
        p[u][0] = q[0];
        p[u][1] = q[1];
        p[u][2] = q[2];
        r[u] = c.rank[(size_t)t * c.n + i];
    }
    stage_cells(cells_of(c, blk.gy, t), cells);
    // the workgroup's points are of one part (a part is a whole number of workgroups)
    const int part = blk.x / (c.part / OC_POINTS);
    const unsigned *start = c.start + (((size_t)t * c.parts + min(part, c.parts - 1)) << c.bits);
#pragma unroll
    for (int u = 0; u < OC_PER; ++u) r[u] += start[cell_of(cells, p[u][0], p[u][1], p[u][2])];
    nfloat4 *dst = c.pts + (size_t)t * order_npad(c.n);
#pragma unroll
    for (int u = 0; u < OC_PER; ++u) {
        const int i = i0 + u * OC_THREADS;
        if (i < c.n)
            dst[r[u]] = ordered_point(p[u][0], p[u][1], p[u][2], i);
        else if (i < order_npad(c.n))
            dst[i] = padding_point();
    }
}

__global__ __launch_bounds__(OC_THREADS) void k_order_deal(OrderParams p) {
    order_deal_body(p, grid_blk_xcd());
}

// x = super-block, y = frame, z = cloud
__device__ __forceinline__ void order_box_body(const OrderParams &pr, const Blk &blk) {
    static_assert(OC_THREADS == 4 * OSUPER, "four lanes per block");
    const OrderCloud c = blk.z ? pr.c[1] : pr.c[0];
    const int t = blk.y, supers = order_supers(c.n);
    if (blk.x >= supers) return;
    float *box = c.box + (size_t)t * supers * OBOX;
    block_box(c.pts + (size_t)t * order_npad(c.n), blk.x * OSUPER + (int)(threadIdx.x >> 2),
              order_blocks(c.n), threadIdx.x, box);
    __syncthreads();
    if (threadIdx.x < 64)
        super_box(box, blk.x, threadIdx.x, c.sbox + (size_t)t * ((supers + 63) / 64) * 6 * 64);
}

__global__ __launch_bounds__(OC_THREADS) void k_order_box(OrderParams p) {
    order_box_body(p, grid_blk_xcd());
}

// The search of both directions: side 0 finds the neighbours of cloud 0's points in cloud 1, side 1
// the other way round (`waves` stops after side 0 when only that is wanted).
struct NearCloud {
    const nfloat4 *pts;
    const float *box;
    const float *sbox;
    const float *src;  // the points in their own order
    int32_t *idx;      // results of this cloud's points as queries
    float *dist;
    int n, pad;
};

struct NearParams {
    NearCloud c[2];
    unsigned long long *stats;  // search counters, or NULL
    int wgs0;                   // workgroups of side 0 (side 1's follow)
    short both, share[2], few;  // whether side 1 runs; log2 of the waves that share a query wave; near_blk
};

// One wave per workgroup, so that a long wave keeps no finished ones' registers (100 frames: 1.22 ms
// against 1.27 ms with four), and registers for six waves on a SIMD.
constexpr int NEAR_THREADS = 64;
constexpr int NEAR_WAVES = 6;
// Where that would leave the chip idle, workgroups of sixteen waves of which 1, 4 or 16 share their 64
// queries: each takes every fourth or sixteenth block, and they prune by the best distances of all, kept
// in LDS.  A side shares sixteen ways up to NEAR_SHARE16 query waves (with 110 and 256 of them in the
// call: 33.5 -> 13.1 and 40 -> 17.8 us, before the blocks of unshared waves were screened) and four ways
// up to as many among few targets, which make short searches, and up to NEAR_SHARE4 among more.
// Shared against not, ordering included: 550 waves on a side, 3,500 targets 44.2 and 36.3 us; 640 waves,
// 8,192 targets 57.4 and 49.5 us; 1,024 waves, 65,536 targets 93 and 101 us; 1,100 waves, 3,500 targets
// 52.6 and 40.7 us; 2,048 waves, 65,536 targets 130 and 114 us.
constexpr long NEAR_SHARE16 = 512, NEAR_SHARE4 = 1024;
constexpr int NEAR_FEW_TARGETS = 16384;
constexpr int NEAR_SHARED_THREADS = 1024;
constexpr int NEAR_FEW_FRAMES = 64;

// a box held by the lanes (lane b: block b), and one lane's box in scalar registers
struct Box {
    float l[3], h[3];
};

__device__ __forceinline__ Box lane_box(const float *b, int lane) {
    Box r;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r.l[k] = b[k * 64 + lane];
        r.h[k] = b[(3 + k) * 64 + lane];
    }
    return r;
}

__device__ __forceinline__ Box box_of_lane(const Box &b, int l) {
    Box r;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        r.l[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b.l[k]), l));
        r.h[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b.h[k]), l));
    }
    return r;
}

// whether all points of the box are the same, finite one (a box without points is inverted): then the
// distance to the box is the canonical distance to each of them, bit for bit
__device__ __forceinline__ bool one_point(const Box &b) {
    bool r = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) r = r && b.l[k] == b.h[k] && fabsf(b.l[k]) < __builtin_inff();
    return r;
}

// the least original index of the lane's block
__device__ __forceinline__ int lane_least(const float *b, int lane) {
    return __float_as_int(b[6 * 64 + lane]);
}

// fmaxf drops a NaN gap (a box at infinity): the distance only gets smaller
__device__ __forceinline__ float box_box(const Box &a, const Box &b) {
    float g[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) g[k] = fmaxf(fmaxf(a.l[k] - b.h[k], b.l[k] - a.h[k]), 0.f);
    return canon_gap(g[0], g[1], g[2]);
}

__device__ __forceinline__ float point_box(float x, float y, float z, const Box &b) {
    const float g0 = fmaxf(fmaxf(b.l[0] - x, x - b.h[0]), 0.f);
    const float g1 = fmaxf(fmaxf(b.l[1] - y, y - b.h[1]), 0.f);
    const float g2 = fmaxf(fmaxf(b.l[2] - z, z - b.h[2]), 0.f);
    return canon_gap(g0, g1, g2);
}

// squared distance of the boxes' doubled centres
__device__ __forceinline__ float centre_dist(const Box &a, const Box &b) {
    const float dx = (a.l[0] + a.h[0]) - (b.l[0] + b.h[0]);
    const float dy = (a.l[1] + a.h[1]) - (b.l[1] + b.h[1]);
    const float dz = (a.l[2] + a.h[2]) - (b.l[2] + b.h[2]);
    return canon_gap(dx, dy, dz);
}

// the first lane that holds the smallest v (lane 0 when all are NaN)
__device__ __forceinline__ int arg_min_lane(float v) {
    const float m = wave_min(v);
    const unsigned long long b = __ballot(v == m);
    return b ? (int)__builtin_ctzll(b) : 0;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned bf16_pair(float lo, float hi) {
    bf16x2 v;
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(unsigned, v);
}

__device__ __forceinline__ float pair_lo(unsigned v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float pair_hi(unsigned v) { return __uint_as_float(v & 0xffff0000u); }

// the low halves, or the high halves, of two pairs
__device__ __forceinline__ unsigned lows(unsigned a, unsigned b) {
    return __builtin_amdgcn_perm(b, a, 0x05040100u);
}
__device__ __forceinline__ unsigned highs(unsigned a, unsigned b) {
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

constexpr unsigned BF16_1 = 0x3f80u, BF16_11 = 0x3f803f80u;

// The screen of a block: its 32 points against the wave's 64 queries in two matrix instructions.  With
// p' and q' the coordinates less the centre of the queries' box, |p'|^2 - 2 q'.p' + |q'|^2 is a sum of
// 16 products of bf16 numbers, each coordinate in two parts (their smallest products dropped) and each
// square in three: lanes 0..31 hold the first eight factors of a row or column, lanes 32..63 the rest.
//   points   xh yh zh  xl yl zl  sh sm | xh yh zh  sl  1  1  1  0      (s = |p'|^2)
//   queries  xh yh zh  xh yh zh   1  1 | xl yl zl   1 uh um ul  0      (of -2 q'; u = |q'|^2 + slack)
__device__ __forceinline__ bf16x8 screen_point(float x, float y, float z, bool upper) {
    const float s = canon_gap(x, y, z);
    const unsigned xy = bf16_pair(x, y), zs = bf16_pair(z, s);
    const unsigned xs = bf16_pair(x - pair_lo(xy), s - pair_hi(zs));
    const unsigned yz = bf16_pair(y - pair_hi(xy), z - pair_lo(zs));
    const unsigned sl = bf16_pair(s - pair_hi(zs) - pair_hi(xs), 0.f);
    u32x4 r;
    r[0] = xy;
    r[1] = lows(zs, upper ? sl : xs);
    r[2] = upper ? BF16_11 : yz;
    r[3] = upper ? BF16_1 : highs(zs, xs);
    return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ bf16x8 screen_query(float x, float y, float z, float u, bool upper) {
    x = -2.f * x;
    y = -2.f * y;
    z = -2.f * z;
    const unsigned xy = bf16_pair(x, y), zu = bf16_pair(z, u);
    const float ur = u - pair_hi(zu);
    const unsigned xyl = bf16_pair(x - pair_lo(xy), y - pair_hi(xy));
    const unsigned zul = bf16_pair(z - pair_lo(zu), ur);
    u32x4 r;
    r[0] = upper ? xyl : xy;
    r[1] = upper ? lows(zul, BF16_1) : lows(zu, xy);
    r[2] = upper ? highs(zu, zul) : (xy >> 16 | zu << 16);
    r[3] = upper ? bf16_pair(ur - pair_hi(zul), 0.f) : BF16_11;
    return __builtin_bit_cast(bf16x8, r);
}

// Error of the screen.  The parts leave out at most 2^-18 of each factor and the products of 2^-18:
// 6 2^-18 |q'| |p'| together, and the sum of the products rounds by no more than 2^-18 (|p'|^2 + |q'|^2):
// the products are exact in fp32, and 15 fp32 additions of them in any order, even if each only cut off, are
// off by at most 30 2^-24 of the sum of their magnitudes, which is at most 2.02 (|p'|^2 + |q'|^2).  How the
// instruction adds is not documented; the most it was off by, measured against 64 bits over 25 million results
// (factors of one size, over 2^+-10 and over 2^+-30, and this screen's own at scales of 1e-12, 1 and 1e12, of
// points far apart to nearly alike), was 5.6 2^-24 of that sum.
// With |p'| <= |q'| + d and |p'|^2 <= 2 |q'|^2 + 2 d^2 that is within 2^-18 (9 |q'|^2 + 6 |q'| d + 2 d^2),
// and, a third more for the roundings of p', q' and of the canonical distance d^2 itself, within
//   E(d) = 2^-18 (12 |q'|^2 + 8 |q'| d + 3 d^2) <= NEAR_ERR (3 |q'|^2 + 2 d^2),  NEAR_ERR = 2^-15.
// The slack in u is 3 NEAR_ERR |q'|^2 (and 1e-36 for what is below the normal range).  So a screened
// value v is never negative, d^2 is at most NEAR_UP v, and a point at the smallest distance d has
// v <= d^2 + slack + E(d).
constexpr float NEAR_ERR = 0x1p-15f, NEAR_UP = 1.f + 0x1p-13f;
constexpr float NEAR_SAFE = 1e30f;  // |q'|^2 and v up to which nothing overflows
// The slack is small against the differences between a query's nearest points where the queries' box is
// about as wide as a block of the targets.  On a jump of the curve it is wider, and more than two
// sub-tiles remain for many of the wave's queries: then the blocks in reach are evaluated once more for
// all of them, or the queries searched one by one where those are few.  Both are a wait for one wave
// that shows where few frames run beside it: a query takes about 4 us, a sweep of the blocks as long as
// the tests of their boxes, so the line lies at NEAR_FEW and one query more per 256 blocks.  Two frames
// of 131,072 points take 181 us with it, 268 us with three queries at any size; one frame of 262,144
// points 264 and 302 us (ordering included, both directions).  It ends at NEAR_FEW_MOST more: the waves of
// larger clouds fill the chip, and past half of the queries the sweep is the less work (one frame of
// 1,048,576 points in 27 clumps 3.65 -> 2.45 ms; 524,288 targets on a sphere about the queries, whose blocks
// are all in reach of each, 738 -> 73 ms; of 4,194,304 and 16,777,216 points in one sheet no change).
constexpr int NEAR_FEW = 3, NEAR_FEW_MOST = 32;

// Adds n to a counter: 0 queries, 1 sub-tiles read again, 2 queries searched again.
__device__ __forceinline__ void near_count(const NearParams &pr, int lane, int which, unsigned long long n) {
    if (pr.stats && lane == 0 && n)
        atomicAdd(pr.stats + (size_t)((blockIdx.x + gridDim.x * blockIdx.y) % STATS_SLOTS) * STATS_SLOT_WORDS +
                      which,
                  n);
}

// The end of a search: the queries without a finite distance, and the results.  The first wave counts the
// call's queries, and one sub-tile read again for each.
__device__ __forceinline__ void near_finish(const NearParams &pr, const Blk &blk, const NearCloud &qc,
                                            const NearCloud &pc, int lane, bool writes, bool first,
                                            const nfloat4 &q, float best, int found, bool finite) {
    const int t = blk.y, qi = __float_as_int(q.w);
    const float inf = __builtin_inff();
    // no finite distance: the first of the first 64 targets at an infinite distance, or target 0
    unsigned long long none = writes ? __ballot(qi >= 0 && !finite) : 0ull;
    while (none) {
        const int l = (int)__builtin_ctzll(none);
        none &= none - 1;
        const float x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.x), l));
        const float y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.y), l));
        const float z = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.z), l));
        bool hit = false;
        if (lane < pc.n) {
            const float *p = pc.src + ((size_t)t * pc.n + lane) * 3;
            hit = canon_gap(x - p[0], y - p[1], z - p[2]) == inf;
        }
        const unsigned long long m = __ballot(hit);
        if (lane == l) {
            found = m ? (int)__builtin_ctzll(m) : 0;
            best = inf;
        }
    }
    if (qi >= 0 && writes) {
        const size_t o = (size_t)t * qc.n + qi;
        qc.idx[o] = found;
        qc.dist[o] = best;
    }
    if (first) {
        const unsigned long long all =
            (unsigned long long)blk.gy * (pr.c[0].n + (pr.both ? pr.c[1].n : 0));
        near_count(pr, lane, 0, all);
        near_count(pr, lane, 1, all);
    }
}

// The search of query waves that several waves share.
__device__ __forceinline__ void near_shared_body(const NearParams &pr, const Blk &blk) {
    constexpr int WAVES = NEAR_SHARED_THREADS / 64;
    const int t = blk.y;
    const int lane = threadIdx.x & 63;
    const bool second = blk.x >= pr.wgs0;
    const NearCloud &qc = pr.c[second ? 1 : 0], &pc = pr.c[second ? 0 : 1];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // `group` of the workgroup's query waves, and this wave's place `r` among those that share it
    const int logw = pr.share[second ? 1 : 0];
    const int group = wave >> logw, r = wave & ((1 << logw) - 1);
    const int qw = (blk.x - (second ? pr.wgs0 : 0)) * (WAVES >> logw) + group;
    const bool run = qw * 64 < qc.n;
    __shared__ unsigned sbest[WAVES][64];
    __shared__ int sidx[WAVES][64];
    __shared__ int stie[WAVES][64];
    const float inf = __builtin_inff();
    if (r == 0) {
        sbest[group][lane] = __float_as_uint(inf);
        sidx[group][lane] = 0x7fffffff;
        stie[group][lane] = 0;
    }
    __syncthreads();
    // the wave's share of a super-block's blocks
    unsigned long long share = ~0ull;
    if (logw == 2) share = 0x1111111111111111ull << r;
    if (logw == 4) share = 0x0001000100010001ull << r;
    const int supers_q = order_supers(qc.n), supers = order_supers(pc.n);
    const int chunks = (supers + 63) / 64;
    const int nblk = order_blocks(pc.n);
    const nfloat4 *P = pc.pts + (size_t)t * order_npad(pc.n);
    const float *pbox = pc.box + (size_t)t * supers * OBOX;
    const float *psbox = pc.sbox + (size_t)t * chunks * 6 * 64;
    nfloat4 q = padding_point();
    if (run) q = qc.pts[(size_t)t * order_npad(qc.n) + qw * 64 + lane];
    const int qi = __float_as_int(q.w);
    // a NaN query has no distances; padding has no query
    const bool live = q.x == q.x && q.y == q.y && q.z == q.z && qi >= 0;
    float best = live ? inf : -1.f;
    int sub = -1;
    bool tie = false;
    Box Q;
    {  // the queries' box: two blocks of their own cloud
        const int b = run ? qw * 2 : 0;
        scalar_f o = (scalar_f)(uintptr_t)(qc.box + ((size_t)t * supers_q + b / OSUPER) * OBOX +
                                           b % OSUPER);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            Q.l[k] = fminf(o[k * OSUPER], o[k * OSUPER + 1]);
            Q.h[k] = fmaxf(o[(3 + k) * OSUPER], o[(3 + k) * OSUPER + 1]);
        }
    }
    auto take = [&](float m, int at) {
        tie = m < best ? false : (tie || m == best);
        sub = m < best ? at : sub;
        best = fminf(best, m);
    };
    // what a lane's candidates have to come up to: its best, or that of the waves it shares with
    float bound = best;
    auto share_best = [&]() {
        if (live) {
            atomicMin(&sbest[group][lane], __float_as_uint(best));
            bound = fminf(best, __uint_as_float(sbest[group][lane]));
        }
    };
    auto evaluate = [&](int b) {
        // the block's points in scalar registers, OLOAD at a time
        scalar_f4 p = (scalar_f4)(uintptr_t)(P + (size_t)b * OB);
#pragma unroll
        for (int h = 0; h < OB / OSUB; ++h) {
            float m = inf;
#pragma unroll
            for (int g = 0; g < OSUB; g += OLOAD) {
                nfloat4 v[OLOAD];
#pragma unroll
                for (int j = 0; j < OLOAD; ++j) v[j] = p[h * OSUB + g + j];
                __builtin_amdgcn_sched_barrier(0);  // a group's loads go out together
#pragma unroll
                for (int j = 0; j < OLOAD; ++j)
                    m = fminf(m, canon_gap(q.x - v[j].x, q.y - v[j].y, q.z - v[j].z));
                __builtin_amdgcn_sched_barrier(0);
            }
            take(m, b * (OB / OSUB) + h);
        }
    };
    if (__ballot(live)) {
        // the block nearest to the queries by its centre gives the first distances
        int seed_super;
        {
            float dmin = inf;
            int at = 0;
            for (int c = 0; c < chunks; ++c) {
                const int g = c * 64 + lane;
                const float v = centre_dist(Q, lane_box(psbox + (size_t)c * 6 * 64, lane));
                if (g < supers && v < dmin) {
                    dmin = v;
                    at = g;
                }
            }
            seed_super = __builtin_amdgcn_readlane(at, arg_min_lane(dmin));
        }
        int seed = -1;
        float near = -1.f;
        {
            const Box bx = lane_box(pbox + (size_t)seed_super * OBOX, lane);
            const bool mine = seed_super * OSUPER + lane < nblk && (share >> lane & 1);
            const float v = mine ? centre_dist(Q, bx) : inf;
            // (by their bits: the compiler takes `v < inf` for `v != inf`, which holds for a NaN)
            if (__ballot(__float_as_uint(v) < 0x7F800000u)) {
                const int k = arg_min_lane(v);
                seed = seed_super * OSUPER + k;
                near = box_box(Q, box_of_lane(bx, k));
                evaluate(seed);
                share_best();
            }
        }
        // first the blocks as near to the queries' box as the seed, which mostly hold the
        // neighbours, then the others within the distances found
        for (int pass = 0; pass < 2; ++pass) {
            for (int c = 0; c < chunks; ++c) {
                const int g = c * 64 + lane;
                const Box sb = lane_box(psbox + (size_t)c * 6 * 64, lane);
                float far = wave_max(bound);
                if (pass == 0) far = fminf(far, near);
                unsigned long long todo = __ballot(g < supers && !(box_box(Q, sb) > far));
                // the next super-block's boxes are on their way while this one's are worked on
                int s = todo ? c * 64 + (int)__builtin_ctzll(todo) : -1;
                Box ahead = sb;
                if (s >= 0) ahead = lane_box(pbox + (size_t)s * OBOX, lane);
                while (s >= 0) {
                    const Box bx = ahead;
                    const int s_at = s, b0 = s * OSUPER;
                    todo &= todo - 1;
                    s = todo ? c * 64 + (int)__builtin_ctzll(todo) : -1;
                    if (s >= 0) ahead = lane_box(pbox + (size_t)s * OBOX, lane);
                    const float l = box_box(Q, bx);
                    share_best();
                    far = wave_max(bound);
                    if (pass == 0) far = fminf(far, near);
                    unsigned long long in =
                        __ballot(b0 + lane < nblk && b0 + lane != seed && !(l > far) &&
                                 (pass == 0 || l > near)) & share;
                    // a block of one point repeated needs no more than its box and least index
                    const unsigned long long one = __ballot(one_point(bx)) & in;
                    int least = 0;
                    if (one) least = lane_least(pbox + (size_t)s_at * OBOX, lane);
                    while (in) {
                        const int k = (int)__builtin_ctzll(in);
                        in &= in - 1;
                        const float e = point_box(q.x, q.y, q.z, box_of_lane(bx, k));
                        if (!__ballot(!(e > bound))) continue;
                        if (one >> k & 1)
                            take(e, ~__builtin_amdgcn_readlane(least, k));
                        else
                            evaluate(b0 + k);
                        share_best();
                    }
                }
            }
        }
    }
    share_best();
    __syncthreads();
    bound = live ? __uint_as_float(sbest[group][lane]) : -1.f;
    // the winning sub-tile again, for the smallest original index at the minimum
    bool finite = live && best < inf && best == bound;
    int found = sub < 0 ? ~sub : 0x7fffffff;
    if (finite && sub >= 0) {
        const nfloat4 *p = P + (size_t)sub * OSUB;
#pragma unroll 1
        for (int j0 = 0; j0 < OSUB; j0 += 8) {
            nfloat4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = p[j0 + j];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float e = canon_gap(q.x - v[j].x, q.y - v[j].y, q.z - v[j].z);
                if (e == best) found = min(found, __float_as_int(v[j].w));
            }
        }
    }
    // a minimum met in more than one sub-tile: every point at exactly that distance
    unsigned long long again = __ballot(finite && tie);
    const bool same = one_point(Q);  // as in near_body
    if (same) again &= ~again + 1;
    while (again) {
        const int l = (int)__builtin_ctzll(again);
        again &= again - 1;
        const float x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.x), l));
        const float y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.y), l));
        const float z = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.z), l));
        const float bl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(best), l));
        int mine = 0x7fffffff;
        for (int c = 0; c < chunks; ++c) {
            const int g = c * 64 + lane;
            const float lb = point_box(x, y, z, lane_box(psbox + (size_t)c * 6 * 64, lane));
            unsigned long long todo = __ballot(g < supers && !(lb > bl));
            while (todo) {
                const int s = c * 64 + (int)__builtin_ctzll(todo);
                todo &= todo - 1;
                const Box bx = lane_box(pbox + (size_t)s * OBOX, lane);
                const bool near = s * OSUPER + lane < nblk && (share >> lane & 1) &&
                                  !(point_box(x, y, z, bx) > bl);
                const bool one = near && one_point(bx);
                if (one) mine = min(mine, lane_least(pbox + (size_t)s * OBOX, lane));
                unsigned long long in = __ballot(near && !one);
                while (in) {
                    const int b = s * OSUPER + (int)__builtin_ctzll(in);
                    in &= in - 1;
                    const nfloat4 v = P[(size_t)b * OB + (lane & (OB - 1))];
                    if (canon_gap(x - v.x, y - v.y, z - v.z) == bl)
                        mine = min(mine, __float_as_int(v.w));
                }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mine = min(mine, __shfl_xor(mine, off, 64));
        if (lane == l || (same && finite && tie)) found = mine;
    }
    // (also met by another wave: a tie between the waves)
    if (finite && (atomicMin(&sidx[group][lane], found) != 0x7fffffff || tie))
        stie[group][lane] = 1;
    __syncthreads();
    if (r == 0) {  // queries whose minimum was met more than once
        const int ties = __popcll(__ballot(stie[group][lane]));
        near_count(pr, lane, 1, ties);
        near_count(pr, lane, 2, ties);
    }
    found = sidx[group][lane];
    best = bound;
    finite = live && bound < inf;
    near_finish(pr, blk, qc, pc, lane, r == 0, blk.x == 0 && t == 0 && wave == 0, q, best, found,
                finite);
}

// The search of waves that have their queries to themselves, blocks screened on the matrix cores.
__device__ __forceinline__ void near_body(const NearParams &pr, const Blk &blk) {
    const int t = blk.y;
    const int lane = threadIdx.x;
    const bool second = blk.x >= pr.wgs0;
    const NearCloud &qc = pr.c[second ? 1 : 0], &pc = pr.c[second ? 0 : 1];
    const int qw = blk.x - (second ? pr.wgs0 : 0);
    const float inf = __builtin_inff();
    const int supers_q = order_supers(qc.n), supers = order_supers(pc.n);
    const int chunks = (supers + 63) / 64;
    const int nblk = order_blocks(pc.n);
    const nfloat4 *P = pc.pts + (size_t)t * order_npad(pc.n);
    const float *pbox = pc.box + (size_t)t * supers * OBOX;
    const float *psbox = pc.sbox + (size_t)t * chunks * 6 * 64;
    const nfloat4 q = qc.pts[(size_t)t * order_npad(qc.n) + qw * 64 + lane];
    // a NaN query has no distances; padding has no query
    const bool live = q.x == q.x && q.y == q.y && q.z == q.z && __float_as_int(q.w) >= 0;
    Box Q;
    {  // the queries' box: two blocks of their own cloud
        const int b = qw * 2;
        scalar_f o = (scalar_f)(uintptr_t)(qc.box + ((size_t)t * supers_q + b / OSUPER) * OBOX +
                                           b % OSUPER);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            Q.l[k] = fminf(o[k * OSUPER], o[k * OSUPER + 1]);
            Q.h[k] = fmaxf(o[(3 + k) * OSUPER], o[(3 + k) * OSUPER + 1]);
        }
    }
    // the queries about the centre of their box, and the slack of their screened values
    const float cx = 0.5f * Q.l[0] + 0.5f * Q.h[0],
                cy = 0.5f * Q.l[1] + 0.5f * Q.h[1],
                cz = 0.5f * Q.l[2] + 0.5f * Q.h[2];
    const bool upper = lane >= 32;
    bf16x8 B[2];
    float slack, widest;
    {
        const float x = live ? q.x - cx : 0.f, y = live ? q.y - cy : 0.f, z = live ? q.z - cz : 0.f;
        const float u = canon_gap(x, y, z);
        slack = __builtin_fmaf(u, 3.f * NEAR_ERR, 1e-36f);
        widest = wave_max(u);  // (without the NaN ones)
        if (__ballot(!(u < NEAR_SAFE))) widest = inf;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int from = k * 32 + (lane & 31);
            B[k] = screen_query(__shfl(x, from, 64), __shfl(y, from, 64), __shfl(z, from, 64),
                                __shfl(u + slack, from, 64), upper);
        }
    }
    // the least screened values of sub-tiles (their bits), and where the first two were met: a sub-tile,
    // or ~index of the least point of a block that is one point
    constexpr unsigned INF = 0x7F800000u;
    unsigned m1 = INF, m2 = INF, m3 = INF;
    int at1 = 0, at2 = 0;
    auto take = [&](unsigned v, int at) {
        const bool c1 = v < m1, c2 = v < m2;
        m3 = min(m3, max(m2, v));
        m2 = min(m2, max(m1, v));
        m1 = min(m1, v);
        at2 = c1 ? at1 : (c2 ? at : at2);
        at1 = c1 ? at : at1;
    };
    // Row m of the instruction is the point 16 h + 4 g + j of the block, m = 8 g + 4 h + j: then lanes
    // 0..31 get the first sub-tile's values and lanes 32..63 the second's, of 32 queries at a time.
    const int row = (lane & 4) * 4 + (lane >> 3 & 3) * 4 + (lane & 3);
    float bound = live ? inf : -1.f;
    auto screen = [&](int b) {
        const nfloat4 p = P[(size_t)b * OB + row];
        const bf16x8 A = screen_point(p.x - cx, p.y - cy, p.z - cz, upper);
        unsigned m[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const f32x16 zero = {0.f};
            const f32x16 d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, B[k], zero, 0, 0, 0);
            unsigned n[4];
#pragma unroll
            for (int g = 0; g < 4; ++g)
                n[g] = min(min(__float_as_uint(d[4 * g]), __float_as_uint(d[4 * g + 1])),
                           min(__float_as_uint(d[4 * g + 2]), __float_as_uint(d[4 * g + 3])));
            m[k] = min(min(n[0], n[1]), min(n[2], n[3]));
        }
        const auto sw = __builtin_amdgcn_permlane32_swap(m[0], m[1], false, false);
        take(sw[0], 2 * b);
        take(sw[1], 2 * b + 1);
    };
    // The canonical distances, and the smallest original index at the smallest.
    float best = inf;
    int found = 0x7fffffff;
    auto meet = [&](float e, int i) {
        found = e < best ? i : (e == best ? min(found, i) : found);
        best = fminf(best, e);
    };
    auto refine = [&](int at) {
        if (at < 0) {
            const float *p = pc.src + ((size_t)t * pc.n + ~at) * 3;
            meet(canon_gap(q.x - p[0], q.y - p[1], q.z - p[2]), ~at);
            return;
        }
        const nfloat4 *p = P + (size_t)at * OSUB;
        float e = inf;
        int i = 0x7fffffff;
#pragma unroll 1
        for (int j0 = 0; j0 < OSUB; j0 += 8) {
            nfloat4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = p[j0 + j];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float d = canon_gap(q.x - v[j].x, q.y - v[j].y, q.z - v[j].z);
                const int k = __float_as_int(v[j].w);
                i = d < e ? k : (d == e ? min(i, k) : i);
                e = fminf(e, d);
            }
        }
        meet(e, i);
    };
    bool screened = false;
    unsigned long long again = 0;
    // The live queries are one point repeated: of those to be searched again one is searched for all.  Where
    // targets are repeated too (a frame padded with one point) all of them are: one frame of 262,144 such
    // points 16.6 -> 4.8 ms, 40 frames of 8,192 698 -> 233 us, one of 2,048, whose query waves are shared,
    // 79 -> 33 us.
    const bool same = one_point(Q);
    if (__ballot(live)) {
        // the block nearest to the queries by its centre gives the first distances
        int seed_super;
        {
            float dmin = inf;
            int at = 0;
            for (int c = 0; c < chunks; ++c) {
                const int g = c * 64 + lane;
                const float v = centre_dist(Q, lane_box(psbox + (size_t)c * 6 * 64, lane));
                if (g < supers && v < dmin) {
                    dmin = v;
                    at = g;
                }
            }
            seed_super = __builtin_amdgcn_readlane(at, arg_min_lane(dmin));
        }
        int seed = -1;
        float near = -1.f;
        {
            const Box bx = lane_box(pbox + (size_t)seed_super * OBOX, lane);
            const float v = seed_super * OSUPER + lane < nblk ? centre_dist(Q, bx) : inf;
            // (by their bits: the compiler takes `v < inf` for `v != inf`, which holds for a NaN)
            if (__ballot(__float_as_uint(v) < 0x7F800000u)) {
                const int k = arg_min_lane(v);
                seed = seed_super * OSUPER + k;
                near = box_box(Q, box_of_lane(bx, k));
                screened = widest < NEAR_SAFE;
                if (screened) screen(seed);
            }
        }
        // screened values up to this one may be of a point at the canonical distance d or less
        auto limit = [&](float d) {
            const float qq = slack * (1.f / (3.f * NEAR_ERR));
            const float e = 12.f * qq + 8.f * __builtin_sqrtf(qq * d) + 3.f * d;
            return __builtin_fmaf(e, 0x1p-18f, d + slack);
        };
        if (screened) {
            bound = live ? NEAR_UP * __uint_as_float(m1) : -1.f;
            // first the blocks as near to the queries' box as the seed, which mostly hold the
            // neighbours, then the others within the distances found
            for (int pass = 0; pass < 2; ++pass) {
                for (int c = 0; c < chunks; ++c) {
                    const int g = c * 64 + lane;
                    const Box sb = lane_box(psbox + (size_t)c * 6 * 64, lane);
                    float far = wave_max(bound);
                    if (pass == 0) far = fminf(far, near);
                    unsigned long long todo = __ballot(g < supers && !(box_box(Q, sb) > far));
                    // the next super-block's boxes are on their way while this one's are worked on
                    int s = todo ? c * 64 + (int)__builtin_ctzll(todo) : -1;
                    Box ahead = sb;
                    if (s >= 0) ahead = lane_box(pbox + (size_t)s * OBOX, lane);
                    while (s >= 0) {
                        const Box bx = ahead;
                        const int s_at = s, b0 = s * OSUPER;
                        todo &= todo - 1;
                        s = todo ? c * 64 + (int)__builtin_ctzll(todo) : -1;
                        if (s >= 0) ahead = lane_box(pbox + (size_t)s * OBOX, lane);
                        const float l = box_box(Q, bx);
                        far = wave_max(bound);
                        if (pass == 0) far = fminf(far, near);
                        unsigned long long in =
                            __ballot(b0 + lane < nblk && b0 + lane != seed && !(l > far) &&
                                     (pass == 0 || l > near));
                        // a block of one point repeated needs no more than its box and least index
                        const unsigned long long one = __ballot(one_point(bx)) & in;
                        int least = 0;
                        if (one) least = lane_least(pbox + (size_t)s_at * OBOX, lane);
                        while (in) {
                            const int k = (int)__builtin_ctzll(in);
                            in &= in - 1;
                            const float e = point_box(q.x, q.y, q.z, box_of_lane(bx, k));
                            if (!__ballot(!(e > bound))) continue;
                            if (one >> k & 1)
                                take(__float_as_uint(e), ~__builtin_amdgcn_readlane(least, k));
                            else
                                screen(b0 + k);
                            if (live) bound = NEAR_UP * __uint_as_float(m1);
                        }
                    }
                }
            }
            // the sub-tiles that may hold the smallest distance
            const bool known = live && __uint_as_float(m1) < NEAR_SAFE;
            bool two = false;
            if (known) {
                refine(at1);
                two = __uint_as_float(m2) <= limit(best);
                if (two) refine(at2);
            }
            near_count(pr, lane, 1, __popcll(__ballot(two)));
            again = __ballot(live && (!known || __uint_as_float(m3) <= limit(best)));
            near_count(pr, lane, 2, __popcll(again));
            if (same) again &= ~again + 1;
        }
        // More sub-tiles than that for some queries, or values that may have overflowed: every point
        // again whose box is no further than the best so far, for a few queries one by one with a
        // point per lane, for more of them for all at once.  That sweep settles ties as it meets them: on
        // clouds whose points are nearly all as far (targets on a sphere about the queries) most queries
        // meet their minimum more than once, and searched one by one for it one frame of 262,144 points
        // took 168 ms, settled here 25 ms (20 frames of 65,536: 43.6 and 20.7; the exhaustive fp32 search
        // 11.4 and 10.9).
        if (!screened || __popcll(again) > NEAR_FEW + min(nblk / 256, NEAR_FEW_MOST)) {
            // the block of the least screened value is known once its other half is, too: otherwise each
            // query would stop the sweep there
            int done = -1;
            if (screened && live && __uint_as_float(m1) < NEAR_SAFE && at1 >= 0) {
                refine(at1 ^ 1);
                done = at1 >> 1;
            }
            // of the last tested super-block hardly a block was ruled out by the queries' own distances:
            // then three of four super-blocks go untested (a quarter of the sweep's time)
            bool all = false;
            near_count(pr, lane, 2, __popcll(__ballot(live) & ~again));  // the others of the wave
            for (int c = 0; c < chunks; ++c) {
                const int g = c * 64 + lane;
                float far = wave_max(live ? best : -1.f);
                unsigned long long todo = __ballot(
                    g < supers && !(box_box(Q, lane_box(psbox + (size_t)c * 6 * 64, lane)) > far));
                while (todo) {
                    const int s = c * 64 + (int)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    const Box bx = lane_box(pbox + (size_t)s * OBOX, lane);
                    far = wave_max(live ? best : -1.f);
                    unsigned long long in =
                        __ballot(s * OSUPER + lane < nblk && !(box_box(Q, bx) > far));
                    const unsigned long long one = __ballot(one_point(bx)) & in;
                    int least = 0;
                    if (one) least = lane_least(pbox + (size_t)s * OBOX, lane);
                    auto evaluate = [&](int b) {
                        scalar_f4 p = (scalar_f4)(uintptr_t)(P + (size_t)b * OB);
                        float m = inf;
#pragma unroll 1
                        for (int h = 0; h < OB; h += OSUB)
#pragma unroll
                            for (int j0 = 0; j0 < OSUB; j0 += OLOAD) {
                                nfloat4 v[OLOAD];
#pragma unroll
                                for (int j = 0; j < OLOAD; ++j) v[j] = p[h + j0 + j];
                                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                                for (int j = 0; j < OLOAD; ++j)
                                    m = fminf(m, canon_gap(q.x - v[j].x, q.y - v[j].y,
                                                           q.z - v[j].z));
                                __builtin_amdgcn_sched_barrier(0);
                            }
                        // seldom, for lanes at or below their smallest distance: the least point there
                        if (!__ballot(live && !(m > best) && b != done)) return;
                        int i = 0x7fffffff;
#pragma unroll 8
                        for (int j = 0; j < OB; ++j) {
                            const nfloat4 v = p[j];
                            if (canon_gap(q.x - v.x, q.y - v.y, q.z - v.z) == m)
                                i = min(i, __float_as_int(v.w));
                        }
                        meet(m, i);
                    };
                    if (all && s % 4) {  // untested
                        for (unsigned long long now = in & ~one; now; now &= now - 1)
                            evaluate(s * OSUPER + (int)__builtin_ctzll(now));
                        in &= one;
                    }
                    const int tested = __popcll(in);
                    int kept = 0;
                    while (in) {
                        const int k = (int)__builtin_ctzll(in);
                        in &= in - 1;
                        const float e = point_box(q.x, q.y, q.z, box_of_lane(bx, k));
                        if (!__ballot(live && !(e > best))) continue;
                        ++kept;
                        if (one >> k & 1)
                            meet(e, __builtin_amdgcn_readlane(least, k));
                        else
                            evaluate(s * OSUPER + k);
                    }
                    if (s % 4 == 0 || !all) all = kept > tested - tested / 8;
                }
            }
            again = 0;
        }
    }
    while (again) {
        const int l = (int)__builtin_ctzll(again);
        again &= again - 1;
        const float x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.x), l));
        const float y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.y), l));
        const float z = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(q.z), l));
        float bl = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(best), l));
        float low = bl;
        int mine = 0x7fffffff;
        auto meet_one = [&](float e, int i) {
            mine = e < low ? i : (e == low ? min(mine, i) : mine);
            low = fminf(low, e);
        };
        for (int c = 0; c < chunks; ++c) {
            const int g = c * 64 + lane;
            const float lb = point_box(x, y, z, lane_box(psbox + (size_t)c * 6 * 64, lane));
            unsigned long long todo = __ballot(g < supers && !(lb > bl));
            while (todo) {
                const int s = c * 64 + (int)__builtin_ctzll(todo);
                todo &= todo - 1;
                const Box bx = lane_box(pbox + (size_t)s * OBOX, lane);
                const float e = point_box(x, y, z, bx);
                const bool near = s * OSUPER + lane < nblk && !(e > bl);
                const bool one = near && one_point(bx);
                if (one) meet_one(e, lane_least(pbox + (size_t)s * OBOX, lane));
                unsigned long long in = __ballot(near && !one);
                while (in) {
                    const int b = s * OSUPER + (int)__builtin_ctzll(in);
                    in &= in - 1;
                    const nfloat4 v = P[(size_t)b * OB + (lane & (OB - 1))];
                    if (lane < OB)
                        meet_one(canon_gap(x - v.x, y - v.y, z - v.z), __float_as_int(v.w));
                }
                bl = wave_min(low);
            }
        }
        if (low != bl) mine = 0x7fffffff;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mine = min(mine, __shfl_xor(mine, off, 64));
        if (lane == l || (same && live)) {
            found = mine;
            best = bl;
        }
    }
    const bool finite = live && best < inf;
    near_finish(pr, blk, qc, pc, lane, true, blk.x == 0 && t == 0, q, best, found, finite);
}

// For few frames, the grid with each XCD given a contiguous eighth of each side's workgroups: one side may
// take many times as long as the other, and would leave half of the chip idle (262,144 queries amid targets
// on a sphere about them 34 -> 25 ms, in the other's unit cube a tenth as large 2.9 -> 1.9; 20 frames of 65,536
// 24.8 -> 20.7 and 2.2 -> 1.8).  Of 100 frames each XCD has whole ones, and both sides of a frame at a time are
// the better order (100 frames of 65,536: 0.6% of the step).
__device__ __forceinline__ Blk near_blk(const NearParams &p) {
    const unsigned gx = gridDim.x, all = gx * gridDim.y, b = blockIdx.x + gx * blockIdx.y;
    const unsigned x0 = p.wgs0, n0 = x0 * gridDim.y;
    const unsigned xcd = b % NUM_XCD, k = b / NUM_XCD;
    auto before = [&](unsigned n) { return xcd * (n / NUM_XCD) + min(xcd, n % NUM_XCD); };
    const unsigned first0 = before(n0), own0 = n0 / NUM_XCD + (xcd < n0 % NUM_XCD ? 1u : 0u);
    Blk r = grid_blk();
    if (k < own0) {
        const unsigned l = first0 + k;
        r.y = (int)(l / x0);
        r.x = (int)(l % x0);
    } else {
        const unsigned l = before(all) - first0 + (k - own0);
        r.y = (int)(l / (gx - x0));
        r.x = (int)(x0 + l % (gx - x0));
    }
    return r;
}

__global__ __launch_bounds__(NEAR_THREADS, NEAR_WAVES) void k_near(NearParams p) {
    near_body(p, p.few ? near_blk(p) : grid_blk_xcd());
}

__global__ __launch_bounds__(NEAR_SHARED_THREADS, 8) void k_near_shared(NearParams p) {
    near_shared_body(p, grid_blk_xcd());
}

// about two points per cell
int order_bits(int n) {
    const int most = n <= ORD_SMALL ? ORD_SMALL_BITS : ORD_BITS;
    int b = 6;
    while (b < most && (1 << (b + 2)) <= n) ++b;
    return b;
}

// scratch of one cloud; with ar.base == NULL only its size (ar.off) is of interest
OrderCloud carve_cloud(Arena &ar, const float *src, int T, int n, bool small) {
    OrderCloud o;
    o.src = src;
    o.n = n;
    o.bits = order_bits(n);
    o.pts = ar.take<nfloat4>((size_t)T * order_npad(n));
    o.box = ar.take<float>((size_t)T * order_supers(n) * OBOX);
    o.sbox = ar.take<float>((size_t)T * ((order_supers(n) + 63) / 64) * 6 * 64);
    o.cnt = o.start = nullptr;
    o.rank = nullptr;
    o.part = o.parts = 0;
    if (!small) {
        // parts for the whole chip (two workgroups fit a compute unit) of 8,192 to ORD_PART points
        const int wanted = std::max(512 / (2 * T), 1);
        const int part = std::min(std::max((n + wanted - 1) / wanted, 8192), ORD_PART);
        o.part = (part + OC_POINTS - 1) / OC_POINTS * OC_POINTS;
        o.parts = (n + o.part - 1) / o.part;
        o.cnt = ar.take<unsigned>((size_t)T * o.parts << (o.bits - 1));
        o.start = ar.take<unsigned>(((size_t)T * o.parts << o.bits) +
                                    (size_t)T * (sizeof(OrderCells) / 4 + o.parts * OC_CHUNKS));
        o.rank = ar.take<unsigned short>((size_t)T * n);
    }
    return o;
}

// one workgroup per cloud, or all of the chip for each step
bool order_is_small(int Na, int Nb) { return std::max(Na, Nb) <= ORD_SMALL; }

}  // namespace

// Where this search is the fastest, measured over 1 to 4,096 frames of 16 to 65,536 points, 1,968 calls on
// clouds of a sheet (us, ordered / bf16 screen / every pair).  No call is slower than the search that its
// precision had without this one (noise aside); the least of the three is missed by 1.2% on average in one
// direction, by nothing in both (at most by 20%, 256 frames of 16 x 32: 27 / 91 / 32).
//
// Both directions: nearly everywhere (64 frames of 64 x 64: 24 / 82 / 28; 1,024 of 16 x 2,048: 151 / 297 /
// 647).  Every pair is faster for many rows that fill the chip against few targets, the line rising with the
// rows of a frame (256 frames of 2,048 x 128: 74 / 192 / 60, 64 of 8,192 x 256: 83 / 194 / 75, 16 of 65,536 x 384:
// 169 / 350 / 155), for 16 targets of many frames or of rows by the ten thousand, and for a handful of rows
// against targets by the ten thousand (16 frames of 64 x 65,536: 209 / 670 / 160).
//
// One direction (a to b): ordering both clouds for one search pays with targets by the hundred and rows enough
// for them (4 frames of 512 x 384: 24 / 69 / 26; 1,024 of 512 x 256: 78 / 178 / 61; one of 2,048 x 65,536: 83 / 470 /
// 72; 4 of them: 80 / 486 / 152), for fewer targets where rows fill the chip, and, on few frames, for 1,024
// to 4,096 targets, which the exhaustive search walks in a chain (one frame of 16 x 2,048: 30 / 47 / 55).
bool ordered_pays(int T, int Na, int Nb, bool two) {
    const long rows = (long)T * Na;
    if (two) {
        const int few = Na < 384    ? 16
                        : Na < 2048 ? 32
                                    : std::min(std::max(128, Na / 32),
                                               std::max(256, std::min(Na / 64, 512)));
        if (rows >= 1 << 18 && Nb <= few) return false;
        if ((T >= 256 && Nb <= 16) || Nb <= Na / 1024) return false;
        if (Nb >= 16384 && (Na <= Nb / 1024 || (T >= 4 && Nb >= 32768 && Na <= Nb / 340))) return false;
        return (long)Na * Nb > 512;
    }
    return (Nb >= (T < 256 ? 384 : 512) && Na >= 384 && (Nb / 16 <= Na || (rows >= 8192 && Nb / 48 <= Na))) ||
           (Nb >= 192 && Na >= 1024 && T >= 256) ||
           (Na >= 8192 && Nb >= (rows <= 1 << 19 ? 64 : 256)) ||
           (T <= 64 && Nb >= 1024 && Nb <= 4096);
}

size_t ordered_scratch_bytes(int T, int Na, int Nb) {
    Arena ar;
    carve_cloud(ar, nullptr, T, Na, order_is_small(Na, Nb));
    carve_cloud(ar, nullptr, T, Nb, order_is_small(Na, Nb));
    return ar.off;
}

void launch_ordered(const float *a, int Na, const float *b, int Nb, int T, int32_t *idx_a,
                    float *dist_a, int32_t *idx_b, float *dist_b, char *scratch,
                    unsigned long long *stats, dc_ctx *prof, hipStream_t s) {
    Arena ar;
    ar.base = scratch;
    ar.cap = ordered_scratch_bytes(T, Na, Nb);
    const bool small = order_is_small(Na, Nb);
    OrderParams op;
    op.c[0] = carve_cloud(ar, a, T, Na, small);
    op.c[1] = carve_cloud(ar, b, T, Nb, small);
    {
        ProfScope ps(prof, 1, s);
        if (small) {
            dispatch(KT_ORDER_SMALL, k_order_small, dim3(2, T), ORD_THREADS, op, s);
        } else {
            const int n = std::max(Na, Nb);
            const unsigned cells = 1u << std::max(op.c[0].bits, op.c[1].bits);
            const unsigned chunks = (unsigned)(order_npad(n) + OC_POINTS - 1) / OC_POINTS;
            dispatch(KT_ORDER_COUNT, k_order_count,
                     dim3(std::max(op.c[0].parts, op.c[1].parts), T, 2), ORD_THREADS, op, s);
            dispatch(KT_ORDER_SCAN, k_order_scan, dim3((cells + OC_CELLS - 1) / OC_CELLS, T, 2),
                     ORD_THREADS, op, s);
            dispatch(KT_ORDER_DEAL, k_order_deal, dim3(chunks, T, 2), OC_THREADS, op, s);
            dispatch(KT_ORDER_BOX, k_order_box, dim3(order_supers(n), T, 2), OC_THREADS, op,
                     s);
        }
    }
    NearParams np;
    for (int k = 0; k < 2; ++k) {
        const OrderCloud &o = op.c[k];
        NearCloud &c = np.c[k];
        c.pts = o.pts;
        c.box = o.box;
        c.sbox = o.sbox;
        c.src = o.src;
        c.idx = k ? idx_b : idx_a;
        c.dist = k ? dist_b : dist_a;
        c.n = o.n;
    }
    np.stats = stats;
    // waves that share a query wave: enough for the chip on each side
    long waves[2];
    bool shared = false;
    for (int k = 0; k < 2; ++k) {
        waves[k] = order_npad(op.c[k].n) / 64;
        const long all = waves[k] * T;
        const bool few = op.c[k ? 0 : 1].n <= NEAR_FEW_TARGETS;
        np.share[k] = all < NEAR_SHARE16 ? 4 : (all <= NEAR_SHARE4 && !few ? 2 : 0);
        shared |= np.share[k] > 0 && (k == 0 || idx_b);
    }
    np.both = idx_b != nullptr;
    np.few = T < NEAR_FEW_FRAMES;
    const int per = (shared ? NEAR_SHARED_THREADS : NEAR_THREADS) / 64;
    long wgs = 0;
    for (int k = 0; k < (idx_b ? 2 : 1); ++k) {
        const int groups = shared ? per >> np.share[k] : per;
        wgs += (waves[k] + groups - 1) / groups;
        if (k == 0) np.wgs0 = (int)wgs;
    }
    ProfScope ps(prof, 0, s);
    if (shared)
        dispatch(KT_NEAR_SHARED, k_near_shared, dim3((unsigned)wgs, T), NEAR_SHARED_THREADS, np, s);
    else
        dispatch(KT_NEAR, k_near, dim3((unsigned)wgs, T), NEAR_THREADS, np, s);
}

void register_ordered_kernels(BatchedKernel *table) {
    table[KT_ORDER_SMALL] = batched_kernel<OrderParams, order_small_body, ORD_THREADS, 512>();
    table[KT_ORDER_COUNT] = batched_kernel<OrderParams, order_count_body, ORD_THREADS, 512>();
    table[KT_ORDER_SCAN] = batched_kernel<OrderParams, order_scan_body, ORD_THREADS, 512>();
    table[KT_ORDER_DEAL] = batched_kernel<OrderParams, order_deal_body, OC_THREADS, 1024>();
    table[KT_ORDER_BOX] = batched_kernel<OrderParams, order_box_body, OC_THREADS, 1024>();
    // (one wave per SIMD less than the direct kernel, where it would spill: 41.5 -> 39.4 us for 38 frames)
    table[KT_NEAR] = batched_kernel<NearParams, near_body, NEAR_THREADS, 8192, NEAR_WAVES - 1>();
    table[KT_NEAR_SHARED] =
        batched_kernel<NearParams, near_shared_body, NEAR_SHARED_THREADS, 512, 8>();
}

}  // namespace dc

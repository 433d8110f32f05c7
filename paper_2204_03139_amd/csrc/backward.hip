// Backward passes: the Chamfer gradient through the saved neighbours (Sec. III-A, Eq. 1/2) and
// the sampling gradient through Eq. 4 (Sec. III-B).  Both are gathers over segments of equal keys
// (listed in LDS, or for very many items built by a stable sort), each put into increasing index
// order first and summed in an order fixed by that and by the sizes, in double (each output rounded
// once to float), so every result is bitwise reproducible, independent of scheduling, and within a
// few units of 2^-24 of the sum of its terms' magnitudes however long a segment is.
#include <algorithm>

#include "batch.h"

namespace dc {
namespace {

constexpr int BW_THREADS = 256;

// g_x[t,i] = g_t w_t ( cs * (x_i - y_{nn_x[i]}) + cm * sum_{j: nn_y[j]=i} (x_i - y_j) )
// for x = a (cs = 2 alpha, cm = 2 beta) or x = b (cs = 2 beta, cm = 2 alpha).
struct ChamferBwdParams {
    const double *grad_loss;
    const float *X;
    const float *Y;
    const int32_t *nn_x;
    const int32_t *ystart;        // [T][Nx + 1]: first sorted position of each neighbour in x
    const int32_t *yvals_sorted;
    const float *frame_w;
    float *gX;
    double cself, cmutual;
    int Nx, Ny;
};

__device__ __forceinline__ void chamfer_bwd_body(const ChamferBwdParams &pr, const Blk &blk) {
    const double *__restrict__ grad_loss = pr.grad_loss;
    const float *__restrict__ X = pr.X;
    const float *__restrict__ Y = pr.Y;
    const int32_t *__restrict__ nn_x = pr.nn_x;
    const int32_t *__restrict__ ystart = pr.ystart;
    const int32_t *__restrict__ yvals_sorted = pr.yvals_sorted;
    const int Nx = pr.Nx, Ny = pr.Ny;
    const double cself = pr.cself, cmutual = pr.cmutual;
    const float *__restrict__ frame_w = pr.frame_w;
    float *__restrict__ gX = pr.gX;
    const int t = blk.y;
    const int i = blk.x * BW_THREADS + threadIdx.x;
    if (i >= Nx) return;
    const double g = grad_loss[t] * (frame_w ? (double)frame_w[t] : 1.0);
    const double cs = cself * g;
    const double cm = cmutual * g;
    const float *xt = X + (size_t)t * Nx * 3;
    const float *yt = Y + (size_t)t * Ny * 3;
    // in double (each difference of two floats is exact there) and rounded once to float: the
    // result stays within a few units of 2^-24 of the sum of the terms' magnitudes however many
    // points share this neighbour
    const double x0 = xt[3 * (size_t)i], x1 = xt[3 * (size_t)i + 1], x2 = xt[3 * (size_t)i + 2];
    double g0 = 0.0, g1 = 0.0, g2 = 0.0;
    // the own-neighbour term exists only when cself != 0 (nn_x may be NULL otherwise: the b side of
    // the unidirectional loss has no neighbour indices), whatever the upstream gradient: 0 NaN is
    // not 0
    const int jn = (cself != 0.0 && cs != 0.0) ? nn_x[(size_t)t * Nx + i] : -1;
    if ((unsigned)jn < (unsigned)Ny) {  // indices outside [0, Ny) contribute nothing
        const int j = jn;
        g0 = cs * (x0 - (double)yt[3 * (size_t)j]);
        g1 = cs * (x1 - (double)yt[3 * (size_t)j + 1]);
        g2 = cs * (x2 - (double)yt[3 * (size_t)j + 2]);
    }
    if (cmutual != 0.0 && cm != 0.0) {  // (the segments are there only when cmutual != 0)
        const int32_t *vs = yvals_sorted + (size_t)t * Ny;
        const int32_t *st = ystart + (size_t)t * (Nx + 1);
        const int lo = st[i], hi = st[i + 1];
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
        for (int p = lo; p < hi; ++p) {
            const int j = vs[p];
            if (j < 0) continue;  // a neighbour index outside [0, Nx): contributes nothing
            s0 += x0 - (double)yt[3 * (size_t)j];
            s1 += x1 - (double)yt[3 * (size_t)j + 1];
            s2 += x2 - (double)yt[3 * (size_t)j + 2];
        }
        g0 += cm * s0;
        g1 += cm * s1;
        g2 += cm * s2;
    }
    float *o = gX + ((size_t)t * Nx + i) * 3;
    o[0] = (float)g0;
    o[1] = (float)g1;
    o[2] = (float)g2;
}

__global__ __launch_bounds__(BW_THREADS) void k_chamfer_bwd(ChamferBwdParams p) {
    chamfer_bwd_body(p, grid_blk_xcd());
}

// start[t][k] = first position of the sorted keys of frame t whose key is >= k, for k in [0, K]
// (the sort clamps its keys into [0, K]).  The thread of position q in [0, N] writes the entries
// of the keys in (key[q-1], key[q]] (key[-1] = -1, key[N] = K), so every entry is written exactly
// once, by adjacent differences instead of a binary search per key.
struct BoundsParams {
    const int32_t *sorted;
    int32_t *start;
    int N, K;
};

__device__ __forceinline__ void bounds_body(const BoundsParams &p, const Blk &blk) {
    const int t = blk.y;
    const int q = blk.x * BW_THREADS + threadIdx.x;
    if (q > p.N) return;
    const int32_t *s = p.sorted + (size_t)t * p.N;
    const int lo = q == 0 ? -1 : min(s[q - 1], p.K);
    const int hi = q == p.N ? p.K : min(s[q], p.K);
    int32_t *st = p.start + (size_t)t * (p.K + 1);
    for (int k = lo + 1; k <= hi; ++k) st[k] = q;
}

__global__ __launch_bounds__(BW_THREADS) void k_bounds(BoundsParams p) { bounds_body(p, grid_blk()); }

// per face and corner: fg[t,f,c] = sum over the points i of face f, in increasing i, of
// bary[t,i,c] * g[t,i]
struct FaceGradParams {
    const float *gpts;
    const float *bary;
    const int32_t *pts_by_face;
    const int32_t *face_start;
    float *fg;
    int F, N;
};

__device__ __forceinline__ void face_grad_body(const FaceGradParams &pr, const Blk &blk) {
    const float *__restrict__ gpts = pr.gpts;
    const float *__restrict__ bary = pr.bary;
    const int32_t *__restrict__ pts_by_face = pr.pts_by_face;
    const int32_t *__restrict__ face_start = pr.face_start;
    const int F = pr.F, N = pr.N;
    float *__restrict__ fg = pr.fg;
    const int t = blk.y;
    const int f = blk.x * BW_THREADS + threadIdx.x;
    if (f >= F) return;
    const int32_t *fs = face_start + (size_t)t * (F + 1);
    const int32_t *pf = pts_by_face + (size_t)t * N;
    const float *gt = gpts + (size_t)t * N * 3;
    const float *bt = bary + (size_t)t * N * 3;
    // in double (a product of two floats is exact there), rounded once to float per (face, corner)
    double acc[3][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
    for (int p = fs[f]; p < fs[f + 1]; ++p) {
        const int i = pf[p];
        const double g0 = gt[3 * (size_t)i], g1 = gt[3 * (size_t)i + 1], g2 = gt[3 * (size_t)i + 2];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double w = bt[3 * (size_t)i + c];
            acc[c][0] = __builtin_fma(w, g0, acc[c][0]);
            acc[c][1] = __builtin_fma(w, g1, acc[c][1]);
            acc[c][2] = __builtin_fma(w, g2, acc[c][2]);
        }
    }
    float *o = fg + ((size_t)t * F + f) * 9;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int d = 0; d < 3; ++d) o[3 * c + d] = (float)acc[c][d];
}

__global__ __launch_bounds__(BW_THREADS) void k_face_grad(FaceGradParams p) {
    face_grad_body(p, grid_blk_xcd());
}

// grad_verts[t,v] = sum over the incident (face f, corner c), in increasing (f, c), of fg[t,f,c]
struct VertexGradParams {
    const float *fg;
    const int32_t *corners_by_vertex;
    const int32_t *vert_start;
    float *gverts;
    int V, F;
};

__device__ __forceinline__ void vertex_grad_body(const VertexGradParams &pr, const Blk &blk) {
    const float *__restrict__ fg = pr.fg;
    const int32_t *__restrict__ corners_by_vertex = pr.corners_by_vertex;
    const int32_t *__restrict__ vert_start = pr.vert_start;
    const int V = pr.V, F = pr.F;
    float *__restrict__ gverts = pr.gverts;
    const int t = blk.y;
    const int v = blk.x * BW_THREADS + threadIdx.x;
    if (v >= V) return;
    const float *ft = fg + (size_t)t * F * 9;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;  // in double, rounded once to float
    for (int q = vert_start[v]; q < vert_start[v + 1]; ++q) {
        const int fc = corners_by_vertex[q];  // 3 f + c
        a0 += ft[3 * (size_t)fc];
        a1 += ft[3 * (size_t)fc + 1];
        a2 += ft[3 * (size_t)fc + 2];
    }
    float *o = gverts + ((size_t)t * V + v) * 3;
    o[0] = (float)a0;
    o[1] = (float)a1;
    o[2] = (float)a2;
}

__global__ __launch_bounds__(BW_THREADS) void k_vertex_grad(VertexGradParams p) {
    vertex_grad_body(p, grid_blk_xcd());
}

// ---------------------------------------------------------------- sums over small segments
// The same three sums without a sort in memory, for up to GP_MAX items: a workgroup takes a range of
// keys (rows, faces or vertices), reads all of the items' keys, lists the items of its own keys in
// LDS, puts each key's items into increasing order and sums over them.  Every workgroup reads all
// keys, but as a coalesced stream that its neighbours on the XCD read too; nothing is scattered
// through memory, and one launch takes the place of seven.  The items are listed by LDS atomics in
// whatever order, but counting, for each, the smaller items of its segment gives each its place:
// the sums run in the same order on every run.
//
// Workgroups of 512 threads, four to a compute unit, for up to GP_WIDE items a frame, else of 1,024,
// two to a compute unit: fewer workgroups then read the keys.  The kernels of a backward, 512 against
// 1,024 threads: 40 frames of 8,192 points 40 / 55 us (124 us with sorts), 17 frames of 30,011 x 5,003
// (both gradients) 69 / 79 (192), 24 frames of 32,768 x 20,011 78 / 92 (158), 100 frames of 65,536
// 533 / 445 (719).
constexpr int GP_SMALL = 512, GP_LARGE = 1024;
constexpr int GP_WIDE = 49152;
constexpr int GP_IBITS = 17;      // bits of an item in a listed word, below its key
constexpr int GP_MAX = 1 << GP_IBITS;
constexpr float GP_HEAVY = 12.f;
constexpr int GP_LONG = 16;       // most keys of a round that are listed thread by thread

// items listed at once, and most keys, of a workgroup of TH threads
template <int TH>
constexpr int gp_cap() { return 4 * TH; }
static_assert(gp_cap<GP_LARGE>() <= 1 << (32 - GP_IBITS), "a key and an item share a word");

template <int TH>
struct GroupLds {
    int start[gp_cap<TH>() + 4];  // first position of each key's items, over the workgroup's range
    union {
        struct {
            union {
                struct {
                    int cursor[gp_cap<TH>()];
                    unsigned listed[gp_cap<TH>()];
                };
                unsigned short own[GP_LONG][TH];  // of long keys: the threads' items, then their places
            };
            int item[gp_cap<TH>()];  // the items, by key and then in a fixed order
        };
        float row[3][gp_cap<TH>()];  // in their place, what the items stand for
    };
    int wsum[TH / 64];
    int heavy;  // the first heavy key of a round; before the rounds: whether there is one
    int some_long;  // whether there are keys of which a list holds no more than GP_LONG
    double part[TH / 64][9];
};

// Whether a key of `len` of n items is heavy: summed by the whole workgroup, where the comparisons of its items
// with each other, len^2 over all threads, would take longer than two more passes over the n keys.  More items
// than a list holds always are.
__device__ __forceinline__ bool heavy_key(int len, int n) {
    return (float)len * (float)len > GP_HEAVY * (float)n;
}
static_assert((float)gp_cap<GP_SMALL>() * gp_cap<GP_SMALL>() > GP_HEAVY * GP_MAX, "a list holds a light key");

// a sum of M components by the G lanes of a key's team (in every lane), in a fixed order
template <int M>
__device__ __forceinline__ void team_sum(double (&v)[M], int G) {
    for (int off = 1; off < G; off <<= 1)
#pragma unroll
        for (int k = 0; k < M; ++k) v[k] += __shfl_xor(v[k], off, 64);
}

// visit(i, keys[i]) for every i, by the workgroup: four keys a load (keys are 4-byte aligned, which
// is all a 16-byte load needs), four loads of a thread in flight
struct __attribute__((packed, aligned(4))) Keys4 {
    int32_t k[4];
};

template <int TH, class Visit>
__device__ __forceinline__ void each_key(const int32_t *__restrict__ keys, int n, const Visit &visit) {
    constexpr int U = 4;
    const int whole = n & ~3;
    for (int i0 = 4 * (int)threadIdx.x; i0 < whole; i0 += 4 * U * TH) {
        Keys4 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            w[u] = *reinterpret_cast<const Keys4 *>(keys + min(i0 + 4 * u * TH, whole - 4));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + 4 * u * TH;
            if (i < whole)
#pragma unroll
                for (int e = 0; e < 4; ++e) visit(i + e, w[u].k[e]);
        }
    }
    if ((int)threadIdx.x < n - whole) visit(whole + (int)threadIdx.x, keys[whole + threadIdx.x]);
}

struct Row3 {
    float v[3];
};

// For every key in [k0, k0 + nk): `own(key)` reads what the key itself needs, `each(own, item, on, sum)`
// adds what `fetch(item)` gives to its sum (nothing unless `on`), `put(key, own, sum)` takes the total; at
// least G lanes share a key.  A round lists as many keys as fit CAP items.  Rows of three floats (STAGE) are
// fetched into LDS before the sums, by all lanes and four at a time: fetched by the lanes of a key, most
// of a wave's lanes wait for its longest key, and two keys in hand to fill the waits spilled registers
// (Chamfer backward of 100 x 65,536 points 256 -> 191 us, of 40 x 8,192 18.2 -> 12.7 us).
//
// A heavy key has a round and the whole workgroup for itself.  Its items, and those of a round of few long
// keys, are listed thread by thread: each thread counts its own, and puts them behind those of the threads
// before.  (More items than fit are summed straight from the keys, each thread its every TH-th.)  20 of 19,602
// faces with all of a frame's 65,536 points take 435 us, ranked like the others 4,460 us; 200 of them in 40
// frames 0.87 and 1.33 ms.  Rounds for ranges
// without such keys (HEAVY false) are compiled by themselves: in common code the others' registers spilled.
template <int TH, int M, bool STAGE, bool HEAVY, class Own, class Fetch, class Each, class Put>
__device__ __forceinline__ void sum_rounds(const int32_t *__restrict__ keys, int n, int k0, int nk, int G,
                                           GroupLds<TH> &s, const Own &own, const Fetch &fetch,
                                           const Each &each, const Put &put) {
    constexpr int CAP = gp_cap<TH>(), WAVES = TH / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int kb = 0; kb < nk;) {
        const int base = s.start[kb];
        int ke = nk;  // the keys of the round: the last one whose items still fit
        if (s.start[nk] - base > CAP) {
            int lo = kb, hi = nk;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s.start[mid] - base <= CAP)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            ke = lo;
        }
        bool heavy = false;
        if (HEAVY) {  // the round ends before a heavy key, or is one
            __syncthreads();
            if (tid == 0) s.heavy = nk;
            __syncthreads();
            for (int k = kb + tid; k < max(ke, kb + 1); k += TH)
                if (heavy_key(s.start[k + 1] - s.start[k], n)) atomicMin(&s.heavy, k);
            __syncthreads();
            heavy = s.heavy == kb;
            ke = heavy ? kb + 1 : min(ke, s.heavy);
        }
        const int total = s.start[ke] - base;
        const bool over = HEAVY && total > CAP, listed = total > 0 && !over;
        // few long keys: comparing their items would take longer than two more passes over the keys
        const bool by_thread = HEAVY && listed && ke - kb <= GP_LONG &&
                               heavy_key(total, n * (ke - kb));
        if (by_thread) {
            const int keys_now = ke - kb;
            for (int k = 0; k < keys_now; ++k) s.own[k][tid] = 0;
            each_key<TH>(keys, n, [&](int, int key) {
                const unsigned k = key - k0 - kb;
                if (k < (unsigned)keys_now) ++s.own[k][tid];
            });
            __syncthreads();
            for (int k = wave; k < keys_now; k += WAVES) {  // counts to places, a wave a key
                constexpr int PER = TH / 64;
                unsigned short *c = &s.own[k][lane * PER];
                int sum = 0;
                for (int u = 0; u < PER; ++u) sum += c[u];
                int at = sum;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int o = __shfl_up(at, off, 64);
                    if (lane >= off) at += o;
                }
                at += s.start[kb + k] - base - sum;
                for (int u = 0; u < PER; ++u) {
                    const int next = at + c[u];
                    c[u] = (unsigned short)at;
                    at = next;
                }
            }
            __syncthreads();
            each_key<TH>(keys, n, [&](int i, int key) {
                const unsigned k = key - k0 - kb;
                if (k < (unsigned)keys_now) s.item[s.own[k][tid]++] = i;
            });
            __syncthreads();
        } else if (listed) {
            for (int k = kb + tid; k < ke; k += TH) s.cursor[k] = s.start[k] - base;
            __syncthreads();
            each_key<TH>(keys, n, [&](int i, int key) {
                const int k = key - k0;
                if (k >= kb && k < ke)
                    s.listed[atomicAdd(&s.cursor[k], 1)] = ((unsigned)k << GP_IBITS) | (unsigned)i;
            });
            __syncthreads();
            for (int p = tid; p < total; p += TH) {
                const unsigned w = s.listed[p];
                const int k = (int)(w >> GP_IBITS);
                const int lo = s.start[k] - base, hi = s.start[k + 1] - base;
                int at = lo;
#pragma unroll 4
                for (int e = lo; e < hi; ++e) at += s.listed[e] < w ? 1 : 0;
                s.item[at] = (int)(w & (GP_MAX - 1));
            }
            __syncthreads();
        }
        if constexpr (STAGE) {
            if (listed) {
                constexpr int PER = CAP / TH;
                decltype(fetch(0)) f[PER];
#pragma unroll
                for (int u = 0; u < PER; ++u) f[u] = fetch(s.item[min(tid + u * TH, total - 1)]);
                __syncthreads();
#pragma unroll
                for (int u = 0; u < PER; ++u)
                    if (tid + u * TH < total)
#pragma unroll
                        for (int d = 0; d < 3; ++d) s.row[d][tid + u * TH] = f[u].v[d];
                __syncthreads();
            }
        }
        if (over) {
            const auto whole = own(k0 + kb);
            double v[M];
#pragma unroll
            for (int m = 0; m < M; ++m) v[m] = 0.0;
#pragma unroll 1
            for (int i = tid; i < n; i += TH) each(whole, fetch(i), keys[i] == k0 + kb, v);
            team_sum(v, 64);
            if (lane == 0)
#pragma unroll
                for (int m = 0; m < M; ++m) s.part[wave][m] = v[m];
            __syncthreads();
        }
        // Lanes per key: G, and more where the round's keys have far more items than the average key that G
        // is for (a few neighbouring keys then hold most items, and most lanes would have none: points of 50
        // of 4,802 faces, 8,192 of them, 102 us with four lanes a face, 47 with more).
        int team = G;
        while (team < 64 && total > 8 * team * (ke - kb) && 2 * team * (ke - kb) <= TH) team *= 2;
        if (heavy) team = TH;
        const int per = TH / team, l = tid & (team - 1);
#pragma unroll 1
        for (int k = kb + tid / team; k < ke; k += per) {
            double v[M];
            const auto mine = own(k0 + k);
            const int hi = over ? 0 : s.start[k + 1] - base;
#pragma unroll
            for (int m = 0; m < M; ++m) v[m] = 0.0;
#pragma unroll 1
            for (int e = s.start[k] - base + l; e < hi; e += team) {
                decltype(fetch(0)) f;
                if constexpr (STAGE)
#pragma unroll
                    for (int d = 0; d < 3; ++d) f.v[d] = s.row[d][e];
                else
                    f = fetch(s.item[e]);
                each(mine, f, true, v);
            }
            team_sum(v, min(team, 64));
            if (heavy) {  // one key, so all threads are here
                if (!over && lane == 0)
#pragma unroll
                    for (int m = 0; m < M; ++m) s.part[wave][m] = v[m];
                __syncthreads();
#pragma unroll 1
                for (int w = over ? 0 : 1; w < WAVES; ++w)
#pragma unroll
                    for (int m = 0; m < M; ++m) v[m] += s.part[w][m];
            }
            if (l == 0) put(k0 + k, mine, v);
        }
        __syncthreads();  // the next round lists anew
        kb = ke;
    }
}

template <int TH, int M, bool STAGE, class Own, class Fetch, class Each, class Put>
__device__ __forceinline__ void grouped_sums(const int32_t *__restrict__ keys, int n, int k0, int nk,
                                             int G, GroupLds<TH> &s, const Own &own, const Fetch &fetch,
                                             const Each &each, const Put &put) {
    constexpr int CAP = gp_cap<TH>();
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int k = tid; k < nk; k += TH) s.cursor[k] = 0;
    if (tid == 0) s.heavy = s.some_long = 0;
    __syncthreads();
    each_key<TH>(keys, n, [&](int i, int key) {
        const int k = key - k0;
        if ((unsigned)k < (unsigned)nk) atomicAdd(&s.cursor[k], 1);
    });
    __syncthreads();
    {  // counts to starts
        constexpr int PER = CAP / TH;
        int c[PER], sum = 0, most = 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int k = tid * PER + u;
            c[u] = k < nk ? s.cursor[k] : 0;
            sum += c[u];
            most = max(most, c[u]);
        }
        if (heavy_key(most, n)) s.heavy = 1;
        if (most >= CAP / GP_LONG) s.some_long = 1;
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        if (lane == 63) s.wsum[wave] = incl;
        __syncthreads();
        int at = incl - sum;
        for (int w = 0; w < wave; ++w) at += s.wsum[w];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int k = tid * PER + u;
            if (k <= nk) s.start[k] = at;
            at += c[u];
        }
        if (tid == TH - 1 && nk == CAP) s.start[nk] = at;
        __syncthreads();
    }
    if (s.heavy || (s.some_long && s.start[nk] > CAP))
        sum_rounds<TH, M, STAGE, true>(keys, n, k0, nk, G, s, own, fetch, each, put);
    else
        sum_rounds<TH, M, STAGE, false>(keys, n, k0, nk, G, s, own, fetch, each, put);
}

// keys per workgroup, workgroups, and lanes per key for `n` items of `K` keys, `sets` times over
struct GroupPlan {
    int threads, keys, ranges, team;
};

// x = range of rows, y = frame, z = side - first (side 0: the gradient to a, 1: to b)
struct GroupChamferParams {
    const double *grad_loss;
    const float *frame_w;
    struct Side {
        const float *X;
        const int32_t *nn;  // x's neighbours in y, or NULL
        float *gX;
        int N, keys, team, pad;
    } side[2];
    double cself[2];  // cs of the two sides; cm of one is cs of the other
    int first, pad;   // the side of z = 0
};

template <int TH>
__device__ __forceinline__ void group_chamfer_body(const GroupChamferParams &pr, const Blk &blk) {
    __shared__ GroupLds<TH> lds;
    const bool b = blk.z + pr.first != 0;
    const GroupChamferParams::Side x = b ? pr.side[1] : pr.side[0], y = b ? pr.side[0] : pr.side[1];
    const int t = blk.y, k0 = blk.x * x.keys;
    if (k0 >= x.N) return;
    const int nk = min(x.keys, x.N - k0);
    const double g = pr.grad_loss[t] * (pr.frame_w ? (double)pr.frame_w[t] : 1.0);
    const double cself = b ? pr.cself[1] : pr.cself[0], cmutual = b ? pr.cself[0] : pr.cself[1];
    const double cs = cself * g, cm = cmutual * g;
    // a side without the term has no indices for it, whatever the upstream gradient (0 NaN is not 0)
    const bool self = cself != 0.0 && cs != 0.0, mutual = cmutual != 0.0 && cm != 0.0;
    const float *xt = x.X + (size_t)t * x.N * 3;
    const float *yt = y.X + (size_t)t * y.N * 3;
    struct Own {
        float x[3], y[3];  // the row, and its neighbour
        bool near;
    };
    auto own = [&](int i) {
        Own o;
        const int j = self ? x.nn[(size_t)t * x.N + i] : -1;
        o.near = (unsigned)j < (unsigned)y.N;  // indices outside [0, Ny) contribute nothing
        const float *py = yt + 3 * (size_t)(o.near ? j : 0);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            o.x[d] = xt[3 * (size_t)i + d];
            o.y[d] = py[d];
        }
        return o;
    };
    // in double (each difference of two floats is exact there) and rounded once to float, as below
    auto fetch = [&](int j) {
        const float *py = yt + 3 * (size_t)j;
        return Row3{{py[0], py[1], py[2]}};
    };
    auto each = [](const Own &o, const Row3 &y, bool on, double (&v)[3]) {
#pragma unroll
        for (int d = 0; d < 3; ++d) v[d] += on ? (double)o.x[d] - (double)y.v[d] : 0.0;
    };
    auto put = [&](int i, const Own &o, double (&v)[3]) {
        float *g3 = x.gX + ((size_t)t * x.N + i) * 3;
        float r[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double s = 0.0;
            if (o.near) s = cs * ((double)o.x[d] - (double)o.y[d]);
            if (mutual) s += cm * v[d];
            r[d] = (float)s;
        }
        g3[0] = r[0];
        g3[1] = r[1];
        g3[2] = r[2];
    };
    // without the mutual term there is nothing to group
    grouped_sums<TH, 3, true>(y.nn ? y.nn + (size_t)t * y.N : nullptr, mutual ? y.N : 0, k0, nk,
                                 x.team, lds, own, fetch, each, put);
}

template <int TH>
__global__ __launch_bounds__(TH, 8) void k_group_chamfer(GroupChamferParams p) {
    group_chamfer_body<TH>(p, grid_blk_xcd());
}

// x = range of faces, y = frame
struct GroupFaceParams {
    const float *gpts;
    const float *bary;
    const int32_t *face_idx;
    float *fg;
    int F, N, keys, team;
};

template <int TH>
__device__ __forceinline__ void group_face_body(const GroupFaceParams &pr, const Blk &blk) {
    __shared__ GroupLds<TH> lds;
    const int t = blk.y, k0 = blk.x * pr.keys;
    const float *gt = pr.gpts + (size_t)t * pr.N * 3;
    const float *bt = pr.bary + (size_t)t * pr.N * 3;
    float *ft = pr.fg + (size_t)t * pr.F * 9;
    auto own = [](int) { return 0; };
    auto fetch = [](int i) { return i; };
    auto each = [&](int, int i, bool on, double (&v)[9]) {
        const float *g = gt + 3 * (size_t)i, *b = bt + 3 * (size_t)i;
        const float f0 = g[0], f1 = g[1], f2 = g[2], w3[3] = {b[0], b[1], b[2]};
        const double g0 = on ? f0 : 0.f, g1 = on ? f1 : 0.f, g2 = on ? f2 : 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double w = on ? w3[c] : 0.f;
            v[3 * c] = __builtin_fma(w, g0, v[3 * c]);
            v[3 * c + 1] = __builtin_fma(w, g1, v[3 * c + 1]);
            v[3 * c + 2] = __builtin_fma(w, g2, v[3 * c + 2]);
        }
    };
    auto put = [&](int f, int, double (&v)[9]) {
#pragma unroll
        for (int m = 0; m < 9; ++m) ft[9 * (size_t)f + m] = (float)v[m];
    };
    grouped_sums<TH, 9, false>(pr.face_idx + (size_t)t * pr.N, pr.N, k0, min(pr.keys, pr.F - k0),
                                  pr.team, lds, own, fetch, each, put);
}

template <int TH>
__global__ __launch_bounds__(TH, 8) void k_group_face(GroupFaceParams p) {
    group_face_body<TH>(p, grid_blk_xcd());
}

// x = range of vertices, y = frame
struct GroupVertexParams {
    const float *fg;
    const int32_t *faces;
    float *gverts;
    int V, F, keys, team;
};

template <int TH>
__device__ __forceinline__ void group_vertex_body(const GroupVertexParams &pr, const Blk &blk) {
    __shared__ GroupLds<TH> lds;
    const int t = blk.y, k0 = blk.x * pr.keys;
    const float *ft = pr.fg + (size_t)t * pr.F * 9;
    float *gv = pr.gverts + (size_t)t * pr.V * 3;
    auto own = [](int) { return 0; };
    auto fetch = [&](int fc) {  // fc = 3 f + c
        const float *p = ft + 3 * (size_t)fc;
        return Row3{{p[0], p[1], p[2]}};
    };
    auto each = [](int, const Row3 &r, bool on, double (&v)[3]) {
#pragma unroll
        for (int d = 0; d < 3; ++d) v[d] += on ? (double)r.v[d] : 0.0;
    };
    auto put = [&](int v, int, double (&s)[3]) {
#pragma unroll
        for (int d = 0; d < 3; ++d) gv[3 * (size_t)v + d] = (float)s[d];
    };
    grouped_sums<TH, 3, true>(pr.faces, 3 * pr.F, k0, min(pr.keys, pr.V - k0), pr.team, lds, own,
                                 fetch, each, put);
}

template <int TH>
__global__ __launch_bounds__(TH, 8) void k_group_vertex(GroupVertexParams p) {
    group_vertex_body<TH>(p, grid_blk_xcd());
}

// keys per workgroup, so that its items are about 3/4 of what fits at once and there are workgroups
// for the chip; lanes per key, by the items an average key has
GroupPlan group_plan(long n, long K, long sets) {
    GroupPlan g;
    g.threads = n > GP_WIDE ? GP_LARGE : GP_SMALL;
    const long cap = 4L * g.threads;
    const long spread = (K * sets + 511) / 512;  // 512 workgroups
    const long keys = std::min({K * (cap * 3 / 4) / std::max(n, 1L), std::max(spread, 16L), cap, K});
    g.keys = (int)std::max(keys, 1L);
    g.ranges = (int)((K + g.keys - 1) / g.keys);
    const long avg = n / std::max(K, 1L);
    g.team = avg < 2 ? 1 : (avg < 16 ? 4 : (avg < 128 ? 16 : 64));
    return g;
}

// Up to GP_MAX items: beyond, so many workgroups would read all keys that the sort is the cheaper way.
bool grouped_pays(long n) { return n <= GP_MAX; }

template <class P>
void dispatch_group(int type, void (*small)(P), void (*large)(P), int threads, dim3 grid, const P &p,
                    hipStream_t s) {
    if (threads == GP_LARGE)
        dispatch(type + 1, large, grid, GP_LARGE, p, s);
    else
        dispatch(type, small, grid, GP_SMALL, p, s);
}

}  // namespace

size_t chamfer_bwd_scratch_bytes(int T, int Na, int Nb, bool want_b) {
    size_t s = 2 * Arena::need((size_t)T * Nb, 4) + segsort_scratch_bytes(T, Nb) +
               Arena::need((size_t)T * (Na + 1), 4);
    if (want_b)
        s += 2 * Arena::need((size_t)T * Na, 4) + segsort_scratch_bytes(T, Na) +
             Arena::need((size_t)T * (Nb + 1), 4);
    return s;
}

// one side by the sort: x's mutual terms are the y's grouped by their neighbour in x
static void launch_sorted_side(ChamferBwdParams &cp, const int32_t *nn_y, int T, Arena &ar,
                               hipStream_t s) {
    int32_t *k = ar.take<int32_t>((size_t)T * cp.Ny);
    int32_t *v = ar.take<int32_t>((size_t)T * cp.Ny);
    char *ss = ar.take<char>(segsort_scratch_bytes(T, cp.Ny));
    int32_t *st = ar.take<int32_t>((size_t)T * (cp.Nx + 1));
    cp.ystart = st;
    cp.yvals_sorted = v;
    if (cp.cmutual != 0.0) {
        // valid neighbours lie in [0, Nx): Nx - 1 is the key limit, out-of-range ones are marked
        launch_segsort(nn_y, T, cp.Ny, cp.Nx - 1, k, v, ss, s, true);
        BoundsParams bp;
        bp.sorted = k;
        bp.start = st;
        bp.N = cp.Ny;
        bp.K = cp.Nx;
        dispatch(KT_BOUNDS, k_bounds, dim3((cp.Ny + BW_THREADS) / BW_THREADS, T), BW_THREADS, bp, s);
    }
    dispatch(KT_CHAMFER_BWD, k_chamfer_bwd, dim3((cp.Nx + BW_THREADS - 1) / BW_THREADS, T),
             BW_THREADS, cp, s);
}

void launch_chamfer_bwd(const double *grad_loss, const float *a, const float *b,
                        const int32_t *idx_a, const int32_t *idx_b, int T, int Na, int Nb,
                        int reduction, const float *frame_w, float *grad_a, float *grad_b,
                        char *scratch, hipStream_t s) {
    const bool eq2 = reduction == DC_RED_SIM2REAL_SUM;
    const double alpha = eq2 ? 1.0 : 1.0 / (double)Na;
    const double beta = eq2 ? 0.0 : 1.0 / (double)Nb;
    Arena ar;
    ar.base = scratch;
    ar.cap = chamfer_bwd_scratch_bytes(T, Na, Nb, grad_b != nullptr);
    // the a side groups the b points (when beta != 0), the b side the a points
    const long items_a = beta != 0.0 ? Nb : 0;
    // (with nothing to group, the path of the sort only has its last kernel: 100 x 65,536 rows take 73 us
    // in it, 113 us in the grouped one)
    const bool group_a = items_a > 0 && grouped_pays(items_a), group_b = grad_b && grouped_pays(Na);
    if (group_a || group_b) {
        GroupChamferParams gp;
        gp.grad_loss = grad_loss;
        gp.frame_w = frame_w;
        const GroupPlan pa = group_plan(items_a, Na, T), pb = group_plan(Na, Nb, T);
        gp.side[0] = {a, idx_a, grad_a, Na, pa.keys, pa.team, 0};
        gp.side[1] = {b, beta != 0.0 ? idx_b : nullptr, grad_b, Nb, pb.keys, pb.team, 0};
        gp.cself[0] = 2.0 * alpha;
        gp.cself[1] = 2.0 * beta;
        gp.pad = 0;
        auto launch = [&](int first, int sides, int threads, int ranges) {
            gp.first = first;
            dispatch_group(KT_GROUP_CHAMFER, k_group_chamfer<GP_SMALL>, k_group_chamfer<GP_LARGE>,
                           threads, dim3(ranges, T, sides), gp, s);
        };
        // One launch for both sides where they take workgroups of one size.  The size decides how a key of
        // many items is summed, so a side keeps its own: its sums don't depend on whether the other side's
        // are wanted.
        if (group_a && group_b && pa.threads == pb.threads) {
            launch(0, 2, pa.threads, std::max(pa.ranges, pb.ranges));
        } else {
            if (group_a) launch(0, 1, pa.threads, pa.ranges);
            if (group_b) launch(1, 1, pb.threads, pb.ranges);
        }
    }
    ChamferBwdParams cp;
    cp.grad_loss = grad_loss;
    cp.frame_w = frame_w;
    if (!group_a) {
        cp.X = a;
        cp.Y = b;
        cp.nn_x = idx_a;
        cp.gX = grad_a;
        cp.cself = 2.0 * alpha;
        cp.cmutual = 2.0 * beta;
        cp.Nx = Na;
        cp.Ny = Nb;
        launch_sorted_side(cp, idx_b, T, ar, s);
    }
    if (grad_b && !group_b) {
        cp.X = b;
        cp.Y = a;
        cp.nn_x = idx_b;
        cp.gX = grad_b;
        cp.cself = 2.0 * beta;
        cp.cmutual = 2.0 * alpha;
        cp.Nx = Nb;
        cp.Ny = Na;
        launch_sorted_side(cp, idx_a, T, ar, s);
    }
}

size_t sample_bwd_scratch_bytes(int T, int V, int F, int N) {
    return 2 * Arena::need((size_t)T * N, 4) + segsort_scratch_bytes(T, N) +
           Arena::need((size_t)T * (F + 1), 4) + 2 * Arena::need((size_t)3 * F, 4) +
           segsort_scratch_bytes(1, 3 * F) + Arena::need((size_t)V + 1, 4) +
           Arena::need((size_t)T * F * 9, 4);
}

void launch_sample_bwd(const float *grad_points, const int32_t *faces, const int32_t *face_idx,
                       const float *bary, int T, int V, int F, int N, float *grad_verts,
                       char *scratch, hipStream_t s) {
    Arena ar;
    ar.base = scratch;
    ar.cap = sample_bwd_scratch_bytes(T, V, F, N);
    float *fg = ar.take<float>((size_t)T * F * 9);
    BoundsParams bp;
    // points grouped by face (face -1 of a degenerate frame is left out: it belongs to no face)
    if (grouped_pays(N)) {
        const GroupPlan pf = group_plan(N, F, T);
        GroupFaceParams gf;
        gf.gpts = grad_points;
        gf.bary = bary;
        gf.face_idx = face_idx;
        gf.fg = fg;
        gf.F = F;
        gf.N = N;
        gf.keys = pf.keys;
        gf.team = pf.team;
        dispatch_group(KT_GROUP_FACE, k_group_face<GP_SMALL>, k_group_face<GP_LARGE>, pf.threads,
                       dim3(pf.ranges, T), gf, s);
    } else {
        int32_t *fk = ar.take<int32_t>((size_t)T * N);
        int32_t *fv = ar.take<int32_t>((size_t)T * N);
        char *ss1 = ar.take<char>(segsort_scratch_bytes(T, N));
        int32_t *fstart = ar.take<int32_t>((size_t)T * (F + 1));
        // (face -1 sorts last, as key F, and is unused)
        launch_segsort(face_idx, T, N, F, fk, fv, ss1, s);
        bp.sorted = fk;
        bp.start = fstart;
        bp.N = N;
        bp.K = F;
        dispatch(KT_BOUNDS, k_bounds, dim3((N + BW_THREADS) / BW_THREADS, T), BW_THREADS, bp, s);
        FaceGradParams fp;
        fp.gpts = grad_points;
        fp.bary = bary;
        fp.pts_by_face = fv;
        fp.face_start = fstart;
        fp.fg = fg;
        fp.F = F;
        fp.N = N;
        dispatch(KT_FACE_GRAD, k_face_grad, dim3((F + BW_THREADS - 1) / BW_THREADS, T), BW_THREADS,
                 fp, s);
    }
    // (face, corner) slots grouped by vertex: the vertex-incidence lists of the topology
    if (grouped_pays(3L * F)) {
        const GroupPlan pv = group_plan(3L * F, V, T);
        GroupVertexParams gv;
        gv.fg = fg;
        gv.faces = faces;
        gv.gverts = grad_verts;
        gv.V = V;
        gv.F = F;
        gv.keys = pv.keys;
        gv.team = pv.team;
        dispatch_group(KT_GROUP_VERTEX, k_group_vertex<GP_SMALL>, k_group_vertex<GP_LARGE>, pv.threads,
                       dim3(pv.ranges, T), gv, s);
        return;
    }
    int32_t *ck = ar.take<int32_t>((size_t)3 * F);
    int32_t *cv = ar.take<int32_t>((size_t)3 * F);
    char *ss2 = ar.take<char>(segsort_scratch_bytes(1, 3 * F));
    int32_t *vstart = ar.take<int32_t>((size_t)V + 1);
    launch_segsort(faces, 1, 3 * F, V, ck, cv, ss2, s);
    bp.sorted = ck;
    bp.start = vstart;
    bp.N = 3 * F;
    bp.K = V;
    dispatch(KT_BOUNDS, k_bounds, dim3((3 * F + BW_THREADS) / BW_THREADS, 1), BW_THREADS, bp, s);
    VertexGradParams vp;
    vp.fg = fg;
    vp.corners_by_vertex = cv;
    vp.vert_start = vstart;
    vp.gverts = grad_verts;
    vp.V = V;
    vp.F = F;
    dispatch(KT_VERTEX_GRAD, k_vertex_grad, dim3((V + BW_THREADS - 1) / BW_THREADS, T), BW_THREADS,
             vp, s);
}

void register_backward_kernels(BatchedKernel *table) {
    table[KT_CHAMFER_BWD] = batched_kernel<ChamferBwdParams, chamfer_bwd_body, BW_THREADS, 1024>();
    table[KT_BOUNDS] = batched_kernel<BoundsParams, bounds_body, BW_THREADS, 512>();
    table[KT_FACE_GRAD] = batched_kernel<FaceGradParams, face_grad_body, BW_THREADS, 1024>();
    // each type's large workgroups follow its small ones
    // (at the eight waves per SIMD of the direct kernels the batched ones of the chamfer and face sums
    // spill: a request of 38 frames 12.2 -> 11.0 and 15.7 -> 13.3 us without)
    table[KT_GROUP_CHAMFER] = batched_kernel<GroupChamferParams, group_chamfer_body<GP_SMALL>, GP_SMALL, 1024, 6>();
    table[KT_GROUP_CHAMFER + 1] = batched_kernel<GroupChamferParams, group_chamfer_body<GP_LARGE>, GP_LARGE, 512, 4>();
    table[KT_GROUP_FACE] = batched_kernel<GroupFaceParams, group_face_body<GP_SMALL>, GP_SMALL, 1024, 6>();
    table[KT_GROUP_FACE + 1] = batched_kernel<GroupFaceParams, group_face_body<GP_LARGE>, GP_LARGE, 512, 4>();
    table[KT_GROUP_VERTEX] = batched_kernel<GroupVertexParams, group_vertex_body<GP_SMALL>, GP_SMALL, 1024, 8>();
    table[KT_GROUP_VERTEX + 1] = batched_kernel<GroupVertexParams, group_vertex_body<GP_LARGE>, GP_LARGE, 512, 8>();
    table[KT_VERTEX_GRAD] = batched_kernel<VertexGradParams, vertex_grad_body, BW_THREADS, 1024>();
}

}  // namespace dc

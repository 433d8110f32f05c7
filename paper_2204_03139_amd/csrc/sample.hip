// Area-weighted surface sampling (arXiv 2204.03139, Sec. III-B, Eq. 3).
//
// Two kernels per call:
//   k_area_cdf   one workgroup per frame: face areas in double, then the running sum
//                C_k = C_{k-1} + A_k in double, equal bit for bit to the left-to-right sum (index
//                stability needs the same rounding as a sequential sum).  Bounded by the doubles'
//                instructions of the one CU: 6 us for the areas and sums of 2,560 faces.  One wave
//                on the sums, the others on the next areas, took 38.7 us for 40 frames of 4,802 faces
//                and 77.8 us for 100 of 19,602; all waves on both take 18.0 and 52.8 us.
//   k_sample     one lane per point: random words (given, or Philox4x64-10), inverse-CDF face
//                choice by an upper-bound search, barycentric point in float (k_sample_wide where
//                there are enough points).
// Built with -ffp-contract=off: only the fma calls written out below are fused.
#include <algorithm>

#include "batch.h"

namespace dc {
namespace {

// Threads of a workgroup and most faces per thread and chunk.  Fewer threads have their sums sooner,
// more of them share the doubles' instructions of a longer mesh: with 512 x 5 faces one frame of 1,152
// faces takes 10.8 us, 40 frames of 4,802 18.0 us, 24 of 12,482 34.4 us and 100 of 19,602 52.8 us (launch
// included), with 256 x 5 9.5, 21.8, 44.2 and 70.2 us and with 1,024 x 5 15.1, 19.8, 37.0 and 52.8 us.
// The smallest meshes, of one face per thread, are bound by the length of the code alone: 25 frames of
// 72 faces take 6.6 us with 256 x 1 and 9.4 us with 512 x 5.
constexpr int AC_THREADS = 512, AC_PER = 5;
constexpr int AC_SMALL = 256;  // threads, and most faces, of a small mesh
constexpr int AC_STEPS = 64;   // most single additions of a chunk summed by all waves

__device__ __forceinline__ bool face_ok(const int32_t *fv, int V) {
    const int32_t i0 = fv[0], i1 = fv[1], i2 = fv[2];
    return (unsigned)i0 < (unsigned)V && (unsigned)i1 < (unsigned)V && (unsigned)i2 < (unsigned)V;
}

// |(p2-p1) x (p3-p1)| / 2 with every product and difference rounded in double.
__device__ __forceinline__ double tri_area_f64(const float *p1, const float *p2, const float *p3) {
    const double ax = (double)p2[0] - (double)p1[0];
    const double ay = (double)p2[1] - (double)p1[1];
    const double az = (double)p2[2] - (double)p1[2];
    const double bx = (double)p3[0] - (double)p1[0];
    const double by = (double)p3[1] - (double)p1[1];
    const double bz = (double)p3[2] - (double)p1[2];
    const double nx = ay * bz - az * by;
    const double ny = az * bx - ax * bz;
    const double nz = ax * by - ay * bx;
    const double sq = nx * nx + ny * ny + nz * nz;
    return 0.5 * __builtin_sqrt(sq);
}

// The running sum over one chunk, in place over entries [0, n) of cur, continuing from `run` (the
// sum of the chunks before it), by the 64 lanes of one wave.  The result is the left-to-right
// double sum C_k = C_{k-1} + A_k bit for bit, without its chain of dependent additions:
//   While a partial sum s lies in one binade [2^E, 2^(E+1)), it is an integer multiple m of the
//   spacing u = 2^(E-52) there, and rounding s + A to that grid does not depend on m: with
//   A / u = q + f (q an integer, 0 <= f < 1) the rounded sum is (m + q + [f > 1/2]) u, except
//   when f is exactly 1/2 (the tie goes to the even multiple, which depends on m) or when
//   m + q + [f > 1/2] reaches 2^53 (the sum leaves the binade and the grid changes).
// So the sums over a window of 64 x RS_PER areas are m_0 plus a prefix sum of the integers
// q + [f > 1/2], taken by a wave scan in double: a sum of non-negative integers is exact while it
// is below 2^53 and, rounded, stays at or above 2^53 once it reaches it, whatever the order.  The
// first area of the window that is a tie or leaves the binade (a NaN or infinite area does) is
// added by one lane exactly as in the plain chain, and the next window starts after it; when a
// window stops within its first RS_BURST positions the lane goes on through RS_BURST areas, so ties
// or binade changes in a row cost no more than the plain chain.  A zero sum skips the zero areas
// after it (0 + 0 = 0); a sum that is not finite, or below the normal range, ends the chunk in the
// plain chain.  `cur` is a chunk buffer: entries [n, n + RS_WIN) are padding that a window may
// load, and the 64 slots from CHUNK + RS_WIN on take the stores a window does not want.
constexpr int RS_PER = 15;  // odd: lanes 120 bytes apart read and write on different LDS banks
constexpr int RS_WIN = 64 * RS_PER;
constexpr int RS_BURST = 64;

// the value of lane (l - n) in the same row of 16 lanes, or 0 where that is outside the row
template <int CTRL>
__device__ __forceinline__ double row_shifted(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo =
        (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// the value of lane l - 1 (0 on lane 0)
__device__ __forceinline__ double lane_before(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo =
        (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x138, 0xF, 0xF, true);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x138, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double lane_value(double v, int l) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// sum of v over lanes 0..lane (v: non-negative integers in double)
__device__ __forceinline__ double wave_prefix(double v, int lane) {
    v = v + row_shifted<0x111>(v);  // row_shr:1
    v = v + row_shifted<0x112>(v);  // row_shr:2
    v = v + row_shifted<0x114>(v);  // row_shr:4
    v = v + row_shifted<0x118>(v);  // row_shr:8
    const double r0 = lane_value(v, 15), r1 = lane_value(v, 31), r2 = lane_value(v, 47);
    const double r01 = r0 + r1;
    const int row = lane >> 4;
    if (row == 1) v = v + r0;
    if (row == 2) v = v + r01;
    if (row == 3) v = v + (r01 + r2);
    return v;
}

// the sums of d and of n over lanes 0..lane (d modulo 2^64)
template <int CTRL>
__device__ __forceinline__ void add_shifted(unsigned long long &d, int &n) {
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)d, CTRL, 0xF, 0xF, true);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(d >> 32), CTRL, 0xF, 0xF, true);
    n += __builtin_amdgcn_update_dpp(0, n, CTRL, 0xF, 0xF, true);
    d += ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ unsigned long long lane_word(unsigned long long d, int l) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)d, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(d >> 32), l);
    return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ void wave_count(unsigned long long &d, int &n, int lane) {
    add_shifted<0x111>(d, n);  // row_shr:1
    add_shifted<0x112>(d, n);  // row_shr:2
    add_shifted<0x114>(d, n);  // row_shr:4
    add_shifted<0x118>(d, n);  // row_shr:8
    unsigned long long ad = 0;
    int an = 0;
#pragma unroll
    for (int row = 1; row < 4; ++row) {
        const unsigned long long rd = lane_word(d, 16 * row - 1);
        const int rn = __builtin_amdgcn_readlane(n, 16 * row - 1);
        if (lane >> 4 >= row) {
            ad += rd;
            an += rn;
        }
    }
    d += ad;
    n += an;
}

__device__ __forceinline__ void plain_sum(double *cur, int i0, int i1, double &run) {
    double r = run;
    int i = i0;
    for (; i + 8 <= i1; i += 8) {  // eight loads in flight, then eight dependent additions
        double x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = cur[i + j];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            r = r + x[j];
            cur[i + j] = r;
        }
    }
    for (; i < i1; ++i) {
        r = r + cur[i];
        cur[i] = r;
    }
    run = r;
}

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int CHUNK>
__device__ void running_sum(double *cur, int n, double &run, int lane) {
    constexpr double LIM = 9007199254740992.0;  // 2^53
    int k = 0;
    while (k < n) {
        const int avail = n - k;
        const double s = run;  // the same on every lane
        const int eb = (int)(((unsigned long long)__double_as_longlong(s) >> 52) & 0x7FF);
        const int base = lane * RS_PER;
        int stop;  // window position where the plain chain takes over
        if (s == 0.0) {
            int first = RS_PER;
#pragma unroll
            for (int i = RS_PER - 1; i >= 0; --i) {
                const double a = cur[k + base + i];  // past the chunk: the buffer's padding
                if (base + i < avail && a != 0.0) first = i;
            }
            const unsigned long long bal = __ballot(first < RS_PER);
            if (!bal) {  // only zero areas here: their entries are already the zero sums
                k += min(RS_WIN, avail);
                continue;
            }
            const int l = __ffsll((long long)bal) - 1;
            stop = l * RS_PER + __builtin_amdgcn_readlane(first, l);
        } else if (eb == 0 || eb == 0x7FF) {  // below the normal range, infinite or NaN
            if (lane == 0) plain_sum(cur, k, n, run);
            run = lane_value(run, 0);
            return;
        } else {
            const int sh = 1075 - eb;                  // the spacing of s's binade is 2^-sh
            const double ms = __builtin_ldexp(s, sh);  // s / u: an integer in [2^52, 2^53)
            double pre[RS_PER];
            int tie = RS_PER;  // the lane's first tie
            double acc = 0.0;
#pragma unroll
            for (int i = 0; i < RS_PER; ++i) {
                const double raw = cur[k + base + i];  // past the chunk: the buffer's padding
                const double a = base + i < avail ? raw : 0.0;
                // A / u + 1/2 is exact while A / u < 2^52, and an area whose A / u is larger
                // leaves the binade whatever its rounding: floor gives q + [f >= 1/2], and the
                // sum is exactly an integer when f is exactly 1/2 (a tie, which stops the window,
                // so that it rounds up here does not matter)
                const double y = __builtin_ldexp(a, sh) + 0.5;
                const double d = __builtin_floor(y);
                if (d == y && tie == RS_PER) tie = i;
                acc = acc + d;  // NaN and infinite areas make the sums leave the binade
                pre[i] = acc;
            }
            const double incl = wave_prefix(acc, lane);
            const double ex = lane_before(incl);  // wave_shr:1
            int inside = 0;  // positions whose sum stays in the binade (sums never decrease)
#pragma unroll
            for (int i = 0; i < RS_PER; ++i) {
                pre[i] = ms + (ex + pre[i]);  // m of position i, in units of u
                inside += pre[i] < LIM ? 1 : 0;
            }
            const int first = min(inside, tie);
            const unsigned long long bal = __ballot(first < RS_PER);
            if (bal) {
                const int l = __ffsll((long long)bal) - 1;
                stop = l * RS_PER + __builtin_amdgcn_readlane(first, l);
            } else {
                stop = RS_WIN;
            }
            // entries at or after the stop go to the lane's spare slot instead (no branches)
#pragma unroll
            for (int i = 0; i < RS_PER; ++i)
                cur[base + i < stop ? k + base + i : CHUNK + RS_WIN + lane] =
                    __builtin_ldexp(pre[i], -sh);
            if (stop == RS_WIN && avail >= RS_WIN) {  // the whole window stayed in the binade
                run = __builtin_ldexp(ms + lane_value(incl, 63), -sh);
                k += RS_WIN;
                continue;
            }
            wave_sync_lds();
            if (stop >= avail || stop == RS_WIN) {
                const int done = min(RS_WIN, avail);
                run = cur[k + done - 1];
                k += done;
                continue;
            }
        }
        // the plain chain from window position `stop`
        const int len = min(stop < RS_BURST ? RS_BURST : 1, avail - stop);
        if (lane == 0) {
            double r = stop == 0 ? s : cur[k + stop - 1];
            plain_sum(cur, k + stop, k + stop + len, r);
            run = r;
        }
        run = lane_value(run, 0);
        wave_sync_lds();
        k += stop + len;
    }
    wave_sync_lds();
}

__device__ __forceinline__ int binade(double v) {
    return (int)(((unsigned long long)__double_as_longlong(v) >> 52) & 0x7FF);
}

// what the waves of a workgroup tell each other over a chunk
template <int WAVES>
struct ChunkSums {
    double near_total[WAVES];             // sums of the waves' areas, in any order
    unsigned long long d[WAVES];          // the waves' integers, modulo 2^64
    int steps[WAVES];                     // the waves' single additions
    double area[AC_STEPS];                // of each single addition: its area,
    unsigned long long before[AC_STEPS];  // the integers before it,
    int e[AC_STEPS];                      // the binade of the sum before it
    double end;                           // the sum of the chunk
    // one wave has to sum the chunk (of even and odd chunks): seen before or after its integers
    // were summed
    int odd[2], wrong[2];
};

// The running sums of a chunk by all lanes at once, each the areas a[0..per) that follow those of the
// lane before it, from the sum `start` of the chunks before: the same integers on the grid of a binade
// as in running_sum, over several binades.  Every lane takes the binades of its partial sums from sums
// in any order (near sums).  An area whose near sums before and after it lie in one binade, and that is
// no tie, becomes an integer; the others are single additions, done in order by every wave for itself
// over at most AC_STEPS of them, each after the sum of the integers since the one before.  The integers
// are summed modulo 2^64, where the difference of two sums is exact although the units change on the
// way.  A near sum may lie on the wrong side of a binade's edge: each lane checks, against the exact
// sums, that its integers' unit is that of the binade in which their run starts and that they end in
// the same binade; then every rounding was the one of the sequential sum.  Where a check fails, or there
// are more single additions, sums that are not finite or are below the normal range, it returns false on
// all lanes and one wave sums the chunk.
template <int WAVES, int PER>
__device__ __forceinline__ bool chunk_sums(double (&a)[PER], int per, int n, double start,
                                           ChunkSums<WAVES> &c, int side, int wave, int lane) {
    double near = 0.0;
#pragma unroll
    for (int k = 0; k < PER; ++k) near = near + a[k];
    const double incl = wave_prefix(near, lane);
    if (lane == 63) c.near_total[wave] = incl;
    __syncthreads();
    double before = start;
#pragma unroll
    for (int w = 0; w < WAVES - 1; ++w) before = before + (w < wave ? c.near_total[w] : 0.0);
    before = before + lane_before(incl);
    unsigned long long run = 0, d[PER];
    int e[PER];
    int mine = 0, single = 0;
    bool odd = false;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const double after = before + a[k];
        e[k] = binade(before);
        const int e1 = binade(after);
        odd = odd || e1 == 0x7FF || (e1 == 0 && after != 0.0);
        const double y = __builtin_ldexp(a[k], 1075 - e[k]) + 0.5;
        const double q = __builtin_floor(y);
        const bool one = e[k] != e1 || q == y;
        if (one) {
            single |= 1 << k;
            ++mine;
        } else {
            run += (unsigned long long)q;
        }
        d[k] = run;
        before = after;
    }
    unsigned long long di = run;
    int ni = mine;
    wave_count(di, ni, lane);
    if (lane == 63) {
        c.d[wave] = di;
        c.steps[wave] = ni;
    }
    if (odd) c.odd[side] = 1;
    __syncthreads();
    unsigned long long base = di - run;
    int first = ni - mine, steps = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const int s = c.steps[w];
        steps += s;
        if (w < wave) {
            base += c.d[w];
            first += s;
        }
    }
    if (steps > AC_STEPS || c.odd[side]) return false;
    double sum = start, after = 0.0;  // after: of lane j, the sum after the j-th single addition
    unsigned long long at = 0;        // and the integers up to it
    if (steps) {
        int j = first;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (single >> k & 1) {
                c.area[j] = a[k];
                c.before[j] = base + d[k];
                c.e[j] = e[k];
                ++j;
            }
        }
        __syncthreads();
        double area = 0.0, gap = 0.0;
        int ej = 0;
        bool some = false;
        if (lane < steps) {
            area = c.area[lane];
            at = c.before[lane];
            ej = c.e[lane];
            const unsigned long long last = lane ? c.before[lane - 1] : 0;
            some = at != last;
            gap = __builtin_ldexp((double)(at - last), ej - 1075);
        }
        bool wrong = false;
        for (int i = 0; i < steps; ++i) {
            const double from = sum;
            sum = (sum + lane_value(gap, i)) + lane_value(area, i);
            if (lane == i) {
                wrong = some && binade(from) != ej;
                after = sum;
            }
        }
        if (wrong) c.wrong[side] = 1;
    }
    // each lane's run: the sum it starts from and the integers up to there
    double from = start;
    unsigned long long zero = 0;
    if (steps) {
        const int r = max(first - 1, 0);
        const double fs = __shfl(after, r, 64);
        const unsigned long long fz = __shfl(at, r, 64);
        if (first) {
            from = fs;
            zero = fz;
        }
    }
    int j = first;
    bool wrong = false;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const bool one = single >> k & 1;
        if (__ballot(one)) {
            const int r = min(j, 63);
            const double fs = __shfl(after, r, 64);
            const unsigned long long fz = __shfl(at, r, 64);
            if (one) {
                from = fs;
                zero = fz;
                ++j;
            }
        }
        const double v = from + __builtin_ldexp((double)(base + d[k] - zero), e[k] - 1075);
        if (!one) wrong = wrong || binade(from) != e[k] || binade(v) != e[k];
        a[k] = one ? from : v;
    }
    if (wrong) c.wrong[side] = 1;
    const int at_end = (n - 1) - (int)threadIdx.x * per;  // the chunk's last area, if it is this lane's
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (k == at_end && k < per) c.end = a[k];
    __syncthreads();
    return !c.wrong[side];
}

struct AreaCdfParams {
    const float *verts;
    const int32_t *faces;
    const uint8_t *mask;  // optional: nonzero = the face may be drawn (row t at t * mask_stride)
    size_t mask_stride;
    int V, F;
    double *cdf;
    int32_t *lastpos;
    unsigned *status;
};

// One workgroup per frame, a chunk of faces after the other, each thread on up to PER faces in a row:
// their index and corner gathers are in flight together, and the indices of the next chunk are loaded
// before the sums of this one.
template <int THREADS, int PER>
__device__ __forceinline__ void area_cdf_body(const AreaCdfParams &p, const Blk &blk) {
    const float *__restrict__ verts = p.verts;
    const int32_t *__restrict__ faces = p.faces;
    constexpr int CHUNK = THREADS * PER, WAVES = THREADS / 64;
    const int V = p.V, F = p.F;
    // a chunk that one wave sums: its areas, then their running sums; a window of padding lets the wave
    // load whole windows past the end of the chunk, and 64 spare slots take its unwanted stores
    __shared__ __align__(16) double area[CHUNK + RS_WIN + 64];
    __shared__ ChunkSums<WAVES> sums;
    __shared__ int bad;
    __shared__ int lastw[WAVES];
    const int t = blk.x, tid = threadIdx.x;
    const float *vt = verts + (size_t)t * V * 3;
    double *ct = p.cdf + (size_t)t * F;
    const int wave = tid >> 6, lane = tid & 63;
    if (tid == 0) bad = 0;
    if (tid < 2) sums.odd[tid] = sums.wrong[tid] = 0;
    int last = -1;  // last face with a positive area, per thread, then per workgroup
    auto spread = [&](int base) { return min(PER, (F - base + THREADS - 1) / THREADS); };
    int32_t fv[PER][3];
    auto load = [&](int base) {
        const int per = spread(base);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int32_t *f = faces + 3 * (size_t)min(base + tid * per + k, F - 1);
            fv[k][0] = f[0];
            fv[k][1] = f[1];
            fv[k][2] = f[2];
        }
    };
    load(0);
    __syncthreads();  // the flags are cleared before any thread may set them
    double run = 0.0;  // the running sum
    for (int base = 0, side = 0; base < F; base += CHUNK, side ^= 1) {
        const int n = min(CHUNK, F - base);
        const int per = spread(base);
        bool ok[PER];
        float q[PER][3][3];
        unsigned char keep[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = tid * per + k;
            ok[k] = face_ok(fv[k], V);
#pragma unroll
            for (int c3 = 0; c3 < 3; ++c3) {
                const float *v = vt + 3 * (size_t)(ok[k] ? fv[k][c3] : 0);
                q[k][c3][0] = v[0];
                q[k][c3][1] = v[1];
                q[k][c3][2] = v[2];
            }
            keep[k] = p.mask ? p.mask[(size_t)t * p.mask_stride + min(base + i, F - 1)] : 1;
        }
        if (base + CHUNK < F) load(base + CHUNK);
        double a[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int i = tid * per + k;
            a[k] = 0.0;
            if (k < per && i < n) {
                if (!ok[k])
                    bad = 1;
                else if (keep[k])  // a face outside the subset takes part with area 0: never drawn
                    a[k] = tri_area_f64(q[k][0], q[k][1], q[k][2]);
                if (a[k] > 0.0) last = base + i;
            }
        }
        double one[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) one[k] = a[k];
        if (chunk_sums(a, per, n, run, sums, side, wave, lane)) {
#pragma unroll
            for (int k = 0; k < PER; ++k)
                if (k < per && tid * per + k < n) ct[base + tid * per + k] = a[k];
            run = sums.end;
            if (tid == 0) sums.odd[side ^ 1] = sums.wrong[side ^ 1] = 0;
        } else {
            __syncthreads();
            if (tid < 2) sums.odd[tid] = sums.wrong[tid] = 0;
#pragma unroll
            for (int k = 0; k < PER; ++k)
                if (k < per && tid * per + k < n) area[tid * per + k] = one[k];
            __syncthreads();
            if (wave == 0) {
                running_sum<CHUNK>(area, n, run, lane);
                if (lane == 0) sums.end = run;
            }
            __syncthreads();
            for (int k = tid; k < n; k += THREADS) ct[base + k] = area[k];
            run = sums.end;
            __syncthreads();  // before the next chunk's sum takes its place
        }
    }
    // faces are visited in increasing order per thread, so the maximum is the last positive one
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) last = max(last, __shfl_xor(last, off, 64));
    if (lane == 0) lastw[wave] = last;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < WAVES; ++w) last = max(last, lastw[w]);
        const bool degenerate = !(run > 0.0) || !__builtin_isfinite(run);
        p.lastpos[t] = (degenerate || bad) ? -1 : last;
        if (bad) atomicOr(p.status, (unsigned)ST_BAD_FACE);
        if (degenerate) atomicOr(p.status, (unsigned)ST_DEGENERATE);
    }
}

template <int THREADS, int PER>
__global__ __launch_bounds__(THREADS) void k_area_cdf(AreaCdfParams p) {
    area_cdf_body<THREADS, PER>(p, grid_blk());
}

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 64x64->128 products
// with a Weyl key schedule.
struct Words4 {
    uint32_t w0, w1, w2, w3;
};

__device__ __forceinline__ Words4 philox_words(uint64_t seed, uint32_t t, uint32_t i) {
    uint64_t c0 = i, c1 = t, c2 = 0, c3 = 0;
    uint64_t k0 = seed, k1 = 0;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t m0 = 0xD2E7470EE14C6C93ull, m1 = 0xCA5A826395121157ull;
        const uint64_t p0hi = __umul64hi(m0, c0), p0lo = m0 * c0;
        const uint64_t p1hi = __umul64hi(m1, c2), p1lo = m1 * c2;
        const uint64_t n0 = p1hi ^ c1 ^ k0;
        const uint64_t n2 = p0hi ^ c3 ^ k1;
        c0 = n0;
        c1 = p1lo;
        c2 = n2;
        c3 = p0lo;
        k0 += 0x9E3779B97F4A7C15ull;
        k1 += 0xBB67AE8584CAA73Bull;
    }
    Words4 w;
    w.w0 = (uint32_t)c0;
    w.w1 = (uint32_t)(c0 >> 32);
    w.w2 = (uint32_t)(c1 >> 32);
    w.w3 = (uint32_t)(c2 >> 32);
    return w;
}

// The choice of a face, first k with C_k > r S, is a search over F sums per point.  Searched in
// memory it was a chain of log2(F) gathers (15 at 19,602 faces); most of it now runs in LDS, over
// every 2^shift-th sum laid out as a search tree (root first, each level contiguous: the lanes'
// reads of one level spread over the banks, where a sorted table would put the first levels' few
// entries on one bank), and only the last `shift` steps, within one or two cache lines, in memory.
// Monotone sums make it the same face bit for bit.  Over 100 x 19,602 faces and 100 x 65,536 points
// with given words k_sample took 298 us with the search in memory and takes 237 us with the tree.
//
// What bounds it then is cache lines: a point touches one line of the sums, one of the faces and
// two or three of the corners, and 64 lanes touch 64 different ones.  The wide kernel also holds the
// frame's corners in LDS, with as many pivots as the rest holds, one workgroup per CU walking a
// contiguous share of all points of all frames, and streams its outputs past L2, which keeps the
// sums and faces there: 117 us for the same call (183 MB written, 105 MB of words read: 2.5 TB/s),
// 164 us without the streaming.
constexpr int SP_THREADS = 512;
constexpr int SP_LEVELS = 12;        // most levels of the pivot tree: 4,095 pivots, 32 KB of LDS
constexpr int SP_CHUNK = 4096;       // most points of a workgroup
constexpr int SP_FILL = 1024;        // workgroups below which a workgroup takes fewer points
constexpr int SW_THREADS = 1024;
constexpr int SW_LEVELS = 13;
constexpr int SW_BYTES = 158 << 10;  // corners and pivots of the wide kernel
constexpr int SW_CUS = 256;

struct SampleParams {
    const float *verts;
    const int32_t *faces;
    int V, F, N, T;
    int chunk;   // points per workgroup (the wide kernel: of all frames' points in a row)
    int levels;  // levels of the pivot tree
    int shift;   // log2 of the faces per pivot
    uint64_t seed;
    const uint32_t *uniforms;
    const double *cdf;
    const int32_t *lastpos;
    float *points;
    int32_t *face_idx;
    float *bary;
};

template <bool STREAM, class T>
__device__ __forceinline__ void put(T *p, T v) {
    if (STREAM)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// the points [i0, i1) of frame t, by THREADS threads; `corners`: the frame's, in LDS or memory
template <int THREADS, bool STREAM>
__device__ __forceinline__ void sample_points(const SampleParams &pr, int t, int i0, int i1, int lp,
                                              const double *pivot, double total,
                                              const float *corners) {
    const int32_t *__restrict__ faces = pr.faces;
    const int F = pr.F, N = pr.N;
    const uint32_t *__restrict__ uniforms = pr.uniforms;
    float *__restrict__ points = pr.points;
    int32_t *__restrict__ face_idx = pr.face_idx;
    float *__restrict__ bary = pr.bary;
    const int levels = pr.levels, shift = pr.shift;
    const double *__restrict__ ct = pr.cdf + (size_t)t * F;
    for (int i = i0 + (int)threadIdx.x; i < i1; i += THREADS) {
        const size_t o = (size_t)t * N + i;
        Words4 w;
        if (uniforms) {
            const uint4 u = reinterpret_cast<const uint4 *>(uniforms)[o];
            w.w0 = u.x;
            w.w1 = u.y;
            w.w2 = u.z;
            w.w3 = u.w;
        } else {
            w = philox_words(pr.seed, (uint32_t)t, (uint32_t)i);
        }
        // inverse CDF: first k with C_k > r * S
        const uint64_t bits = (((uint64_t)w.w1 << 32) | (uint64_t)w.w0) >> 11;
        const double r = (double)bits * 0x1p-53;
        const double target = r * total;
        int h = 1;
        for (int l = 0; l < levels; ++l) h = 2 * h + (pivot[h] > target ? 0 : 1);
        // the pivots at or below the target are the sums that end whole blocks of 2^shift faces
        int lo = (h - (1 << levels)) << shift;
        for (int l = shift - 1; l >= 0; --l) {
            const int mid = lo + (1 << l) - 1;
            if (mid < F && !(ct[mid] > target)) lo = mid + 1;
        }
        const int f = (lo < F) ? lo : lp;
        // barycentric point, Eq. 3, with the square-root weights
        const float r1 = (float)(w.w2 >> 8) * 0x1p-24f;
        const float r2 = (float)(w.w3 >> 8) * 0x1p-24f;
        const float s = __builtin_sqrtf(r1);
        const float bu = 1.0f - s;
        const float bv = s * (1.0f - r2);
        const float bw = s * r2;
        const int32_t *fv = faces + 3 * (size_t)f;
        const float *p1 = corners + 3 * (size_t)fv[0];
        const float *p2 = corners + 3 * (size_t)fv[1];
        const float *p3 = corners + 3 * (size_t)fv[2];
        // the three corners are read whole (one 12-byte load each) before any store
        float c1[3], c2[3], c3[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            c1[k] = p1[k];
            c2[k] = p2[k];
            c3[k] = p3[k];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k)
            put<STREAM>(points + 3 * o + k,
                        __builtin_fmaf(bw, c3[k], __builtin_fmaf(bv, c2[k], bu * c1[k])));
        put<STREAM>(bary + 3 * o, bu);
        put<STREAM>(bary + 3 * o + 1, bv);
        put<STREAM>(bary + 3 * o + 2, bw);
        put<STREAM>(face_idx + o, f);
    }
}

// a degenerate frame or bad faces: reported through the status word
template <int THREADS>
__device__ __forceinline__ void no_points(const SampleParams &pr, int t, int i0, int i1) {
    const float nan = __builtin_nanf("");
    for (int i = i0 + (int)threadIdx.x; i < i1; i += THREADS) {
        const size_t o = (size_t)t * pr.N + i;
        pr.points[3 * o] = nan;
        pr.points[3 * o + 1] = nan;
        pr.points[3 * o + 2] = nan;
        pr.bary[3 * o] = 0.f;
        pr.bary[3 * o + 1] = 0.f;
        pr.bary[3 * o + 2] = 0.f;
        pr.face_idx[o] = -1;
    }
}

// The sums that end the blocks of 2^shift faces, as a tree: node h of level l holds the rank that
// splits its share of the 2^levels - 1 ranks; ranks past the last whole block are infinite.
template <int THREADS>
__device__ __forceinline__ void load_pivots(double *pivot, const double *ct, int F, int levels,
                                            int shift) {
    for (int h = (int)threadIdx.x + 1; h < (1 << levels); h += THREADS) {
        const int l = 31 - __clz(h);
        const int rank = ((2 * (h - (1 << l)) + 1) << (levels - 1 - l)) - 1;
        const int k = ((rank + 1) << shift) - 1;
        pivot[h] = k < F ? ct[k] : __builtin_inf();
    }
}

__device__ __forceinline__ void sample_body(const SampleParams &pr, const Blk &blk) {
    __shared__ double pivot[1 << SP_LEVELS];
    const int t = blk.y;
    const int first = blk.x * pr.chunk, end = min(pr.N, first + pr.chunk);
    const int lp = pr.lastpos[t];
    if (lp < 0) {
        no_points<SP_THREADS>(pr, t, first, end);
        return;
    }
    const double *ct = pr.cdf + (size_t)t * pr.F;
    load_pivots<SP_THREADS>(pivot, ct, pr.F, pr.levels, pr.shift);
    const double total = ct[pr.F - 1];
    __syncthreads();
    sample_points<SP_THREADS, false>(pr, t, first, end, lp, pivot, total, pr.verts + (size_t)t * pr.V * 3);
}

__device__ __forceinline__ void sample_wide_body(const SampleParams &pr, const Blk &blk) {
    __shared__ __align__(16) char lds[SW_BYTES];
    double *pivot = reinterpret_cast<double *>(lds);
    float *corners = reinterpret_cast<float *>(lds + ((size_t)8 << pr.levels));
    const size_t all = (size_t)pr.T * pr.N;
    size_t pos = (size_t)blk.x * pr.chunk;
    const size_t end = min(all, pos + pr.chunk);
    while (pos < end) {
        const int t = (int)(pos / pr.N);
        const int i0 = (int)(pos - (size_t)t * pr.N);
        const int i1 = (int)min((size_t)pr.N, end - (size_t)t * pr.N);
        pos += i1 - i0;
        const int lp = uniform_int(pr.lastpos + t);
        if (lp < 0) {
            no_points<SW_THREADS>(pr, t, i0, i1);
            continue;
        }
        const double *ct = pr.cdf + (size_t)t * pr.F;
        const float *vt = pr.verts + (size_t)t * pr.V * 3;
        load_pivots<SW_THREADS>(pivot, ct, pr.F, pr.levels, pr.shift);
#pragma unroll 4
        for (int k = threadIdx.x; k < 3 * pr.V; k += SW_THREADS) corners[k] = vt[k];
        const double total = ct[pr.F - 1];
        __syncthreads();
        sample_points<SW_THREADS, true>(pr, t, i0, i1, lp, pivot, total, corners);
        __syncthreads();  // the next frame takes the place of this one
    }
}

__global__ __launch_bounds__(SP_THREADS) void k_sample(SampleParams p) {
    sample_body(p, grid_blk_xcd());
}

__global__ __launch_bounds__(SW_THREADS) void k_sample_wide(SampleParams p) {
    sample_wide_body(p, grid_blk_xcd());
}

// blocks of faces as small as 2^levels - 1 pivots allow
void plan_pivots(SampleParams &p, int most) {
    p.levels = 1;
    while (p.levels < most && (1 << p.levels) <= p.F) ++p.levels;
    p.shift = 0;
    while ((p.F >> p.shift) >= (1 << p.levels)) ++p.shift;
}

}  // namespace

size_t sample_scratch_bytes(int T, int F) {
    return Arena::need((size_t)T * F, sizeof(double)) + Arena::need((size_t)T, sizeof(int32_t));
}

void launch_area_cdf(const float *verts, const int32_t *faces, int T, int V, int F,
                     const uint8_t *mask, int mask_per_frame, double *cdf, int32_t *lastpos,
                     unsigned *status, hipStream_t s) {
    AreaCdfParams ap;
    ap.verts = verts;
    ap.faces = faces;
    ap.mask = mask;
    ap.mask_stride = mask_per_frame ? (size_t)F : 0;
    ap.V = V;
    ap.F = F;
    ap.cdf = cdf;
    ap.lastpos = lastpos;
    ap.status = status;
    if (F <= AC_SMALL && !g_record)
        dispatch(KT_AREA_CDF, k_area_cdf<AC_SMALL, 1>, dim3(T), AC_SMALL, ap, s);
    else
        dispatch(KT_AREA_CDF, k_area_cdf<AC_THREADS, AC_PER>, dim3(T), AC_THREADS, ap, s);
}

void launch_sample(const float *verts, const int32_t *faces, int T, int V, int F, int N,
                   uint64_t seed, const uint32_t *uniforms, const uint8_t *mask, int mask_per_frame,
                   float *points, int32_t *face_idx, float *bary, double *cdf_scratch,
                   int32_t *lastpos_scratch, unsigned *status, hipStream_t s) {
    launch_area_cdf(verts, faces, T, V, F, mask, mask_per_frame, cdf_scratch, lastpos_scratch,
                    status, s);
    SampleParams sp;
    sp.verts = verts;
    sp.faces = faces;
    sp.V = V;
    sp.F = F;
    sp.N = N;
    sp.seed = seed;
    sp.uniforms = uniforms;
    sp.cdf = cdf_scratch;
    sp.lastpos = lastpos_scratch;
    sp.points = points;
    sp.face_idx = face_idx;
    sp.bary = bary;
    sp.T = T;
    // The wide kernel where its workgroups have a few thousand points each to load a frame for:
    // sampling 24 x 32,768 points takes 82 us with it against 95, 17 x 30,011 (half a million) 37.1
    // against 37.9, and one frame of 65,536 61.1 against 59.8 (sums of areas included).
    const size_t all = (size_t)T * N;
    const size_t corners = (size_t)V * 12;
    if (all >= size_t(1) << 19 && N >= 8192 && corners + (size_t(8) << 10) <= SW_BYTES) {
        const size_t share = (all + SW_CUS - 1) / SW_CUS;
        sp.chunk = (int)std::min((share + SW_THREADS - 1) / SW_THREADS * SW_THREADS,
                                 size_t(1) << 24);
        int most = 10;
        while (most < SW_LEVELS && corners + (size_t(16) << most) <= SW_BYTES &&
               (1 << most) < sp.chunk)
            ++most;
        plan_pivots(sp, most);
        dispatch(KT_SAMPLE_WIDE, k_sample_wide, dim3((unsigned)((all + sp.chunk - 1) / sp.chunk)),
                 SW_THREADS, sp, s);
        return;
    }
    plan_pivots(sp, SP_LEVELS);
    sp.chunk = SP_CHUNK;
    while (sp.chunk > SP_THREADS && (size_t)T * ((N + sp.chunk - 1) / sp.chunk) < SP_FILL)
        sp.chunk /= 2;
    dispatch(KT_SAMPLE, k_sample, dim3((N + sp.chunk - 1) / sp.chunk, T), SP_THREADS, sp, s);
}

void register_sample_kernels(BatchedKernel *table) {
    table[KT_AREA_CDF] =
        batched_kernel<AreaCdfParams, area_cdf_body<AC_THREADS, AC_PER>, AC_THREADS, 512>();
    table[KT_SAMPLE] = batched_kernel<SampleParams, sample_body, SP_THREADS, 1024>();
    table[KT_SAMPLE_WIDE] = batched_kernel<SampleParams, sample_wide_body, SW_THREADS, 256>();
}

}  // namespace dc

// The sample points of one tile of a gridding grid, found and binned for the matrix units.
//
// The type-1 spread (spread.hip) and the type-2 gather (project.hip) walk the periodic grid in
// tiles of T0 x T1 x T2 window starts.  A point of view m at the disk position (k1, k2) lies at
// t = s (k1 c1_m + k2 c2_m) relative to the grid's centre; along axis d its window covers the W
// cells from floor(tau - W/2) + 1, tau = t_d + L/2, and the tile that owns this start (shifted by
// PADLO so that it is never negative) owns the point.
//
// Why bins: the contribution of a point is an outer product w0 x w1 x w2, so the sum over points
// whose windows start in the same small box is a matrix product with the points as its inner
// dimension.  A bin of B0 x B1 x B2 starts has a footprint of 16 x CJ x 8 cells, which a wavefront
// holds as NJ accumulators of v_mfma_f32_16x16x4_f32 (rows: axis 0; columns: CJ/NJ = 2 rows of axis
// 1 and 8 cells of axis 2).  At W = 7 a bin is 10 x 2 x 2 and a third of the multiplies fall on
// cells of the point's window; one 64-bit LDS atomic per cell and point, as the accumulation was
// before, ran at a seventh of that.
//
// A workgroup (one per CU, 16 wavefronts) takes items of the work list (a tile and a range of views)
// and works on each by queuefuls:
//  1. find: each wavefront takes runs of 64 views (sorted by their normals; runs whose box of
//     normals misses the tile are skipped), keeps the views whose plane meets the tile's box on the
//     half-disk's side, and enumerates their rows k1, one (view, row) per lane: the k2 interval
//     whose points lie in the box, from three slabs in FP32, widened by a margin.  The intervals'
//     points go to an LDS queue, placed by a scan over the wavefront and one atomic.  No barrier.
//  2. when the queue is full: every entry is located exactly (FP64; entries in the margin outside
//     the tile are dropped), its value is formed, and the entries are sorted by bin in LDS.
//  3. the wavefronts take chunks of up to CHUNK points of one bin each, 16 points at a time; those that
//     find none left go on to find points.
// What bounds it, at N = 256 with 10^5 views (the kernel's spread, 2.6e9 points, 133 of 141 ms): issue slots of
// the vector unit, which FP32 matrix instructions take too (a probe of both in different wavefronts ran hardly
// faster than one after the other).  Time saved by leaving one part out, in copies: matrix products 36 ms,
// window weights 29, products' operands 21, adds to the tile 20, finding and locating points about 45; they
// overlap in part, so their sum is more than the whole.  Before, with one 64-bit LDS atomic per cell and
// point, 393 ms.
#pragma once

#include <algorithm>
#include <iterator>

#include "firm_internal.h"

namespace pts {

constexpr int NTH = 1024, NW = NTH / 64;
constexpr int GROUP = 32768;  // views per group: a queue entry holds 15 bits of view, 8 of k1, 9 of k2
constexpr int RUN = SP_VRUN;  // views per run (with one box of normals)
constexpr int SURV = 96;      // surviving views that a wavefront collects before it enumerates rows
constexpr int LDS_MAX = 160 * 1024 - 640;  // 640 bytes are the kernels' own (the disk's row starts)

typedef float f4 __attribute__((ext_vector_type(4)));

struct Args {
    int N, L, nt1, nt2;   // tiles along axes 1 and 2
    const double* c12;    // M x 6, in the gridding's view order, as the arrays below
    const float4* vrec;   // M x 2: (c1, c2x), (c2y, c2z, group, view index of the caller)
    const float4* rbox;   // per run of RUN views: (min normal, 0), (max normal, 0)
    const int4* work;     // (tile, first view, end view, 0)
    int nwork;
    int* taken;           // items handed out so far (0 at the launch)
    int batch;            // items that a workgroup is handed at a time, a power of 2
    float sym[4 * (KB_DEG + 1)];  // window polynomials, even and odd parts (see weights); by value, so that the
                          // coefficients come from scalar registers
};

// Geometry of the tiles of window width W.  NB0: bins along axis 0; P1MAX: bound on the padded extent
// of axis 1; RP: pitch of a tile row in cells, 4 RP = 8 (mod 16), so that the two rows of 8 cells,
// four rows apart, that the lanes of one quarter of an 8-byte access hit at W <= 7 share no bank;
// CELL: bytes per cell of the kernel's LDS tile; NV: floats of a queued value, or of a result (GATHER_).
template <int W_, int S_, int NB0_, int P1MAX, int RP_, int CELL, int NV_, bool GATHER_ = false>
struct Tile {
    static constexpr int W = W_, S = S_, RP = RP_, NV = NV_;  // S: grid cells per lattice step
    static constexpr bool GATHER = GATHER_;
    static constexpr int NJ = W == 8 ? 8 : 4, CJ = 2 * NJ;
    static constexpr int CHUNK = W == 8 ? 32 : 64;  // points of one bin that a wavefront takes at a time
    static constexpr int B0 = 17 - W, B1 = CJ + 1 - W, B2 = 9 - W;
    static constexpr int NB0 = NB0_, NB1 = (P1MAX - W + 1) / B1, NB2 = (RP - W + 1) / B2, NB = NB0 * NB1 * NB2;
    static constexpr int T0 = NB0 * B0, T1 = NB1 * B1, T2 = NB2 * B2;
    static constexpr int P0 = T0 + W - 1, P1 = T1 + W - 1, P2 = T2 + W - 1;
    static constexpr int CELLS = P0 * P1 * RP;
    static constexpr int PADLO = (W + 1) / 2 - 1;
    // A wavefront's 16 staged points.  Axis 0: the W weights of point p at LEAD + p S0, zeros up to
    // the next point's, so that the weight at row i of the bin's footprint, i - o0 cells into the
    // window, is read at that distance from the first without a test.  Axes 1 and 2: rows padded to
    // the footprint; then the value and -4 o0, (v0, -4 o0, v1, 0).
    static constexpr int S0 = 20, LEAD = 12, SB = CJ + 12, OFFV = CJ + 8;
    static constexpr int WAVE = LEAD + 16 * S0 + 16 * SB;
    static_assert(B0 - 1 <= LEAD && S0 - (B0 - 1) >= 8 && S0 >= 16, "zeros on both sides of the window");
    static constexpr int LDS_FIXED = CELLS * CELL + NW * WAVE * 4 + NW * SURV * 2 + (GROUP / RUN) * 2 + NB * 4 + 64;
    static constexpr int lds_of(int q) { return LDS_FIXED + q * (20 + 4 * NV) + (q / CHUNK + NB) * 4; }
    static constexpr int queue_cap() {
        int q = 4096;
        while (q > 1024 && lds_of(q) > LDS_MAX) q -= 256;
        return q;
    }
    static constexpr int QCAP = queue_cap(), EPT = (QCAP + NTH - 1) / NTH, NCT = QCAP / CHUNK + NB;
    static_assert(lds_of(QCAP) <= LDS_MAX, "LDS of one workgroup");
    static_assert(NB1 >= 1 && NB2 >= 1 && P1 <= P1MAX && P2 <= RP && NB <= 192, "tile");
    // half extents of the tile's box and the most rows and row points that it can hold
    static constexpr float H0 = 0.5f * T0, H1 = 0.5f * T1, H2 = 0.5f * T2;
    static constexpr int isqrt_up(int v) { int r = 0; while (r * r < v) ++r; return r; }
    static constexpr int DIAG = isqrt_up(T0 * T0 + T1 * T1 + T2 * T2);
    static constexpr int ROWS = DIAG / S + 1, CMAX = DIAG / S + 2;
    static_assert(64 * CMAX <= QCAP, "one step of a wavefront fits the queue");
};

template <class T>
struct Lds {
    int queue[T::QCAP];           // found points, in the order found
    float f[3 + T::NV][T::QCAP];  // their offsets f of the first cells along axes 0, 1, 2 and their values
    unsigned short off[T::QCAP];  // their starts in the bin, 4 bits per axis
    unsigned short order[T::QCAP];  // the points by bin
    alignas(16) float wave[NW][T::WAVE];
    int ctab[T::NCT];
    int hist[T::NB];
    unsigned short surv[NW][SURV];
    unsigned short live[GROUP / RUN];
    int qn, qfail, nlive, next, ndone, nchunk, cctr, any, item;
};

// Orders a wavefront's own LDS writes before its other lanes' reads.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int CTRL, int ROWMASK>
__device__ __forceinline__ int dpp_add(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWMASK, 0xf, false);
}
// inclusive scan over the 64 lanes: shifts within rows of 16, then row broadcasts
__device__ __forceinline__ int wave_scan(int v) {
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    return dpp_add<0x143, 0xc>(v);
}

__device__ __forceinline__ float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Fine-grid position of a point along one axis: the one expression from which every stage takes the
// window start, so that they agree to the last bit.  |t| <= L/2 in exact arithmetic; the clamp
// takes the rounding excess.
__device__ __forceinline__ double left_of(int s, int W, int k1, int k2, double ca, double cb, int L) {
    const double tau = fma((double)s, fma((double)k2, cb, (double)k1 * ca), 0.5 * L);
    return fmin(fmax(tau, 0.0), (double)L) - 0.5 * W;
}

// The W window weights at the offset f in (0, 1] of the first cell, x = 2 f - 1.  The window is even,
// so cells j and W-1-j share their polynomials: w_j(x) = E_j(x^2) + x O_j(x^2), w_{W-1-j} = E - x O.
// sym holds per pair the 6 even and then the 5 odd coefficients.
template <int W>
__device__ __forceinline__ void weights(const float (&sym)[4 * (KB_DEG + 1)], float x, float* w) {
    const float y = x * x;
#pragma unroll
    for (int j = 0; j < (W + 1) / 2; ++j) {
        const float* c = sym + (KB_DEG + 1) * j;
        float e = c[KB_EVEN - 1], o = c[KB_DEG];
#pragma unroll
        for (int d = KB_EVEN - 2; d >= 0; --d) e = fmaf(e, y, c[d]);
        if (2 * j + 1 == W) {
            w[j] = e;
        } else {
#pragma unroll
            for (int d = KB_DEG - KB_EVEN - 1; d >= 0; --d) o = fmaf(o, y, c[KB_EVEN + d]);
            w[j] = fmaf(o, x, e);
            w[W - 1 - j] = fmaf(-o, x, e);
        }
    }
}

__device__ __forceinline__ int entry_view(int e) { return (int)((unsigned)e >> 17); }
__device__ __forceinline__ int entry_k1(int e) { return (e >> 9) & 255; }
__device__ __forceinline__ int entry_k2(int e) { return (e & 511) - 256; }

// Sixteen points of a chunk (a round of a wavefront), four lanes per point: lanes 0, 1, 2 take the
// window's offset along axes 0, 1, 2, lane 3 the value.  Points past the chunk's end repeat its last
// one with the value zero.
template <class T>
struct Point {
    float f, v1;
    int off;
};
template <class T>
__device__ __forceinline__ Point<T> load_point(const Lds<T>& s, int at, int cnt) {
    const int lane = threadIdx.x & 63, p = lane >> 2;
    const int i = s.order[at + min(p, cnt - 1)];
    const bool zero = (lane & 3) == 3 && p >= cnt;
    Point<T> x;
    const float f = (&s.f[0][0])[(lane & 3) * T::QCAP + i];
    x.f = zero ? 0.f : f;
    x.v1 = 0.f;
    if constexpr (T::NV == 2) {
        const float v = s.f[4][i];
        x.v1 = zero ? 0.f : v;
    }
    x.off = s.off[i];
    return x;
}

// Stages a round: the window weights of axes 1 and 2 shifted to the bin's footprint.
template <class T>
__device__ __forceinline__ void stage(const Args& a, const Point<T>& x, float* __restrict__ wave) {
    constexpr int W = T::W, NF = T::CJ > 8 ? 16 : 8;
    const int lane = threadIdx.x & 63, p = lane >> 2, d = lane & 3;
    float w[NF];
    weights<W>(a.sym, 2.f * x.f - 1.f, w);
#pragma unroll
    for (int j = W; j < NF; ++j) w[j] = 0.f;
    // shift the weights up by the start in the bin, one binary digit at a time
    const int sh = (x.off >> (4 * d)) & (d == 1 || d == 2 ? 15 : 0);
#pragma unroll
    for (int b = 1; b < (T::B1 > T::B2 ? T::B1 : T::B2); b <<= 1) {
        const bool on = (sh & b) != 0;
#pragma unroll
        for (int j = NF - 1; j >= 0; --j) w[j] = on ? (j >= b ? w[j - b] : 0.f) : w[j];
    }
    const bool val = d == 3;
    float* q = wave + (d == 0 ? T::LEAD + p * T::S0 : T::LEAD + 16 * T::S0 + p * T::SB + (d == 1 ? 0 : (d == 2 ? T::CJ : T::OFFV)));
    *reinterpret_cast<f4*>(q) = f4{val ? x.f : w[0], val ? __int_as_float(-4 * (x.off & 15)) : w[1], val ? x.v1 : w[2], w[3]};
    if (!val) *reinterpret_cast<f4*>(q + 4) = f4{w[4], w[5], w[6], w[7]};
    if constexpr (T::CJ > 8) {
        if (d == 1) {
            *reinterpret_cast<f4*>(q + 8) = f4{w[8], w[9], w[10], w[11]};
            *reinterpret_cast<f4*>(q + 12) = f4{w[12], w[13], w[14], w[15]};
        }
    }
    wave_sync();
}

// The workgroups (one per CU) take the items of the work list one at a time, heavy ones first: with a
// workgroup per item, the fixed assignment of workgroups to the eight XCDs left CUs idle for a fifth
// of the time.  Thread 0 holds the next item one ahead; `item(work)` runs for each.
template <class T, class F>
__device__ __forceinline__ void for_items(const Args& a, Lds<T>& s, F&& item) {
    float* const wave = s.wave[threadIdx.x >> 6];
    for (int i = threadIdx.x & 63; i < T::WAVE; i += 64) wave[i] = 0.f;
    int next = 0;
    if (threadIdx.x == 0) next = atomicAdd(a.taken, a.batch);
    while (true) {
        if (threadIdx.x == 0) s.item = next;
        __syncthreads();
        const int i = s.item;
        if (i >= a.nwork) return;
        if (threadIdx.x == 0 && (++next & (a.batch - 1)) == 0) next = atomicAdd(a.taken, a.batch);
        item(a.work[i]);
        __syncthreads();
    }
}

// Runs over the points of the tile whose first window starts (in the shifted count) are t0, t1, t2.
// Per queueful, `fetch(view, k1, k2)` loads what an entry's value needs and `value(loaded, k1, k2, v)`
// forms it; then the wavefronts take chunks of one bin's points: `state = open(bin)`, per round of 16
// staged points `round(state, points, position)`, `close(state, bin)`.  `begin()` runs once, by all threads, before the
// first queueful.  A gather has no values (NV = 2 floats hold a point's result, which `round` stores at
// order[position]): when every chunk of a queueful is done, `finish(first view, entries, places)` takes
// each thread's entries, entry j at tid + j NTH (place -1: none).
template <class T, class FB, class FL, class FV, class FO, class FR, class FC, class FF>
__device__ __forceinline__ void for_points(const Args& a, Lds<T>& s, int4 wk, int t0, int t1, int t2, FB&& begin,
                                           FL&& fetch, FV&& value, FO&& open, FR&& round, FC&& close, FF&& finish) {
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    float* const wave = s.wave[wv];
    // the box of the tile's positions, relative to the grid's centre: starts are floor(tau + HW)
    constexpr float HW = (T::W & 1) ? 0.5f : 0.f;
    const float off = -HW - 0.5f * a.L;
    const float c0 = uniform(t0 + T::H0 + off), c1 = uniform(t1 + T::H1 + off), c2 = uniform(t2 + T::H2 + off);
    const float s0 = uniform(c0 / T::S), s1 = uniform(c1 / T::S), s2 = uniform(c2 / T::S);  // in lattice steps
    const int N = a.N;
    if (tid == 0) {
        s.qn = 0; s.qfail = T::QCAP; s.nlive = 0; s.next = 0; s.ndone = 0; s.cctr = 0; s.any = 0;
    }
    for (int b = tid; b < T::NB; b += NTH) s.hist[b] = 0;
    __syncthreads();
    for (int g0 = wk.y; g0 < wk.z; g0 += GROUP) {
        const int gend = min(wk.z, g0 + GROUP);
        // runs whose box of normals n allows |n . c| within the box's half extent along some n
        for (int r = tid; r * RUN < gend - g0; r += NTH) {
            const float4 lo = a.rbox[2 * (g0 / RUN + r)], hi = a.rbox[2 * (g0 / RUN + r) + 1];
            const float p0 = c0 * lo.x, q0 = c0 * hi.x, p1 = c1 * lo.y, q1 = c1 * hi.y, p2 = c2 * lo.z, q2 = c2 * hi.z;
            const float dmin = fminf(p0, q0) + fminf(p1, q1) + fminf(p2, q2);
            const float dmax = fmaxf(p0, q0) + fmaxf(p1, q1) + fmaxf(p2, q2);
            const float lim = T::H0 * fmaxf(fabsf(lo.x), fabsf(hi.x)) + T::H1 * fmaxf(fabsf(lo.y), fabsf(hi.y)) +
                              T::H2 * fmaxf(fabsf(lo.z), fabsf(hi.z)) + 4e-3f;
            if (dmin <= lim && dmax >= -lim) s.live[atomicAdd(&s.nlive, 1)] = (unsigned short)r;
        }
        __syncthreads();
        // A gather with fewer live runs than wavefronts hands out each run in 2^sh parts of 64 >> sh views, one at
        // a time: with few views it waits for the one wavefront that finds their points (30 views at N = 16
        // 49.2 -> 45.4 us).  Not the spreads: their many sparse tiles pay for the idle lanes (Ker at
        // N = 128 with 30 views 1,156 -> 1,178 us).
        int sh = 0, parts = 0;  // the spreads read the runs' count where it is needed (0.3% of Ker's time)
        if constexpr (T::GATHER) {
            parts = __builtin_amdgcn_readfirstlane(s.nlive);
            while (parts < NW && sh < 4) {
                parts <<= 1;
                ++sh;
            }
        }
        int ent[T::EPT], place[T::EPT];  // the thread's entries of the queueful and their sorted positions
        bool held = false;               // a queueful whose results have not been taken
        int n = 0, ub = 0;  // surviving views collected by the wavefront, first (view, row) not yet queued
        bool counted = false;
        while (true) {
            bool full = false;
            while (!full) {
                if (ub >= n * T::ROWS) {
                    // runs until enough views survive to fill the steps below
                    n = 0;
                    ub = 0;
                    while (sh ? n == 0 : n <= SURV - RUN) {
                        int li = 0;
                        if (lane == 0) li = atomicAdd(&s.next, 1);
                        li = __builtin_amdgcn_readfirstlane(li);
                        if (li >= (T::GATHER ? parts : s.nlive)) break;
                        const int rel = (int)s.live[li >> sh] * RUN + lane;
                        const int64_t m = min(g0 + rel, gend - 1);
                        const float4 ra = a.vrec[2 * m], rb = a.vrec[2 * m + 1];
                        // the plane meets the box, and does so where k1 >= 0 (s k1 is the coordinate along c1)
                        const float nx = ra.y * rb.y - ra.z * rb.x, ny = ra.z * ra.w - ra.x * rb.y, nz = ra.x * rb.x - ra.y * ra.w;
                        const bool ok = g0 + rel < gend && ((lane << sh) >> 6) == (li & ((1 << sh) - 1)) &&
                                        fabsf(c0 * nx + c1 * ny + c2 * nz) <=
                                            T::H0 * fabsf(nx) + T::H1 * fabsf(ny) + T::H2 * fabsf(nz) + 2e-3f &&
                                        c0 * ra.x + c1 * ra.y + c2 * ra.z + T::H0 * fabsf(ra.x) + T::H1 * fabsf(ra.y) +
                                                T::H2 * fabsf(ra.z) >= -2e-3f;
                        const unsigned long long mask = __ballot(ok);
                        if (ok) s.surv[wv][n + __popcll(mask & ((1ull << lane) - 1))] = (unsigned short)rel;
                        n += __popcll(mask);
                    }
                    wave_sync();
                    if (n == 0) break;
                }
                // one (view, row k1) per lane: the k2 interval of the row's points in the box, all in
                // lattice steps; rows past the end repeat the last view and hold no point
                const int un = ub + lane, v = (int)(((float)un + 0.5f) * (1.f / T::ROWS));
                const int rel = s.surv[wv][min(v, n - 1)];
                const float4 ra = a.vrec[2 * (int64_t)(g0 + rel)], rb = a.vrec[2 * (int64_t)(g0 + rel) + 1];
                const float3 u = make_float3(ra.x, ra.y, ra.z), w = make_float3(ra.w, rb.x, rb.y);
                const float uc = s0 * u.x + s1 * u.y + s2 * u.z;
                const float uh = (T::H0 / T::S) * fabsf(u.x) + (T::H1 / T::S) * fabsf(u.y) + (T::H2 / T::S) * fabsf(u.z) + 1e-3f;
                const int k1 = (int)ceilf(uc - uh) + (un - v * T::ROWS);
                const float fk = (float)k1;
                const int left = N * N / 4 - k1 * k1;
                int kd = (int)__builtin_amdgcn_sqrtf((float)max(left, 0));  // the disk's largest |k2| on the row
                kd += (kd + 1) * (kd + 1) <= left ? 1 : 0;
                kd -= kd * kd > left ? 1 : 0;
                float lo = k1 == 0 ? 1.f : (float)-kd, hi = (float)kd;
                // |al + k2 be| <= h per axis.  A slope below 1e-6 counts as 1e-6 (the points move by less than
                // 2e-4 steps, the margin is 2.5e-3 and more); the reciprocal is good to about 1 ulp, far inside it.
                auto slab = [&](float cc, float h, float ca, float cb) {
                    const float al = fmaf(fk, ca, -cc);
                    const float rb = __builtin_amdgcn_rcpf(copysignf(fmaxf(fabsf(cb), 1e-6f), cb));
                    const float mid = -al * rb, half = h * fabsf(rb);
                    lo = fmaxf(lo, mid - half);
                    hi = fminf(hi, mid + half);
                };
                slab(s0, (T::H0 + 1e-2f) / T::S, u.x, w.x);
                slab(s1, (T::H1 + 1e-2f) / T::S, u.y, w.y);
                slab(s2, (T::H2 + 1e-2f) / T::S, u.z, w.z);
                const bool row = v < n && k1 >= 0 && left >= 0 && fk <= uc + uh;
                const int klo = (int)ceilf(lo);
                const int cnt = row ? min(max((int)floorf(hi) - klo + 1, 0), T::CMAX) : 0;
                const int incl = wave_scan(cnt);
                const int total = __builtin_amdgcn_readlane(incl, 63);
                if (total) {
                    int pos = 0;
                    if (lane == 0) pos = atomicAdd(&s.qn, total);
                    pos = __builtin_amdgcn_readfirstlane(pos);
                    if (pos + total > T::QCAP) {
                        // this step waits for the round; the queue holds what was placed before it
                        if (lane == 0) atomicMin(&s.qfail, pos);
                        full = true;
                        break;
                    }
                    int* q = s.queue + pos + incl - cnt;
                    const int e0 = (rel << 17) | (k1 << 9) | (klo + 256);
                    for (int j = 0; j < cnt; ++j) q[j] = e0 + j;
                }
                ub += 64;
            }
            if (!full && !counted) {
                counted = true;
                if (lane == 0) atomicAdd(&s.ndone, 1);
            }
            __syncthreads();
            const int nq = min(s.qn, s.qfail);
            const bool last = s.ndone == NW;
            if (T::GATHER && held) finish(g0, ent, place);
            held = nq > 0;
            if (nq > 0) {
                if (!s.any) begin();
                // exact place of every entry: its offsets, starts and value (by queue position), its bin and
                // its rank in the bin (place: bin << 16 | rank; -1: not a point of this tile).  A thread's
                // entries go one by one, the next one's loads issued before the current one is used: all of
                // their registers at once spill.
                struct Entry {
                    int e;
                    double c[6];
                    decltype(fetch(0, 0, 0)) raw;
                };
                auto load = [&](int j) {
                    Entry x;
                    x.e = s.queue[min(tid + j * NTH, nq - 1)];
                    const int m = g0 + entry_view(x.e);
#pragma unroll
                    for (int d = 0; d < 6; ++d) x.c[d] = a.c12[6 * (int64_t)m + d];
                    x.raw = fetch(m, entry_k1(x.e), entry_k2(x.e));
                    return x;
                };
                Entry cur = load(0);
#pragma unroll
                for (int j = 0; j < T::EPT; ++j) place[j] = -1;
#pragma unroll
                for (int j = 0; j < T::EPT; ++j) {
                    if (j * NTH + wv * 64 >= nq) break;  // nothing for this wavefront
                    const Entry y = cur;
                    if (j + 1 < T::EPT) cur = load(j + 1);
                    const int i = tid + j * NTH, k1 = entry_k1(y.e), k2 = entry_k2(y.e);
                    int x[3];
                    float f[3];
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        const double left = left_of(T::S, T::W, k1, k2, y.c[d], y.c[3 + d], a.L), fl = floor(left);
                        x[d] = (int)fl + 1 + T::PADLO - (d == 0 ? t0 : (d == 1 ? t1 : t2));
                        f[d] = (float)(fl + 1.0 - left);  // in (0, 1]
                    }
                    const unsigned b0 = T::NB0 == 1 ? 0u : (unsigned)x[0] / T::B0, b1 = (unsigned)x[1] / T::B1,
                                   b2 = (unsigned)x[2] / T::B2;
                    if (T::GATHER) ent[j] = y.e;
                    if (i < nq && (unsigned)x[0] < (unsigned)T::T0 && (unsigned)x[1] < (unsigned)T::T1 &&
                        (unsigned)x[2] < (unsigned)T::T2) {
                        const int bin = (int)((b0 * T::NB1 + b1) * T::NB2 + b2);
                        place[j] = (bin << 16) | atomicAdd(&s.hist[bin], 1);
#pragma unroll
                        for (int d = 0; d < 3; ++d) s.f[d][i] = f[d];
                        s.off[i] = (unsigned short)((x[0] - b0 * T::B0) | (x[1] - b1 * T::B1) << 4 | (x[2] - b2 * T::B2) << 8);
                        if constexpr (!T::GATHER) {
                            float val[2];
                            value(y.raw, k1, k2, val);
#pragma unroll
                            for (int d = 0; d < T::NV; ++d) s.f[3 + d][i] = val[d];
                        }
                    }
                }
                __syncthreads();
                if (wv == 0) {
                    // offsets of the bins (left in hist) and the table of chunks
                    int base = 0;  // points and chunks before, (chunks << 16) | points
#pragma unroll
                    for (int b0 = 0; b0 < T::NB; b0 += 64) {
                        const int b = b0 + lane;
                        const int h = b < T::NB ? s.hist[b] : 0;
                        const int x = (((h + T::CHUNK - 1) / T::CHUNK) << 16) | h;
                        const int incl = wave_scan(x) + base;
                        const int ex = incl - x;
                        int at = ex & 0xffff, ci = ex >> 16;
                        if (b < T::NB) s.hist[b] = at;
                        for (int rest = h; rest > 0; rest -= T::CHUNK, at += T::CHUNK, ++ci)
                            s.ctab[ci] = (b << 20) | (at << 7) | min(rest, T::CHUNK);
                        base = __builtin_amdgcn_readlane(incl, 63);
                    }
                    if (lane == 0) {
                        s.nchunk = base >> 16;
                        s.any = 1;
                        s.cctr = 0;
                        s.qn = 0;  // every entry has been read
                        s.qfail = T::QCAP;
                    }
                }
                __syncthreads();
#pragma unroll
                for (int j = 0; j < T::EPT; ++j)
                    if (place[j] >= 0)
                        s.order[s.hist[place[j] >> 16] + (place[j] & 0xffff)] = (unsigned short)(tid + j * NTH);
                __syncthreads();
                for (int b = tid; b < T::NB; b += NTH) s.hist[b] = 0;
                // the chunks, handed out one at a time, and no barrier after them: a wavefront that finds none
                // left goes on to find points; the loads of a wavefront's next round are issued
                // before the current round's products
                int at = 0, cnt = 0, bin = 0;
                auto next = [&]() {
                    int ci = 0;
                    if (lane == 0) ci = atomicAdd(&s.cctr, 1);
                    ci = __builtin_amdgcn_readfirstlane(ci);
                    if (ci >= s.nchunk) return false;
                    const int x = __builtin_amdgcn_readfirstlane(s.ctab[ci]);
                    at = (x >> 7) & 8191;
                    cnt = x & 127;
                    bin = x >> 20;
                    return true;
                };
                bool have = next();
                Point<T> x{};
                if (have) x = load_point<T>(s, at, cnt);
                while (have) {
                    // the chunk's registers live here only: held across the queueful they would spill
                    const int cbin = bin, cat = at, ccnt = cnt;
                    auto st = open(cbin);
                    for (int r0 = 0;; r0 += 16) {
                        stage<T>(a, x, wave);
                        const bool end = r0 + 16 >= ccnt;
                        if (!end) {
                            x = load_point<T>(s, cat + r0 + 16, ccnt - r0 - 16);
                        } else {
                            have = next();
                            if (have) x = load_point<T>(s, at, cnt);
                        }
                        round(st, ccnt - r0, cat + r0);
                        wave_sync();
                        if (end) break;
                    }
                    close(st, cbin);
                }
            }
            if (last) break;
        }
        __syncthreads();
        if (T::GATHER && held) finish(g0, ent, place);
        if (tid == 0) { s.nlive = 0; s.next = 0; s.ndone = 0; }
        __syncthreads();
    }
}

}  // namespace pts

inline pts::Args point_args(firm_plan p, int L, const int* work, int nwork) {
    pts::Args a{};
    a.N = p->N; a.L = L;
    a.c12 = p->c12s; a.vrec = p->vrec; a.rbox = p->rbox;
    std::copy(std::begin(p->kb_sym), std::end(p->kb_sym), a.sym);
    a.work = reinterpret_cast<const int4*>(work);
    a.nwork = nwork;
    a.taken = p->taken;
    // The counter answers one workgroup in 11 ns, which is longer than an item of a few views takes the chip:
    // with few views and a long list (Ker from N = 128 on, all at N = 256) it hands out four at a time.  Ker at
    // N = 256 with one view 7.65 -> 6.74 ms, with 100 views 11.0 -> 10.9; from 500 views on, or with fewer than 64
    // items a workgroup, the uneven end costs as much as that gains.
    a.batch = p->M <= 128 && nwork >= 64 * p->ncu ? 4 : 1;
    return a;
}

template <class T>
TileDims tile_dims() { return TileDims{T::T0, T::T1, T::T2}; }

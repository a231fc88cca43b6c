// Type-1 non-uniform FFT gridding of libfirm (section 3.4, steps 2 and 3).
//
// Ker (eq. kernel) and A*b (eq. backprojection) are sums over the sample points
// xi_{k,m} = R_m^{-1}(omega_k, 0).  In fine-grid units (grid size L = s N) the
// point is t = s (k1 c1_m + k2 c2_m), c1, c2 the first two columns of R_m^{-1}.
// Each point is spread with a separable Kaiser-Bessel window of width W onto a
// periodic grid; a grid FFT divided by the window's transform gives the sums.
//
// A workgroup owns one tile of window starts (or one tile and a range of views):
// points.h finds its points and sorts them into bins, and a wavefront sums a chunk
// of one bin's points as a matrix product on the matrix units: the chunk's 16 x CJ x 8
// cells are W0^T (points x 16 rows) times W1 W2 (points x CJ 8 columns), four points per
// instruction.  The chunk's FP32 sums (at most 64 terms) then go to the
// workgroup's LDS tile as 64-bit integers, one atomic per cell and chunk, where one
// per cell and point was needed without the matrix units; the tile is added to the
// global grid at the end with one atomic per nonzero cell, in FP32 or, where many
// ranges share a tile, as the 64-bit integers (sp_units_from).  Each point is spread
// exactly once.
//
// LDS float atomics run at a small fraction of the plain read/write rate on this
// chip, 64-bit integer atomics at about the plain rate.  The tile is therefore
// accumulated in fixed point: 64-bit integer cells in units of 1/fxs (a power of 2
// with |term| < 2^31).  Integer sums are exact and independent of the order of the
// adds.  Ker's terms are non-negative; A*b's are signed, both components in one pass
// over the points, with a unit that follows from the largest |component| of the data.
// Only the half disk (k1 > 0, or k1 = 0 and k2 > 0) is spread: its partner -k is
// folded in (Ker is real and even; for A*b the pair (k, -k) gives the real part
// exactly), and k = 0 is added afterwards in closed form.
//
// Measured against the spread with one atomic per cell and point (two launches for A*b): the kernel's
// precompute at N = 256 with 10^5 views 400 -> 141 ms, N = 64 with 10^4 views 2.48 -> 1.03 ms; A*b at
// N = 256 with 5 x 10^4 views 398 -> 100 ms.
// Errors against 64-bit sums, of that spread, of this one with every point summed into the integers by itself,
// and of this one: Ker N = 32 with 2 x 10^4 views 2.39, 1.90, 1.89e-7, N = 64 with 5,000 2.95, 2.85, 2.87e-7, there
// at W = 8 1.60, 1.53, 1.56e-7; A*b of slices of one volume N = 32 2.25, 1.55, 1.55e-7, W = 8 1.45, 1.24, 1.24e-7,
// N = 64 with 9,973 views 1.94, 1.48, 1.53e-7, W = 8 1.49, 1.27, 1.27e-7; A*b of white noise N = 32 9.31, 9.17,
// 9.17e-7.  What the FP32 sums of a chunk add is below 1% (N = 64 on an integer grid, Ker 2.855 against 2.851e-7,
// W = 8 1.535 against 1.530e-7), with views that repeat hundreds of times 5% (Ker at W = 8); the gain over the
// spread before is from the polynomials' even and odd parts and the deconvolution by their own transform.
#include <algorithm>
#include <cmath>
#include <vector>

#include "firm_internal.h"
#include "points.h"

namespace {

struct SpreadArgs {
    pts::Args p;
    const float* table;
    int Q;
    float* grid;
    unsigned long long* units;  // when set, the grid's sums as 64-bit integers in fixed-point units, instead of grid
    const float2* b;
    const double* shifts;
    const int* rowstart;  // index of (k1, 0) shifted: idx(k1, k2) = rowstart[k1 + N/2] + k2
    int P;
    float fxs;      // fixed-point accumulation: integer units per unit of grid value (a power of 2)
    double fx_inv;  // 1 / fxs
    // when set, fxs is the largest power of 2 not above fx_coef / bmax, bmax the float whose bits
    // are at fx_bmax (the largest |component| of the data), found on the device before the launch
    const unsigned* fx_bmax;
    float fx_coef;
};

// Tiles at W = 7: the kernel's 10 x 16 x 16 starts (62 KB of 64-bit cells, 64 bins, grid 4N); A*b's
// 10 x 8 x 12 with two components per cell (65 KB, 24 bins, grid 2N, where a view leaves four times
// the points in a tile).  The LDS left holds the queue, and a larger queue fills the bins' chunks:
// 20 x 16 x 16 for the kernel (half the queue per bin, fewer tiles) 180 -> 200 ms at N = 256 with
// 10^5 views, 10 x 8 x 16 (fewer points per view found) 180 -> 210 ms, 10 x 12 x 16 the same; A*b at
// 10 x 10 x 12 115 against 112 ms, 5 x 10^4 views.
template <int W, bool CPLX>
using SpreadTile = pts::Tile<W, (CPLX ? 2 : 4), 1, (CPLX ? (W == 8 ? 16 : 14) : 22), (CPLX ? 18 : 22), (CPLX ? 16 : 8), (CPLX ? 2 : 1)>;

// The integer nearest to x (|x| < 2^51), by the FP64 sum whose last place is one.
__device__ __forceinline__ unsigned long long to_units(float x) {
    return (unsigned long long)__double_as_longlong((double)x + 6755399441055744.0) - 0x4338000000000000ull;
}

// The fixed-point unit of a gridding: integer units per unit of grid value, and its reciprocal.
struct Unit {
    float fxs;
    double inv;
};
__device__ __forceinline__ Unit unit_of(const SpreadArgs& a) {
    if (!a.fx_bmax) return Unit{a.fxs, a.fx_inv};
    const float bm = __uint_as_float(*a.fx_bmax);
    int e = 0;
    if (bm > 0.f) e = (int)fmin(fmax(floor(log2((double)a.fx_coef / (double)bm)), -100.0), 100.0);
    return Unit{ldexpf(1.f, e), ldexp(1.0, -e)};
}

// A point's value in fixed-point units: every term stays below 2^31 for finite data.  NaN counts as
// zero, so that no other point of the bin is touched.  An infinity counts as 2^32 units; in A*b the unit
// then follows it (2^100), every finite point rounds to zero and the grid overflows: no voxel is finite.
__device__ __forceinline__ float bounded(float v) {
    return v == v ? fminf(fmaxf(v, -4294967296.f), 4294967296.f) : 0.f;
}

template <int W, bool CPLX>
__global__ void __launch_bounds__(pts::NTH, pts::NTH / 256) k_spread(SpreadArgs a) {
    using T = SpreadTile<W, CPLX>;
    constexpr int NC = CPLX ? 2 : 1, NJ = T::NJ;
    __shared__ unsigned long long tile[NC][T::CELLS];
    __shared__ pts::Lds<T> s;
    __shared__ int rowstart[CPLX ? 132 : 1];  // the disk's rows k1 >= 0 (N <= 256)

    const int tid = threadIdx.x, lane = tid & 63;
    const Unit unit = unit_of(a);
    const float fxs = unit.fxs;
    const double fx_inv = unit.inv;
    const int N = a.p.N;
    const double inv_n = 1.0 / N;
    if constexpr (CPLX)
        for (int i = tid; i <= N / 2; i += pts::NTH) rowstart[i] = a.rowstart[i + N / 2];

    auto begin = [&]() {
        for (int i = tid; i < NC * T::CELLS; i += pts::NTH) (&tile[0][0])[i] = 0ull;
    };
    struct Raw {
        float h;
        float2 bp, bm;
        double s1, s2;
    };
    auto fetch = [&](int m, int k1, int k2) {
        Raw x{};
        const float4 rec = a.p.vrec[2 * (int64_t)m + 1];
        const int g = __float_as_int(rec.z);
        if constexpr (CPLX) {
            const int64_t mo = (int64_t)__float_as_int(rec.w) * a.P;  // the caller's view
            const int idx = rowstart[k1] + k2;
            x.bp = a.b[mo + idx];
            x.bm = a.b[mo + (a.P - 1 - idx)];
            if (a.shifts) {
                x.s1 = a.shifts[2 * (int64_t)m];
                x.s2 = a.shifts[2 * (int64_t)m + 1];
            }
        }
        x.h = a.table ? a.table[(int64_t)g * a.Q + k1 * k1 + k2 * k2] : 1.f;
        return x;
    };
    auto value = [&](const Raw& x, int k1, int k2, float* v) {
        if constexpr (!CPLX) {
            v[0] = bounded(2.f * x.h * x.h * fxs);
        } else {
            // h exp(i theta) (b(k) + conj b(-k)), theta = 2 pi <k, s_m> / N (re-centring)
            const float sr = x.bp.x + x.bm.x, si = x.bp.y - x.bm.y;
            float cs = 1.f, sn = 0.f;
            if (a.shifts) {
                // theta / 2 pi reduced to [-1/2, 1/2] in FP64, then the FP32 sine and cosine of pi
                // times twice that (N is a power of 2: the product with 1 / N is the quotient)
                const double f = (k1 * x.s1 + k2 * x.s2) * inv_n;
                sincospif((float)(2.0 * (f - rint(f))), &sn, &cs);
            }
            v[0] = bounded(fxs * x.h * (cs * sr - sn * si));
            v[1] = bounded(fxs * x.h * (cs * si + sn * sr));
        }
    };
    // A lane's part of the 16 x CJ x 8 footprint: columns (axis 1, axis 2) = (NJ e + n, kk), rows
    // (axis 0) 4 q + r of accumulator register r; as an operand, point q of the four, row lane & 15.
    const int q = lane >> 4, e = (lane >> 3) & 1, kk = lane & 7;
    // A chunk's sums.  The kernel's terms are all positive, and a chain of roundings over 64 of them
    // raised its error at N = 64 from 2.6e-7 to 2.9e-7: at W <= 7 each round sums on its own (16 terms
    // in a chain) and is added to them (140.0 -> 141.5 ms at N = 256).  At W = 8, where the window's own error is
    // smallest and there are no registers for a second set, each round goes to the tile (EACH): with the
    // chunk's 32 terms in a chain, views that repeat (their terms round alike, again and again) raised Ker's error
    // from 1.53e-7 to 1.85e-7, now 1.61e-7 (N = 16, 20 views 300 times each), for 6 to 10% of the time (N = 64 with
    // 10^4 views Ker 1.51 -> 1.64 ms, A*b 2.43 -> 2.68).  A*b's chains of 64 at W <= 7 do not show in its error, not
    // where its terms add up in phase either (slices of one volume, N = 64: 1.471e-7 against 1.470e-7 with
    // chains of 16); one view repeated 6,000 times has 8.00e-7 against 7.87e-7.  Chains of 32 cost 4.4%, of 16 13%.
    constexpr bool EACH = W == 8;
    struct Sums {
        pts::f4 acc[EACH ? 1 : NC][EACH ? 1 : NJ];
        int bin;
    };
    auto open = [&](int bin) {
        Sums x{};
        x.bin = bin;
        return x;
    };
    // the sums of a bin's 16 x CJ x 8 cells to the tile
    auto add = [&](const pts::f4 (&acc)[NC][NJ], int bin) {
        const int o0 = bin / (T::NB1 * T::NB2) * T::B0, o1 = bin / T::NB2 % T::NB1 * T::B1, o2 = bin % T::NB2 * T::B2;
        const int cell = ((o0 + 4 * q) * T::P1 + o1 + NJ * e) * T::RP + o2 + kk;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int n = 0; n < NJ; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    __hip_atomic_fetch_add(&tile[c][cell + (r * T::P1 + n) * T::RP], to_units(acc[c][n][r]),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    const float* const wave = s.wave[tid >> 6];
    const float* const row0 = wave + T::LEAD + q * T::S0 + (lane & 15);
    const float* const rowb = wave + T::LEAD + 16 * T::S0 + q * T::SB;
    auto round = [&](Sums& x, int cnt, int) {
        // the operands of KB steps (four points each) are read together, then used
        constexpr int KB = NJ == 4 ? 4 : 1;
        constexpr bool APART = EACH || !CPLX;
        pts::f4 part[APART ? NC : 1][APART ? NJ : 1] = {};
        auto& acc = [&]() -> auto& {
            if constexpr (APART) return part;
            else return x.acc;
        }();
#pragma unroll
        for (int kb = 0; kb < 4; kb += KB) {
            float w0[KB], v0[KB], v1[KB], w2[KB], w1[KB][NJ];
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                const float* r = rowb + 4 * (kb + j) * T::SB;
                v0[j] = r[T::OFFV];
                v1[j] = CPLX ? r[T::OFFV + 2] : 0.f;
                const int o = __float_as_int(r[T::OFFV + 1]);
                w0[j] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row0 + 4 * (kb + j) * T::S0) + o);
                w2[j] = r[T::CJ + kk];
#pragma unroll
                for (int n = 0; n < NJ; n += 4) {
                    const pts::f4 v = *reinterpret_cast<const pts::f4*>(r + NJ * e + n);
                    w1[j][n] = v.x; w1[j][n + 1] = v.y; w1[j][n + 2] = v.z; w1[j][n + 3] = v.w;
                }
            }
            if constexpr (KB == 4) {  // all of the reads are issued before the first product waits for one
                asm volatile("" : "+v"(w0[0]), "+v"(w0[1]), "+v"(w0[2]), "+v"(w0[3]), "+v"(w2[0]), "+v"(w2[1]),
                             "+v"(w2[2]), "+v"(w2[3]));
            }
#pragma unroll
            for (int j = 0; j < KB; ++j) {
                if (4 * (kb + j) >= cnt) break;
                const float a0[2] = {w0[j] * v0[j], w0[j] * v1[j]};
#pragma unroll
                for (int n = 0; n < NJ; ++n) {
                    const float w12 = w1[j][n] * w2[j];
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        acc[c][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[c], w12, acc[c][n], 0, 0, 0);
                }
            }
        }
        if constexpr (EACH) {
            add(part, x.bin);
        } else if constexpr (APART) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int n = 0; n < NJ; ++n) x.acc[c][n] += part[c][n];
        }
    };
    auto close = [&](const Sums& x, int bin) {
        if constexpr (!EACH) add(x.acc, bin);
    };
    const int L = a.p.L;
    pts::for_items<T>(a.p, s, [&](int4 wk) {
        const int nt12 = a.p.nt1 * a.p.nt2;
        const int t0 = wk.x / nt12 * T::T0, t1 = wk.x / a.p.nt2 % a.p.nt1 * T::T1, t2 = wk.x % a.p.nt2 * T::T2;
        pts::for_points<T>(a.p, s, wk, t0, t1, t2, begin, fetch, value, open, round, close, [](int, int*, int*) {});
        if (!s.any) return;
        // the tile's sums to the grid, as integers or rounded once to FP32
        auto flush = [&](auto&& to_grid) {
            for (int i = tid; i < T::P0 * T::P1 * T::P2; i += pts::NTH) {
                const int l0 = i / (T::P1 * T::P2), l1 = i / T::P2 % T::P1, l2 = i % T::P2;
                const int li = (l0 * T::P1 + l1) * T::RP + l2;
                // grid index = position mod L (a power of 2), position = cell - L/2
                const int g0 = (t0 - T::PADLO + l0 - L / 2) & (L - 1);
                const int g1 = (t1 - T::PADLO + l1 - L / 2) & (L - 1);
                const int g2 = (t2 - T::PADLO + l2 - L / 2) & (L - 1);
                const unsigned gi = (unsigned)((g0 * L + g1) * L + g2);  // < 2^30 (L <= 1024)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const long long v = (long long)tile[c][li];
                    if (v) to_grid(NC * gi + c, v);
                }
            }
        };
        if (a.units)
            flush([&](unsigned i, long long v) {
                __hip_atomic_fetch_add(a.units + i, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            });
        else
            flush([&](unsigned i, long long v) { unsafeAtomicAdd(a.grid + i, (float)((double)v * fx_inv)); });
    });
}

// grid = units / fxs, each integer sum rounded once to FP32 (n a multiple of 2)
__global__ void __launch_bounds__(256) k_units_grid(SpreadArgs a, int64_t n) {
    const double inv = unit_of(a).inv;
    const longlong2* __restrict__ u = reinterpret_cast<const longlong2*>(a.units);
    float2* __restrict__ g = reinterpret_cast<float2*>(a.grid);
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n / 2; i += (int64_t)gridDim.x * 256) {
        const longlong2 v = u[i];
        g[i] = make_float2((float)((double)v.x * inv), (float)((double)v.y * inv));
    }
}

// bits of the largest |component| of n complex values (atomic max on the bits of non-negative
// floats, which order like the floats); *out starts at 0.  HBM-bound (20.6 GB in 4.3 ms); one atomic
// per workgroup and at most 2,048 of them: with one per wavefront of up to 65,536 workgroups the
// atomics on the one word took 2.8 ms, whatever the size (N = 64 with 9,973 views: 2.84 -> 0.07 ms).
__global__ void __launch_bounds__(256) k_absmax(const float4* __restrict__ b, int64_t n2, const float2* __restrict__ tail,
                                                int ntail, unsigned* out) {
    __shared__ float red[4];
    float m = 0.f;
    const int64_t step = (int64_t)gridDim.x * 256;
    auto take = [&](const float4& v) {
        m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    };
    int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
    for (; i + 3 * step < n2; i += 4 * step) {
        const float4 v0 = b[i], v1 = b[i + step], v2 = b[i + 2 * step], v3 = b[i + 3 * step];
        take(v0);
        take(v1);
        take(v2);
        take(v3);
    }
    for (; i < n2; i += step) take(b[i]);
    if (blockIdx.x == 0 && (int)threadIdx.x < ntail) m = fmaxf(m, fmaxf(fabsf(tail[threadIdx.x].x), fabsf(tail[threadIdx.x].y)));
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(out, __float_as_uint(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))));
}

// zeroes the item counter, and with it the word of the largest component (A*b)
__global__ void k_zero_words(int* taken, unsigned* bmax) {
    *taken = 0;
    if (bmax) *bmax = 0u;
}

__global__ void k_fill_zero(float4* p, size_t n4) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n4; i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Re sum_m h_m(0) b(0, m): the k = 0 term of Re A*b (its exponential is 1 for all n).  Each view's
// sample lies in a line of its own, so the sum waits on memory: block j of the grid sums every
// gridDim.x-th run of 256 views into out[j] (one block for 5 x 10^4 views took 268 us).
__global__ void __launch_bounds__(256) k_atb_k0(const float2* __restrict__ b, const int32_t* group, const float* table,
                                                int Q, int M, int P, double* out) {
    __shared__ double red[4];
    double acc = 0.0;
    const int c = (P - 1) / 2;
    for (int m = blockIdx.x * 256 + threadIdx.x; m < M; m += gridDim.x * 256) {
        const int g = group ? group[m] : 0;
        const float h = table ? table[(int64_t)g * Q] : 1.f;
        acc += (double)h * (double)b[(int64_t)m * P + c].x;
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// out[0] = the sum of n <= 64 partial sums (one wavefront)
__global__ void k_sum64(const double* __restrict__ part, int n, double* out) {
    double v = (int)threadIdx.x < n ? part[threadIdx.x] : 0.0;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (threadIdx.x == 0) out[0] = v;
}

// chalf[p1][p2][n3] (n3 in [0, N)) -> kerc[p1][p2][p3] using Ker(-n) = Ker(n); p3 = N is 0.
__global__ void k_kerc_from_half(const float* __restrict__ chalf, float* __restrict__ kerc, int N) {
    const int N2 = 2 * N;
    const int64_t tot = (int64_t)N2 * N2 * N2;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < tot; i += (int64_t)gridDim.x * blockDim.x) {
        const int p3 = (int)(i % N2), p2 = (int)((i / N2) % N2), p1 = (int)(i / ((int64_t)N2 * N2));
        float v;
        if (p3 < N) v = chalf[((int64_t)p1 * N2 + p2) * N + p3];
        else if (p3 == N) v = 0.f;
        else v = chalf[((int64_t)((N2 - p1) % N2) * N2 + (N2 - p2) % N2) * N + (N2 - p3)];
        kerc[i] = v;
    }
}

// circulant order c[p] (offset o(p)) <-> centred order ker[j] (offset j - N)
__global__ void k_kerc_centred(const float* __restrict__ src, float* __restrict__ dst, int N, int to_centred) {
    const int N2 = 2 * N;
    const int64_t tot = (int64_t)N2 * N2 * N2;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < tot; i += (int64_t)gridDim.x * blockDim.x) {
        const int a3 = (int)(i % N2), a2 = (int)((i / N2) % N2), a1 = (int)(i / ((int64_t)N2 * N2));
        // index a in the destination order; map to the source order
        int s1, s2, s3;
        if (to_centred) {  // dst centred j -> offset j - N -> circulant p = offset mod 2N
            s1 = (a1 - N + N2) % N2; s2 = (a2 - N + N2) % N2; s3 = (a3 - N + N2) % N2;
            const bool wrap = (a1 == 0) || (a2 == 0) || (a3 == 0);
            dst[i] = wrap ? 0.f : src[((int64_t)s1 * N2 + s2) * N2 + s3];
        } else {           // dst circulant p -> offset o(p) -> centred j = o + N; p = N is the wrap
            const bool wrap = (a1 == N) || (a2 == N) || (a3 == N);
            s1 = (a1 + N) % N2; s2 = (a2 + N) % N2; s3 = (a3 + N) % N2;
            dst[i] = wrap ? 0.f : src[((int64_t)s1 * N2 + s2) * N2 + s3];
        }
    }
}

__global__ void k_f2d(const float* __restrict__ a, double* __restrict__ o, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        o[i] = a[i];
}

int grid_blocks(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, 65536); }

template <int W, bool CPLX>
hipError_t launch_w(firm_plan p, SpreadArgs& a, int nwork) {
    using T = SpreadTile<W, CPLX>;
    a.p.nt1 = (a.p.L + T::T1) / T::T1;  // starts 0 .. L
    a.p.nt2 = (a.p.L + T::T2) / T::T2;
    hipLaunchKernelGGL((k_spread<W, CPLX>), dim3(std::min(nwork, p->ncu)), dim3(pts::NTH), 0, p->stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !a.units) return e;
    const int64_t n = (int64_t)a.p.L * a.p.L * a.p.L * (CPLX ? 2 : 1);
    hipLaunchKernelGGL(k_units_grid, dim3(grid_blocks(n / 2)), dim3(256), 0, p->stream, a, n);
    return hipGetLastError();
}

template <bool CPLX>
hipError_t launch_spread(firm_plan p, int L, const int* work, int nwork, float* grid, unsigned long long* units,
                         const float2* b, float fxs, const unsigned* fx_bmax = nullptr, float fx_coef = 0.f) {
    SpreadArgs a;
    a.p = point_args(p, L, work, nwork);
    a.table = p->table; a.Q = p->Q; a.grid = grid; a.units = units;
    a.b = b; a.shifts = p->shiftss; a.rowstart = p->rowstart; a.P = p->P;
    a.fxs = fxs; a.fx_inv = 1.0 / (double)fxs;
    a.fx_bmax = fx_bmax; a.fx_coef = fx_coef;
    if (nwork == 0) return hipSuccess;
    switch (p->kbw) {
        case 4: return launch_w<4, CPLX>(p, a, nwork);
        case 5: return launch_w<5, CPLX>(p, a, nwork);
        case 6: return launch_w<6, CPLX>(p, a, nwork);
        case 7: return launch_w<7, CPLX>(p, a, nwork);
        case 8: return launch_w<8, CPLX>(p, a, nwork);
        default: return hipErrorInvalidValue;
    }
}

template <bool CPLX>
TileDims spread_dims(int W) {
    switch (W) {
        case 4: return tile_dims<SpreadTile<4, CPLX>>();
        case 5: return tile_dims<SpreadTile<5, CPLX>>();
        case 6: return tile_dims<SpreadTile<6, CPLX>>();
        case 7: return tile_dims<SpreadTile<7, CPLX>>();
        default: return tile_dims<SpreadTile<8, CPLX>>();
    }
}

}  // namespace

// Host work list: tiles of window starts (0 .. L; at odd widths start 0 lies half a cell below
// position 0) that can hold points, each split into view ranges, ordered by expected work (tiles near
// the origin meet every view's plane) so that the heavy ones start first.  The ranges hold about
// 1 / SP_ITEMS of all expected (tile, view) meetings: the tiles at the origin meet every view, and
// one workgroup for up to 16,384 views left them running alone (A*b at N = 64 with 9,973 views: 21.9 ->
// 9.1 ms with the atomic spread).
#define SP_ITEMS 2048
std::vector<int> points_worklist(int L, TileDims T, int W, int M) {
    constexpr int gran = 4 * SP_VRUN;  // ranges are whole runs of views
    const double shift = W % 2 ? -0.5 : 0.0;
    const int last = L;
    const int T0 = T.t0, T1 = T.t1, T2 = T.t2;
    const int n0 = last / T0 + 1, n1 = last / T1 + 1, n2 = last / T2 + 1;
    const double Rt = 0.5 * std::sqrt((double)T0 * T0 + (double)T1 * T1 + (double)T2 * T2);
    struct Tile { double expect; int t; };
    std::vector<Tile> tiles;
    tiles.reserve((size_t)n0 * n1 * n2);
    double total = 0.0;
    for (int a = 0; a < n0; ++a)
        for (int b = 0; b < n1; ++b)
            for (int c = 0; c < n2; ++c) {
                const double o = shift - 0.5 * L;
                const double x = (a + 0.5) * T0 + o, y = (b + 0.5) * T1 + o, z = (c + 0.5) * T2 + o;
                const double rho = std::sqrt(x * x + y * y + z * z);
                if (rho - Rt > 0.5 * L + 1.0) continue;
                const double expect = (rho <= Rt ? 1.0 : Rt / rho) * M;
                tiles.push_back({expect, (a * n1 + b) * n2 + c});
                total += expect;
            }
    const double chunk = std::max((double)gran, total / SP_ITEMS);
    // items by descending work, to the resolution of NBK classes (a counting sort: 2.4 x 10^5 items at
    // N = 256)
    constexpr int NBK = 2048;
    auto parts = [&](const Tile& t) { return std::max(1, (int)std::ceil(t.expect / chunk)); };
    double wmax = 1.0;
    for (const Tile& t : tiles) wmax = std::max(wmax, t.expect / parts(t));
    auto cls = [&](const Tile& t, int nch) { return std::min(NBK - 1, (int)(NBK * (1.0 - t.expect / nch / wmax))); };
    auto step = [&](int nch) { return ((M + nch - 1) / nch + gran - 1) / gran * gran; };
    std::vector<size_t> at(NBK + 1, 0);
    for (const Tile& t : tiles) {
        const int nch = parts(t), per = step(nch);
        at[cls(t, nch) + 1] += (size_t)((M + per - 1) / per);
    }
    for (int i = 0; i < NBK; ++i) at[i + 1] += at[i];
    std::vector<int> out(4 * at[NBK]);
    for (const Tile& t : tiles) {
        const int nch = parts(t), per = step(nch);
        size_t& i = at[cls(t, nch)];
        for (int m0 = 0; m0 < M; m0 += per, ++i) {
            int* o = &out[4 * i];
            o[0] = t.t; o[1] = m0; o[2] = std::min(M, m0 + per); o[3] = 0;
        }
    }
    return out;
}

// The work lists of the kernel's spread (cplx = false, grid 4N) and A*b's (grid 2N).
std::vector<int> spread_worklist(int N, int W, int M, bool cplx) {
    return points_worklist((cplx ? 2 : 4) * N, cplx ? spread_dims<true>(W) : spread_dims<false>(W), W, M);
}

hipError_t fill_zero(void* ptr, size_t bytes, hipStream_t s) {
    const size_t n4 = bytes / 16;
    if (n4) hipLaunchKernelGGL(k_fill_zero, dim3(grid_blocks(n4)), dim3(256), 0, s, (float4*)ptr, n4);
    const size_t rem = bytes - n4 * 16;
    if (rem) {
        hipError_t e = hipMemsetAsync((char*)ptr + n4 * 16, 0, rem, s);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

hipError_t spread_ker(firm_plan p, float* grid, unsigned long long* units) {
    const int64_t L = 4 * p->N, n = L * L * L;
    hipError_t e = units ? fill_zero(units, n * sizeof(*units), p->stream) : fill_zero(grid, n * sizeof(float), p->stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(1), 0, p->stream, p->taken, (unsigned*)nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_spread<false>(p, (int)L, p->tiles_ker, p->ntiles_ker, grid, units, nullptr, p->fx_ker);
}

hipError_t spread_atb(firm_plan p, const float2* b, float2* grid, unsigned long long* units) {
    const int64_t L = 2 * p->N, cells = L * L * L;
    hipError_t e = units ? fill_zero(units, 2 * cells * sizeof(*units), p->stream)
                         : fill_zero(grid, cells * sizeof(float2), p->stream);
    if (e != hipSuccess) return e;
    // the fixed-point unit follows from the largest |component| of b, found first
    const int64_t n = (int64_t)p->M * p->P;
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(1), 0, p->stream, p->taken, p->fx_bmax);
    hipLaunchKernelGGL(k_absmax, dim3(std::max(1, std::min(grid_blocks(n / 2), 2048))), dim3(256), 0, p->stream,
                       reinterpret_cast<const float4*>(b), n / 2, b + (n / 2) * 2, (int)(n % 2), p->fx_bmax);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_spread<true>(p, (int)L, p->tiles_atb, p->ntiles_atb, reinterpret_cast<float*>(grid), units, b, 1.f,
                               p->fx_bmax, p->fx_atb_coef);
}

hipError_t atb_k0_term(firm_plan p, const float2* b, double* out) {
    const int nb = std::min(64, (p->M + 1023) / 1024);
    hipLaunchKernelGGL(k_atb_k0, dim3(nb), dim3(256), 0, p->stream, b, p->group, p->table, p->Q, p->M, p->P,
                       nb == 1 ? out : p->partials);
    if (nb > 1) hipLaunchKernelGGL(k_sum64, dim3(1), dim3(64), 0, p->stream, p->partials, nb, out);
    return hipGetLastError();
}

hipError_t kerc_from_half(firm_plan p, const float* chalf) {
    const int64_t n = 8LL * p->N * p->N * p->N;
    hipLaunchKernelGGL(k_kerc_from_half, dim3(grid_blocks(n)), dim3(256), 0, p->stream, chalf, p->kerc, p->N);
    return hipGetLastError();
}

hipError_t kerc_to_centred(firm_plan p, float* out) {
    const int64_t n = 8LL * p->N * p->N * p->N;
    hipLaunchKernelGGL(k_kerc_centred, dim3(grid_blocks(n)), dim3(256), 0, p->stream, p->kerc, out, p->N, 1);
    return hipGetLastError();
}

hipError_t kerc_from_centred(firm_plan p, const float* in) {
    const int64_t n = 8LL * p->N * p->N * p->N;
    hipLaunchKernelGGL(k_kerc_centred, dim3(grid_blocks(n)), dim3(256), 0, p->stream, in, p->kerc, p->N, 0);
    return hipGetLastError();
}

hipError_t kerc_to_double(firm_plan p, double* out) {
    const int64_t n = 8LL * p->N * p->N * p->N;
    hipLaunchKernelGGL(k_f2d, dim3(grid_blocks(n)), dim3(256), 0, p->stream, p->kerc, out, n);
    return hipGetLastError();
}

// Forward projector of libfirm (eq. forward-projector): slices of a volume at the sample
// points xi_{k,m} = R_m^{-1}(omega_k, 0), with the CTF and the image shift applied,
//
//   b(k, m) = h_m(|k|) exp(-i <omega_k, s_m>) sum_n V(n) exp(-i <n, xi_{k,m}>).
//
// This is the adjoint of the back-projection (spread.hip; it re-centres by
// exp(+i <omega_k, s_m>)), evaluated as a type-2 non-uniform FFT on the same grid (L = 2N),
// with the same Kaiser-Bessel window and the same cell convention:
//   1. u(n) = V(n) / phihat(n1) phihat(n2) phihat(n3)      (the window's transform)
//   2. G(g) = sum_n u(n) exp(-2 pi i <n, g> / L), g in [0, L)^3 (three FFT passes; real u,
//      so only q3 in [0, N] is formed, the rest is conj G(-g))
//   3. b = sum over the W^3 window cells of weight * G(cell).
// Step 3 walks the grid in tiles, the transpose of the gridding spread: a workgroup loads its padded
// tile of G into LDS once, points.h finds the tile's points and sorts them into bins, and a wavefront
// takes 16 points of a bin at a time: their axis-0 weights (16 points x 16 rows) times the bin's cells
// (16 rows x CJ 8 columns, held in registers for the chunk) on the matrix units, then the weighted sum
// over the columns.  Every point belongs to exactly one tile, so every output is written once, with
// no atomics.  The half disk (k1 > 0, or k1 = 0 and k2 > 0) is gathered; b(-k) = conj b(k) for
// real V, and b(0) = h(0) sum V is formed exactly.
//
// What bounds it, at N = 256 with 2 x 10^4 views (5.1e8 points, 37.9 ms; 65.4 with one thread per point
// and 343 LDS reads each): vector-unit issue.  Time saved by leaving one part out: the matrix products 13.3 ms,
// their operands and the sums over the columns about 8, window weights 5, the outputs with CTF and phase 5,
// finding and locating points (with the FFTs) 14; these overlap in part.  With few views, the fixed steps of a
// tile: W = 7 at N = 64 with 30 views 81 us (83 with a thread per point).  W = 4 with 30 to 100 views at N <= 64
// is the one range where a thread per point, with 64 cells each, was the faster (N = 64, 50 views: 58 us, now 72).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "firm_internal.h"
#include "points.h"

#define PJ_PREP_BLOCKS 1024

namespace {

struct ProjArgs {
    pts::Args p;
    int P, Q, QP;
    const float* table;
    const float2* X;       // [q1][q2][q3], q3 in [0, N], pitch QP
    const double* shifts;
    const int* rowstart;
    float2* b;
};

// Tiles on the 2N grid.  With many views 10 x 12 x 12 window starts at W = 7 (41 KB of complex cells,
// 36 bins; the rest of the LDS is queue); with few points per tile, where each tile's fixed work
// (its cells, the steps of one queueful) is what counts, 10 x 16 x 16 (62 KB, 64 bins, half the
// tiles).  N = 256: 2 x 10^4 views (10^4 points per narrow tile) 38.3 ms narrow, 40.9 wide; 762
// views (400 points) 4.5 narrow, 3.8 wide.  N = 128 with 5,000 views (5,300 points): 2.60, 2.73.
template <int W, bool WIDE>
using ProjTile = pts::Tile<W, 2, 1, (WIDE ? 22 : 18), (WIDE ? 22 : 18), 8, 2, true>;
constexpr double PJ_WIDE_BELOW = 2000;  // points per narrow tile

// u = V / (phihat(n1) phihat(n2) phihat(n3)) and per-block FP64 partial sums of V.
__global__ void __launch_bounds__(256) k_fp_prep(const float* __restrict__ V, const float* __restrict__ dec, int N,
                                                 float* __restrict__ u, double* __restrict__ partials) {
    __shared__ double red[4];
    const int64_t n3 = (int64_t)N * N * N;
    double acc = 0.0;
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n3; i += (int64_t)gridDim.x * 256) {
        const int i3 = (int)(i % N), i2 = (int)((i / N) % N), i1 = (int)(i / ((int64_t)N * N));
        const float v = V[i];
        acc += (double)v;
        u[i] = v * dec[i1] * dec[i2] * dec[i3];
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// b(0, m) = h_m(0) sum V; every block forms the same sum of the partials in the same order.  Also zeroes
// the gather's item counter.
__global__ void __launch_bounds__(256) k_fp_k0(const double* __restrict__ partials, int nblk,
                                               const int32_t* __restrict__ group, const float* __restrict__ table,
                                               int Q, int M, int P, float2* __restrict__ b, int* taken) {
    __shared__ double red[4];
    __shared__ float total;
    if (blockIdx.x == 0 && threadIdx.x == 0) *taken = 0;
    double acc = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) acc += partials[i];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) total = (float)((red[0] + red[1]) + (red[2] + red[3]));
    __syncthreads();
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m >= M) return;
    const int g = group ? group[m] : 0;
    const float h = table ? table[(int64_t)g * Q] : 1.f;
    b[(int64_t)m * P + (P - 1) / 2] = make_float2(h * total, 0.f);
}

// G at grid index q from the half spectrum X of the array-index transform: the volume sits at
// n = i - N/2, so G(q) = i^(q1 + q2 + q3) X(q) (L is a multiple of 4), and X(q) = conj X(-q).
__device__ __forceinline__ float2 load_half(const float2* __restrict__ X, int L, int N, int QP, int q0, int q1, int q2) {
    const bool neg = q2 > N;
    const int r0 = neg ? (L - q0) & (L - 1) : q0, r1 = neg ? (L - q1) & (L - 1) : q1;
    return X[((int64_t)r0 * L + r1) * QP + (neg ? L - q2 : q2)];
}
__device__ __forceinline__ float2 grid_value(float2 v, int N, int q0, int q1, int q2) {
    if (q2 > N) v.y = -v.y;
    const int q = q0 + q1 + q2;
    if (q & 1) v = make_float2(-v.y, v.x);
    return q & 2 ? make_float2(-v.x, -v.y) : v;
}

// Sum over each row of 16 lanes, in every lane.
template <int CTRL>
__device__ __forceinline__ float dpp_sum(float v) {
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_sum(float v) {
    v = dpp_sum<0xB1>(v);     // lane ^ 1
    v = dpp_sum<0x4E>(v);     // lane ^ 2
    v = dpp_sum<0x141>(v);    // mirrored in 8
    return dpp_sum<0x140>(v);  // mirrored in 16
}

template <int W, bool WIDE>
__global__ void __launch_bounds__(pts::NTH, pts::NTH / 256) k_project(ProjArgs a) {
    using T = ProjTile<W, WIDE>;
    constexpr int NJ = T::NJ;
    __shared__ float2 tile[T::CELLS];
    __shared__ pts::Lds<T> s;
    __shared__ int rowstart[132];  // the disk's rows k1 >= 0 (N <= 256)

    const int tid = threadIdx.x, lane = tid & 63;
    const int L = a.p.L, N = a.p.N;
    const double inv_n = 1.0 / N;
    for (int i = tid; i <= N / 2; i += pts::NTH) rowstart[i] = a.rowstart[i + N / 2];

    // Lane roles: as an operand's row, point lane & 15; as its inner index and the accumulators' rows,
    // q = lane / 16 (cell rows 4 ks + q; points 4 q + r); as columns, (axis 1, axis 2) = (NJ e + n, kk).
    const int q = lane >> 4, e = (lane >> 3) & 1, kk = lane & 7;
    const float* const wave = s.wave[tid >> 6];
    const float* const rowb = wave + T::LEAD + 16 * T::S0;
    struct Cells {
        float2 g[4][4];       // the bin's cells of this lane (W <= 7)
        const float2* first;  // the first of them
    };
    auto open = [&](int bin) {
        Cells c;
        const int o0 = bin / (T::NB1 * T::NB2) * T::B0, o1 = bin / T::NB2 % T::NB1 * T::B1, o2 = bin % T::NB2 * T::B2;
        c.first = tile + ((o0 + q) * T::P1 + o1 + NJ * e) * T::RP + o2 + kk;
        if constexpr (NJ == 4) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int n = 0; n < 4; ++n) c.g[ks][n] = c.first[(4 * ks * T::P1 + n) * T::RP];
        }
        return c;
    };
    auto round = [&](const Cells& c, int cnt, int at) {
        const int pr = lane & 15;
        const int o = __float_as_int(rowb[pr * T::SB + T::OFFV + 1]);
        float w0[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            w0[ks] = *reinterpret_cast<const float*>(
                reinterpret_cast<const char*>(wave + T::LEAD + pr * T::S0 + 4 * ks + q) + o);
        float re[4] = {0.f, 0.f, 0.f, 0.f}, im[4] = {0.f, 0.f, 0.f, 0.f};
        auto columns = [&](const pts::f4& cr, const pts::f4& ci, const pts::f4& w) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                re[r] = fmaf(w[r], cr[r], re[r]);
                im[r] = fmaf(w[r], ci[r], im[r]);
            }
        };
        if constexpr (NJ == 4) {
            pts::f4 cr[4], ci[4];
#pragma unroll
            for (int n = 0; n < 4; ++n) cr[n] = ci[n] = pts::f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    cr[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[ks], c.g[ks][n].x, cr[n], 0, 0, 0);
                    ci[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[ks], c.g[ks][n].y, ci[n], 0, 0, 0);
                }
            pts::f4 w1[4];  // axis-1 weights of the points 4 q + r
#pragma unroll
            for (int r = 0; r < 4; ++r) w1[r] = *reinterpret_cast<const pts::f4*>(rowb + (4 * q + r) * T::SB + NJ * e);
#pragma unroll
            for (int n = 0; n < 4; ++n) columns(cr[n], ci[n], pts::f4{w1[0][n], w1[1][n], w1[2][n], w1[3][n]});
        } else {
#pragma unroll 2
            for (int n = 0; n < NJ; ++n) {
                pts::f4 cr = {0.f, 0.f, 0.f, 0.f}, ci = cr;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const float2 v = c.first[(4 * ks * T::P1 + n) * T::RP];
                    cr = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[ks], v.x, cr, 0, 0, 0);
                    ci = __builtin_amdgcn_mfma_f32_16x16x4f32(w0[ks], v.y, ci, 0, 0, 0);
                }
                const float* w = rowb + 4 * q * T::SB + NJ * e + n;
                columns(cr, ci, pts::f4{w[0], w[T::SB], w[2 * T::SB], w[3 * T::SB]});
            }
        }
        float sr = 0.f, si = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float w2 = rowb[(4 * q + r) * T::SB + T::CJ + kk];
            const float x = row_sum(w2 * re[r]), y = row_sum(w2 * im[r]);
            sr = (lane & 3) == r ? x : sr;
            si = (lane & 3) == r ? y : si;
        }
        const int p = 4 * q + (lane & 3);
        if ((lane & 15) < 4 && p < cnt) {
            const int i = s.order[at + p];
            s.f[3][i] = sr;
            s.f[4][i] = si;
        }
    };
    // the points' outputs, in the order they were found (neighbours along a row together)
    auto finish = [&](int g0, const int* ent, const int* place) {
#pragma unroll
        for (int j = 0; j < T::EPT; ++j) {
            if (place[j] < 0) continue;
            const int64_t m = g0 + pts::entry_view(ent[j]);
            const int k1 = pts::entry_k1(ent[j]), k2 = pts::entry_k2(ent[j]);
            const float4 rec = a.p.vrec[2 * m + 1];  // (.., group, the caller's view)
            const float h = a.table ? a.table[(int64_t)__float_as_int(rec.z) * a.Q + k1 * k1 + k2 * k2] : 1.f;
            const double s1 = a.shifts ? a.shifts[2 * m] : 0.0, s2 = a.shifts ? a.shifts[2 * m + 1] : 0.0;
            const float ar = s.f[3][tid + j * pts::NTH], ai = s.f[4][tid + j * pts::NTH];
            float cs = 1.f, sn = 0.f;
            if (a.shifts) {
                // theta = 2 pi x, x = <k, s_m> / N (N a power of 2) reduced to [-1/2, 1/2] in FP64, then an
                // FP32 sincospi
                const double x = (k1 * s1 + k2 * s2) * inv_n;
                sincospif(2.f * (float)(x - rint(x)), &sn, &cs);
            }
            // h exp(-i theta) (ar + i ai), and its conjugate at -k
            const float2 v = make_float2(h * (ar * cs + ai * sn), h * (ai * cs - ar * sn));
            const int idx = rowstart[k1] + k2;
            const int64_t mo = (int64_t)__float_as_int(rec.w) * a.P;
            a.b[mo + idx] = v;
            a.b[mo + (a.P - 1 - idx)] = make_float2(v.x, -v.y);
        }
    };
    pts::for_items<T>(a.p, s, [&](int4 wk) {
        const int nt12 = a.p.nt1 * a.p.nt2;
        const int t0 = wk.x / nt12 * T::T0, t1 = wk.x / a.p.nt2 % a.p.nt1 * T::T1, t2 = wk.x % a.p.nt2 * T::T2;
        // the padded tile of G: LDS cell l holds grid index (t - PADLO + l - L/2) mod L (a power of 2)
        // (eight loads in flight a thread: with few points in a tile its cells are what it waits for; one at a time,
        // N = 64 with 30 views took 90.6 us, now 83.4, and N = 256 with 300 views 3.12 ms, now 2.94)
        auto begin = [&]() {
            constexpr int CELLS = T::P0 * T::P1 * T::P2, B = 8;
            auto where = [&](int i, int (&g)[3]) {
                const int l[3] = {i / (T::P1 * T::P2), i / T::P2 % T::P1, i % T::P2};
                g[0] = (t0 - T::PADLO + l[0] - L / 2) & (L - 1);
                g[1] = (t1 - T::PADLO + l[1] - L / 2) & (L - 1);
                g[2] = (t2 - T::PADLO + l[2] - L / 2) & (L - 1);
                return (l[0] * T::P1 + l[1]) * T::RP + l[2];
            };
            int first = tid;
            asm volatile("" : "+v"(first));  // or the cells' indices are formed ahead, and spilled
            for (int i0 = first; i0 < CELLS; i0 += B * pts::NTH) {
                float2 v[B];
                int g[3];
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    where(min(i0 + j * pts::NTH, CELLS - 1), g);
                    v[j] = load_half(a.X, L, N, a.QP, g[0], g[1], g[2]);
                }
#pragma unroll
                for (int j = 0; j < B; ++j) {
                    const int i = i0 + j * pts::NTH;
                    if (i >= CELLS) break;
                    const int cell = where(i, g);
                    tile[cell] = grid_value(v[j], N, g[0], g[1], g[2]);
                }
            }
        };
        pts::for_points<T>(a.p, s, wk, t0, t1, t2, begin, [](int, int, int) { return 0; },
                           [](int, int, int, float*) {}, open, round, [](const Cells&, int) {}, finish);
    });
}

template <int W, bool WIDE>
hipError_t launch_w(firm_plan p, ProjArgs& a) {
    using T = ProjTile<W, WIDE>;
    a.p.nt1 = (a.p.L + T::T1) / T::T1;  // starts 0 .. L
    a.p.nt2 = (a.p.L + T::T2) / T::T2;
    hipLaunchKernelGGL((k_project<W, WIDE>), dim3(std::min(a.p.nwork, p->ncu)), dim3(pts::NTH), 0, p->stream, a);
    return hipGetLastError();
}

}  // namespace

// b (M x P complex64, disk order) = forward projection of V (N^3, centred order).
// Workspaces: p->tmp (u), p->T1, p->ws1, p->grid (the caller has sized the gridding workspaces).
hipError_t forward_project(firm_plan p, const float* V, float2* b) {
    const int N = p->N, L = 2 * N;
    hipStream_t st = p->stream;
    const int nblk = std::min<int>(PJ_PREP_BLOCKS, p->npart);
    hipLaunchKernelGGL(k_fp_prep, dim3(nblk), dim3(256), 0, st, V, p->deconv_atb, N, p->tmp, p->partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_fp_k0, dim3((p->M + 255) / 256), dim3(256), 0, st, p->partials, nblk, p->group, p->table,
                       p->Q, p->M, p->P, b, p->taken);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    float2* X = reinterpret_cast<float2*>(p->grid);
    if ((e = fft_project_grid(p, p->tmp, p->T1, reinterpret_cast<float2*>(p->ws1), X)) != hipSuccess) return e;
    if (p->ntiles_prj == 0) return hipSuccess;
    ProjArgs a;
    a.p = point_args(p, L, p->tiles_prj, p->ntiles_prj);
    a.P = p->P; a.Q = p->Q; a.QP = p->QP;
    a.table = p->table; a.X = X; a.shifts = p->shiftss; a.rowstart = p->rowstart; a.b = b;
    switch (p->kbw) {
        case 4: return p->prj_wide ? launch_w<4, true>(p, a) : launch_w<4, false>(p, a);
        case 5: return p->prj_wide ? launch_w<5, true>(p, a) : launch_w<5, false>(p, a);
        case 6: return p->prj_wide ? launch_w<6, true>(p, a) : launch_w<6, false>(p, a);
        case 7: return p->prj_wide ? launch_w<7, true>(p, a) : launch_w<7, false>(p, a);
        case 8: return p->prj_wide ? launch_w<8, true>(p, a) : launch_w<8, false>(p, a);
        default: return hipErrorInvalidValue;
    }
}

std::vector<int> project_worklist(int N, int W, int M, int64_t P, bool& wide) {
    auto dims = [&](auto wd) {
        constexpr bool WD = decltype(wd)::value;
        switch (W) {
            case 4: return tile_dims<ProjTile<4, WD>>();
            case 5: return tile_dims<ProjTile<5, WD>>();
            case 6: return tile_dims<ProjTile<6, WD>>();
            case 7: return tile_dims<ProjTile<7, WD>>();
            default: return tile_dims<ProjTile<8, WD>>();
        }
    };
    const TileDims d = dims(std::false_type{});
    const double tiles = 4.0 / 3.0 * M_PI * std::pow((double)N, 3) / ((double)d.t0 * d.t1 * d.t2);  // in the ball
    wide = 0.5 * (double)P * M < PJ_WIDE_BELOW * tiles;
    return points_worklist(2 * N, wide ? dims(std::true_type{}) : d, W, M);
}

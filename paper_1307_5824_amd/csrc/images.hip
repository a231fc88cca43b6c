// Step 1 of the algorithm (section 3.4): Fourier slices from real-space images, and a
// real-space image generator for synthetic data.
//
// Slices.  An image J_m on the pixel grid x in [-N/2, N/2)^2 (pixel i at x = i - N/2) gives
// b(k, m) = sum_x J_m(x) exp(-2 pi i <k, x> / N) (the centred DFT of section 2.2) at the disk
// points ||k|| <= N/2.  The FFT passes transform the array index i, so b(k) = (-1)^(k1 + k2)
// X(k mod N); the real rows keep q2 in [0, N/2] and X(-q) = conj X(q) supplies the rest.  The
// disk's boundary points k_d = +N/2 take the periodic value X(N/2), equal to X(-N/2).
//
// Images.  A Gaussian blob a exp(-||x - c||^2 / (2 s^2)) projects along the viewing direction
// (third row of R_m) to the 2D Gaussian a sqrt(2 pi) s exp(-||x - p||^2 / (2 s^2)) centred at
// p = ((R_m c)_1, (R_m c)_2); an image of a particle off-centre by s_m is J(x - s_m), so p moves
// by s_m (the back-projection undoes this by its re-centring phase).  Blobs farther than
// PROJ_CUT sigmas from a pixel row are skipped (their weight is below exp(-PROJ_CUT^2 / 2)).
// Pixel noise: N(0, sigma^2) per pixel from Philox4x32-10 keyed by the seed, counter
// (m, pixel, 0, 2), sigma^2 = mean clean pixel power / SNR.
#include <algorithm>
#include <cmath>

#include "fft_core.h"
#include "firm_internal.h"
#include "philox.h"

#define IMG_THREADS 256
#define IMG_MAXB 320
#define PROJ_CUT 9.0f

namespace {

// The disk point (k1, k2) from an image's spectrum: get(q1, q1m, k2) gives X(q1, k2) for 0 <= k2 <= N/2,
// q1m = -q1 mod N; X(k1, -k2) = conj X(-k1, k2).
template <class F>
__device__ __forceinline__ float2 disk_value(int N, int k1, int k2, F&& get) {
    const int q1 = (k1 + N) & (N - 1), q1m = (N - q1) & (N - 1);
    float2 v = k2 >= 0 ? get(q1, q1m, k2) : get(q1m, q1, -k2);
    if (k2 < 0) v.y = -v.y;
    if ((k1 + k2) & 1) { v.x = -v.x; v.y = -v.y; }
    return v;
}

// Gather of the disk points from half spectra in HBM (N = 256): a wavefront per row k1 of an image, the
// image's rows over `parts` workgroups (one image: 98 us with one workgroup, which has 65 rows a wavefront).
__global__ void __launch_bounds__(IMG_THREADS) k_img_gather(const float2* __restrict__ spec, int N, int QPn, int P,
                                                           const int* __restrict__ rowstart, int m0, int parts,
                                                           float2* __restrict__ b) {
    const int g = blockIdx.x / parts, part = blockIdx.x % parts, lane = threadIdx.x & 63;
    const float2* X = spec + (int64_t)g * N * QPn;
    float2* out = b + (int64_t)(m0 + g) * P;
    for (int r = part * (IMG_THREADS / 64) + (threadIdx.x >> 6); r <= N; r += parts * (IMG_THREADS / 64)) {
        const int k1 = r - N / 2, left = N * N / 4 - k1 * k1;
        int kmax = (int)__builtin_amdgcn_sqrtf((float)left);
        kmax += (kmax + 1) * (kmax + 1) <= left ? 1 : 0;
        kmax -= kmax * kmax > left ? 1 : 0;
        for (int k2 = -kmax + lane; k2 <= kmax; k2 += 64)
            out[rowstart[r] + k2] = disk_value(N, k1, k2, [&](int q1, int, int k) { return X[(int64_t)q1 * QPn + k]; });
    }
}

// Step 1 of N <= 128 in one kernel: a workgroup holds one image (1,024 threads at N = 128) or, below
// N = 64, as many as 256 threads transform (16 at N = 16) in LDS, N rows of N/2 columns each, from
// the pixels to the disk points; HBM moves the pixels and the slices only, 168 KB per image at N = 128
// instead of 660 (half spectra written and read between the row transforms, the column transforms
// and the gather).  Rows in pairs, as one complex
// pencil; the columns q2 = 0 and N/2 of a real image are both real before the column transforms, so
// they share one complex column.  The transforms exchange in place: a pencil's exchange buffer
// is its own two rows (9 slots of 8, against bank conflicts), then its own column.  73,728 bytes of LDS
// and the N twiddles (N = 128) leave room for two workgroups per CU, whose loads, transforms and stores
// overlap.  N = 128, 10,007 images: 1,630 -> 430 us, 3.9 TB/s (a large copy reaches 4.8); N = 64, 20,000:
// 1,100 -> 264 us; N = 8, 40,000: 224 -> 21 us.
template <int N>
struct ImgTile {
    static constexpr int H = N / 2, PITCH = H + H / 8;  // complex columns, and the pitch of a row
    static constexpr int T = N / 8, NT = H * T;         // threads per pencil, per image
    static constexpr int NTH = NT > 256 ? NT : 256;     // threads per workgroup
    static constexpr int IPB = NTH / NT;                // images per workgroup
    struct Rows {  // pencil c: rows 2c and 2c + 1
        static __device__ __forceinline__ int idx(int e, int c) { return 2 * c * PITCH + e + (e >> 3); }
    };
    struct Cols {
        static __device__ __forceinline__ int idx(int e, int c) { return e * PITCH + c; }
    };
};

template <int N>
__global__ void __launch_bounds__(ImgTile<N>::NTH, 8) k_img_slices(const float* __restrict__ img, int M, int P,
                                                       const int* __restrict__ rowstart, const float2* __restrict__ tw,
                                                       float2* __restrict__ b) {
    using I = ImgTile<N>;
    constexpr int H = I::H, T = I::T;
    __shared__ float2 slab[I::IPB * N * I::PITCH];
    __shared__ float2 twl[N];  // exp(-2 pi i m / N)
    __shared__ int row[N + 1];  // the disk's row starts (from memory, one image of N = 128 took 14.3 us, now 13.6)
    const int tid = threadIdx.x;
    if (tid < N) twl[tid] = tw[tid * (FIRM_TWN / N)];
    if (tid <= N) row[tid] = rowstart[tid];
    const int li = tid % I::NT;
    const int m = blockIdx.x * I::IPB + tid / I::NT;
    const bool live = m < M;
    const float* x = img + (int64_t)(live ? m : M - 1) * N * N;
    float2* s = slab + tid / I::NT * (N * I::PITCH);
    float2 v[8];
    {
        const int c = li / T, j = li % T;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int e = j + t * T;
            v[t] = make_float2(__builtin_nontemporal_load(x + (2 * c) * N + e),
                               __builtin_nontemporal_load(x + (2 * c + 1) * N + e));
        }
        __syncthreads();  // the twiddles are in place
        reg_stages<typename I::Rows, N, 1, N>(v, s, twl, -1.f, c, j);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 8; ++t) s[I::Rows::idx(j + t * T, c)] = v[t];
        __syncthreads();
        float2 xa[4], xb[4];  // spectra of the rows 2c and 2c + 1 at q = j + t T < N/2
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int q = j + t * T;
            const float2 Z = s[I::Rows::idx(q, c)], Zm = s[I::Rows::idx(q == 0 ? H : N - q, c)];
            if (q == 0) {  // q = 0 and N/2 (Zm), real for each row: the shared column
                xa[t] = make_float2(Z.x, Zm.x);
                xb[t] = make_float2(Z.y, Zm.y);
            } else {
                xa[t] = make_float2(0.5f * (Z.x + Zm.x), 0.5f * (Z.y - Zm.y));
                xb[t] = make_float2(0.5f * (Z.y + Zm.y), -0.5f * (Z.x - Zm.x));
            }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            s[(2 * c) * I::PITCH + j + t * T] = xa[t];
            s[(2 * c + 1) * I::PITCH + j + t * T] = xb[t];
        }
        __syncthreads();
    }
    {
        const int c = li % H, j = li / H;
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = s[I::Cols::idx(j + t * T, c)];
        reg_stages<typename I::Cols, N, 1, N>(v, s, twl, -1.f, c, j);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 8; ++t) s[I::Cols::idx(j + t * T, c)] = v[t];
        __syncthreads();
    }
    // the images' disks: the threads take the points of the (N + 1)^2 squares around them in order
    constexpr int SQ = (N + 1) * (N + 1);
    for (int i = tid; i < I::IPB * SQ; i += I::NTH) {
        const int g = i / SQ, r = i % SQ / (N + 1), k1 = r - N / 2, k2 = i % (N + 1) - N / 2;
        const int mg = blockIdx.x * I::IPB + g;
        if (mg >= M) break;
        if (4 * (k1 * k1 + k2 * k2) > N * N) continue;
        const float2* X = slab + g * (N * I::PITCH);
        b[(int64_t)mg * P + row[r] + k2] = disk_value(N, k1, k2, [&](int q1, int q1m, int k) {
            const float2 a = X[q1 * I::PITCH + (k & (H - 1))];
            if (k & (H - 1)) return a;
            const float2 c = X[q1m * I::PITCH];  // the shared column: X0 + i X_{N/2}
            return k == 0 ? make_float2(0.5f * (a.x + c.x), 0.5f * (a.y - c.y))
                          : make_float2(0.5f * (a.y + c.y), -0.5f * (a.x - c.x));
        });
    }
}

template <int N>
hipError_t launch_slices(firm_plan p, const float* img, float2* b) {
    using I = ImgTile<N>;
    hipLaunchKernelGGL((k_img_slices<N>), dim3((p->M + I::IPB - 1) / I::IPB), dim3(I::NTH), 0, p->stream, img, p->M, p->P,
                       p->rowstart, p->tw, b);
    return hipGetLastError();
}

struct ImgArgs {
    int N, M, B;
    const double* c12;     // rows 1 and 2 of R_m
    const double* shifts;  // M x 2 or null
    const double* blobs;   // B x 5: c (3), sigma, a sqrt(2 pi) sigma
    float* img;
    double* partials;      // per-block clean power
    double snr;
    uint64_t seed;
};

// Clean images: block (m, row band); the blob list of each row is rebuilt in LDS with the
// row factor w exp(-(x1 - p1)^2 / (2 s^2)) folded in.
constexpr int IMG_ROWS = 8;

__global__ void __launch_bounds__(IMG_THREADS) k_synth_images(ImgArgs a) {
    __shared__ float bp1[IMG_MAXB], bp2[IMG_MAXB], binv[IMG_MAXB], bw[IMG_MAXB], bcut[IMG_MAXB];
    __shared__ float lp2[IMG_MAXB], linv[IMG_MAXB], lw[IMG_MAXB], lcut[IMG_MAXB];
    __shared__ int ln;
    __shared__ double red[IMG_THREADS / 64];
    const int N = a.N;
    const int bands = (N + IMG_ROWS - 1) / IMG_ROWS;
    const int m = blockIdx.x / bands, band = blockIdx.x % bands;
    const double* c = a.c12 + 6 * (int64_t)m;
    const double s1 = a.shifts ? a.shifts[2 * (int64_t)m] : 0.0, s2 = a.shifts ? a.shifts[2 * (int64_t)m + 1] : 0.0;
    for (int i = threadIdx.x; i < a.B; i += IMG_THREADS) {
        const double* q = a.blobs + 5 * i;
        const double s = q[3];
        bp1[i] = (float)(c[0] * q[0] + c[1] * q[1] + c[2] * q[2] + s1);
        bp2[i] = (float)(c[3] * q[0] + c[4] * q[1] + c[5] * q[2] + s2);
        binv[i] = (float)(0.5 / (s * s));
        bw[i] = (float)q[4];
        bcut[i] = PROJ_CUT * (float)s;
    }
    double acc = 0.0;
    for (int rr = 0; rr < IMG_ROWS; ++rr) {
        const int i1 = band * IMG_ROWS + rr;
        if (i1 >= N) break;  // uniform
        __syncthreads();
        if (threadIdx.x == 0) ln = 0;
        __syncthreads();
        const float x1 = (float)(i1 - N / 2);
        for (int i = threadIdx.x; i < a.B; i += IMG_THREADS) {
            const float d = x1 - bp1[i];
            if (fabsf(d) <= bcut[i]) {
                const int k = atomicAdd(&ln, 1);
                lp2[k] = bp2[i];
                linv[k] = binv[i];
                lw[k] = bw[i] * expf(-d * d * binv[i]);
                lcut[k] = bcut[i];
            }
        }
        __syncthreads();
        const int n = ln;
        float* row = a.img + ((int64_t)m * N + i1) * N;
        for (int i2 = threadIdx.x; i2 < N; i2 += IMG_THREADS) {
            const float x2 = (float)(i2 - N / 2);
            float v = 0.f;
            for (int k = 0; k < n; ++k) {
                const float d = x2 - lp2[k];
                if (fabsf(d) <= lcut[k]) v = fmaf(lw[k], expf(-d * d * linv[k]), v);
            }
            row[i2] = v;
            acc += (double)v * v;
        }
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) a.partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Per-block sums of the block partials (grid-stride over the partials), then one block totals.
__global__ void __launch_bounds__(256) k_sum(const double* __restrict__ in, int64_t n, double* __restrict__ out) {
    __shared__ double red[4];
    double acc = 0.0;
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) acc += in[i];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ void __launch_bounds__(256) k_img_noise(ImgArgs a, const double* __restrict__ power) {
    const int N = a.N;
    const int64_t per = (int64_t)N * N, total = (int64_t)a.M * per;
    const float sigma = (float)sqrt(power[0] / (double)total / a.snr);
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int m = (int)(i / per);
        const uint32_t pix = (uint32_t)(i - (int64_t)m * per);
        const Philox4 r = philox4x32_10(Philox4{{(uint32_t)m, pix, 0u, 2u}}, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
        a.img[i] += sigma * philox_normal(r);
    }
}

}  // namespace

int64_t synth_images_scratch(int N, int M) { return (int64_t)M * ((N + IMG_ROWS - 1) / IMG_ROWS) + 1025; }

// Slices of all images in one kernel; N <= 128.
hipError_t images_slices(firm_plan p, const float* img, float2* b) {
    switch (p->N) {
        case 8: return launch_slices<8>(p, img, b);
        case 16: return launch_slices<16>(p, img, b);
        case 32: return launch_slices<32>(p, img, b);
        case 64: return launch_slices<64>(p, img, b);
        case 128: return launch_slices<128>(p, img, b);
        default: return hipErrorInvalidValue;
    }
}

// b rows m0 .. m0 + G - 1 from the half spectra of G images.
hipError_t images_gather(firm_plan p, const float2* spec, int G, int m0, float2* b) {
    // eight workgroups per CU, but at least a row for every wavefront
    const int parts = std::min((p->N + IMG_THREADS / 64) / (IMG_THREADS / 64), (8 * p->ncu + G - 1) / G);
    hipLaunchKernelGGL(k_img_gather, dim3((unsigned)G * parts), dim3(IMG_THREADS), 0, p->stream, spec, p->N, p->QPn, p->P,
                       p->rowstart, m0, parts, b);
    return hipGetLastError();
}

// blobs_dev: B x 5 doubles (c, sigma, a sqrt(2 pi) sigma); partials: npart >= synth_images_scratch
// doubles of device scratch.
hipError_t synth_images(firm_plan p, int B, const double* blobs_dev, double snr, uint64_t seed, float* img,
                        double* partials, int64_t npart) {
    const int N = p->N;
    const int64_t blocks = (int64_t)p->M * ((N + IMG_ROWS - 1) / IMG_ROWS);
    if (B > IMG_MAXB || blocks + 1025 > npart) return hipErrorInvalidValue;
    ImgArgs a;
    a.N = N; a.M = p->M; a.B = B; a.c12 = p->c12; a.shifts = p->shifts; a.blobs = blobs_dev; a.img = img;
    a.partials = partials; a.snr = snr; a.seed = seed;
    hipLaunchKernelGGL(k_synth_images, dim3((unsigned)blocks), dim3(IMG_THREADS), 0, p->stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !(snr > 0) || !std::isfinite(snr)) return e;
    double* mid = partials + blocks;
    hipLaunchKernelGGL(k_sum, dim3(1024), dim3(256), 0, p->stream, partials, blocks, mid);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, p->stream, mid, (int64_t)1024, mid + 1024);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_img_noise, dim3(4096), dim3(256), 0, p->stream, a, (const double*)(mid + 1024));
    return hipGetLastError();
}

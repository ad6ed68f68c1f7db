// Non-Cartesian encoding: the voxel x sample contraction for any k-space
// trajectory (the method's non-Cartesian extensibility: Introduction,
// Discussion). Sample k of TR n sits at (kx, ky) cycles per field of view and
//     E[n,k,j] = exp(-2 pi i (ax[n,k] (ix - nx/2) + ay[n,k] (iy - ny/2))),
// ax = kx / nx, ay = ky / ny (FP64 tables). The phase still factors into an x
// and a y part, so per TR the contraction is a dense complex GEMM:
//   forward  s[k] = sum_iy Ey[k,iy] P[k,iy],  P = Ex X^T (nk x ny, K = nx),
//            X[iy,ix] the voxel values of the TR;
//   adjoint  V[iy,ix] = sum_k G[k,iy] H[k,ix],  G = conj(Ey) w, H = conj(Ex),
//            then A_p[j] += mu_p[n,j] V[j] over the TRs of a chunk.
// Both run on the matrix cores as four real products (re re, im im, re im, im
// re), with every phase generated on the fly (argument reduced in FP64,
// sin/cos of the reduced fraction in FP32, neighbours by angle addition).
// MFMA operand layouts (16x16x32): A lane l -> (row l%16, k 8(l/16)..+7), B
// lane l -> (k 8(l/16)..+7, col l%16); D lane l -> (rows 4(l/16)+i, col l%16).
// Measured at 224 x 224, 1120 spokes of 448 samples (FP32 MFMA 16x16x4 tiles
// of 64 samples and 64 x 32 voxels, as before; now): voxel values 0.31 / 0.25
// ms, forward 3.60 / 0.75, adjoint with the trains 5.2 / 1.03 + 0.29 (the
// split-BF16 option's tiles 0.31 + 1.39 / 2.94); errors against the FP64 sums
// of the same trains: J v 3.2e-7 / 2.8e-7, J^H w 5.9e-7 / 4.1e-7.
#include "mrstat_internal.h"

#include <algorithm>
#include <type_traits>

namespace mrstat {

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

// exp(-2 pi i a x) for an FP64 coefficient a and an integer position x: the
// product is reduced to a fraction of a cycle in FP64, then sin and cos of pi
// times twice that fraction in FP32. FINE turns the result by what the
// fraction's rounding to FP32 left out (up to 9e-8): the phases of the forward
// that many products share (offsets, row steps).
template <bool FINE> __device__ __forceinline__ float2 phase_of(double a, int x)
{
    const double t = a * (double)x;
    const double f = -2.0 * (t - rint(t));   // [-1, 1]
    const float h = (float)f;
    float sn, cs;
    sincospif(h, &sn, &cs);
    if constexpr (!FINE) return make_float2(cs, sn);
    const float d = 3.14159265f * (float)(f - (double)h);
    return make_float2(fmaf(-d, sn, cs), fmaf(d, cs, sn));
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}

// ------------------------------------------------------------------------
// Split operands. The products run on v_mfma_f32_16x16x32_f16: each FP32
// operand is written as hi + lo, hi = fp16(v), lo = fp16(v - hi), and the
// product as hi hi + hi lo + lo hi with FP32 accumulation. Operands are first
// scaled by powers of two (phases by 2^14, voxel values so that the largest of
// an image row, samples so that the largest of their TR and coil lies just
// below 2^15), which keeps hi and lo away from fp16's subnormals: 22 bits for
// everything within 2^14 of that largest, a relative error of about 2^-23
// against 2^-24 for FP32 operands, without their K-long serial sums.
// ------------------------------------------------------------------------
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

constexpr float kPhaseScale = 16384.f;

__device__ __forceinline__ void split_h(float a, float b, unsigned& hi, unsigned& lo)
{
    const h2 h = {(_Float16)a, (_Float16)b};
    const h2 l = {(_Float16)(a - (float)h[0]), (_Float16)(b - (float)h[1])};
    hi = __builtin_bit_cast(unsigned, h);
    lo = __builtin_bit_cast(unsigned, l);
}

__device__ __forceinline__ f4 mma(u4 a, u4 b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// 2^e that brings the float of bits m (without its sign) into [2^14, 2^15) (1
// for 0, infinities and NaN; e is bounded so that 2^-e kPhaseScale^-1 stays a
// normal number).
__device__ __forceinline__ float pow2_scale(unsigned m)
{
    const int b = (int)(m >> 23);   // biased exponent
    if (m == 0u || b == 255) return 1.f;
    const int e = min(141 - b, 112);
    return __uint_as_float((unsigned)(e + 127) << 23);
}

// The matrix unit's FP32 sums are off to one side on average, by a part of the
// last place that adds up where sums over many rows or TRs follow. The scale
// takes one sign or the other by row (forward) and TR (adjoint), in the
// Thue-Morse order, which keeps step with no period of phases or pulses. 224 x 224, 1120 spokes of 448 samples: J^H w off by 7.8e-7 without,
// 4.1e-7 with it (FP32 products 5.9e-7); J v with fine phases 3.3e-7 and 3.0e-7
// (3.2e-7).
__device__ __forceinline__ float unbias(float scale, int i) { return __popc(i) & 1 ? -scale : scale; }

// Bits of |x|: their order is that of the magnitudes, NaN above infinity.
__device__ __forceinline__ unsigned mag(float x) { return __float_as_uint(x) & 0x7fffffffu; }

template <int ROR> __device__ __forceinline__ unsigned max_ror(unsigned x)
{
    return max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + ROR, 0xf, 0xf, false));
}
// Maximum over the wave, in every lane.
__device__ __forceinline__ unsigned wave_max(unsigned x)
{
    x = max_ror<1>(max_ror<2>(max_ror<4>(max_ror<8>(x))));
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = max(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return max(b[0], b[1]);
}

template <int ROR> __device__ __forceinline__ float add_ror(float x)
{
    return x + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + ROR, 0xf, 0xf, false));
}
// Sum over the 16 lanes of a row, in every lane.
__device__ __forceinline__ float sum_row16(float x) { return add_ror<8>(add_ror<4>(add_ror<2>(add_ror<1>(x)))); }

typedef __attribute__((address_space(3))) char* lptr;
__device__ __forceinline__ unsigned lds_addr(const void* p) { return (unsigned)(size_t)(lptr)(char*)p; }

// 16 bytes per lane from global memory to LDS (lane l to base + 16 l), past
// the registers.
__device__ __forceinline__ void to_lds16(const void* g, void* wave_base)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)wave_base, 16, 0, 0);
}

// Four MFMA fragments a fixed distance apart. In one block with its wait: with
// loads to LDS in flight, a compiler-made LDS read would wait for all of them.
template <int STEP> __device__ __forceinline__ void read_frag4(u4 (&f)[4], unsigned at)
{
    asm volatile("ds_read_b128 %0, %4\n ds_read_b128 %1, %4 offset:%5\n ds_read_b128 %2, %4 offset:%6\n"
                 "ds_read_b128 %3, %4 offset:%7\n s_waitcnt lgkmcnt(0)"
                 : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3])
                 : "v"(at), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP)
                 : "memory");
}

// ------------------------------------------------------------------------
// Voxel values of the forward, once per product: X[c][n][iy][ix] =
// C_c[j] i rho_j mu0[n,j] (NTRV 1, the signal) or C_c[j] i (rho_j sum_p v_p
// dm_p/dtheta_p + (v3 + i v4) mu0) (NTRV 4: all tangents; 3: without dm/dB1,
// whose direction entry is 0); zero for masked voxels. A wave takes one image
// row of NC_XT TRs (4 columns per lane) and every coil of the pass: scale,
// split, four planes (re hi, re lo, im hi, im lo), zero past nx; the inverse
// scale undoes both operands'. A streaming pass over the trains.
// ------------------------------------------------------------------------
constexpr int NC_XT = 4;

// One TR and coil of split voxel values: four planes of [ny][nx8] fp16, then
// ny floats of inverse scales (16-byte multiple). Records [0, split) lie at
// `a`, the others at `b`.
struct XStore {
    char *a, *b;
    int split, nx8;
    size_t rec;
    __host__ __device__ char* at(int i) const { return i < split ? a + i * rec : b + (i - split) * rec; }
};
__host__ __device__ inline size_t x_planes(int ny, int nx8) { return (size_t)8 * ny * nx8; }

template <int NTRV, bool VEC, typename TT>
__global__ __launch_bounds__(256) void nc_x_kernel(const TT* __restrict__ trains, const float* __restrict__ theta,
                                                   const float* __restrict__ v, const uint8_t* __restrict__ mask,
                                                   const float2* __restrict__ coil, XStore X, int nx, int ny, int nv,
                                                   int T, int n_first, int n_count, int n_coils, int per_block)
{
    const int lane = threadIdx.x & 63;
    const int iy = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (iy >= ny) return;
    const int x0 = 4 * lane;
    const size_t plane = (size_t)T * nv;
    const size_t jrow = (size_t)iy * nx;
    // Four adjacent values of a row, without branches: whole vectors where nx
    // is a multiple of 4 (lanes past the row take its last one), else one by
    // one (columns past the row its last one); both are masked out below.
    auto row4 = [&](const auto* p, auto (&o)[4]) {
        typedef std::remove_const_t<std::remove_reference_t<decltype(*p)>> E;
        if constexpr (VEC) {
            struct __attribute__((packed, aligned(sizeof(E) < 4 ? sizeof(E) : 4))) Q { E e[4]; };
            const Q t = *reinterpret_cast<const Q*>(p + jrow + min(x0, nx - 4));
#pragma unroll
            for (int c = 0; c < 4; ++c) o[c] = t.e[c];
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) o[c] = p[jrow + min(x0 + c, nx - 1)];
        }
    };
    float rr[4], ri[4], w[3][4], nr[4], ni[4];
    bool on[4];
    row4(theta + 3 * (size_t)nv, rr);
    row4(theta + 4 * (size_t)nv, ri);
    if constexpr (NTRV > 1) {
#pragma unroll
        for (int q = 0; q < NTRV - 1; ++q) row4(v + (size_t)q * nv, w[q]);
        row4(v + 3 * (size_t)nv, nr);
        row4(v + 4 * (size_t)nv, ni);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) on[c] = x0 + c < nx;
    if (mask != nullptr) {
        uint8_t mk[4];
        row4(mask, mk);
#pragma unroll
        for (int c = 0; c < 4; ++c) on[c] = on[c] && mk[c] != 0;
    }
    const int nt = min(NC_XT, n_count - (int)blockIdx.y * NC_XT);
    float ar[NC_XT][4], ai[NC_XT][4];   // i (rho t + nu mu0); masked voxels zero whatever their trains hold
#pragma unroll
    for (int k = 0; k < NC_XT; ++k) {
        const int n = n_first + blockIdx.y * NC_XT + (k < nt ? k : 0);
        TT raw[NTRV][4];
        float m[NTRV][4];
#pragma unroll
        for (int q = 0; q < NTRV; ++q) {
            row4(trains + (size_t)n * nv + q * plane, raw[q]);
#pragma unroll
            for (int c = 0; c < 4; ++c) m[q][c] = (float)raw[q][c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float t = 0.f;
#pragma unroll
            for (int q = 1; q < NTRV; ++q) t = fmaf(w[q - 1][c], m[q][c], t);
            if constexpr (NTRV == 1) {
                ar[k][c] = on[c] ? -ri[c] * m[0][c] : 0.f;
                ai[k][c] = on[c] ? rr[c] * m[0][c] : 0.f;
            } else {
                ar[k][c] = on[c] ? -(ri[c] * t + ni[c] * m[0][c]) : 0.f;
                ai[k][c] = on[c] ? rr[c] * t + nr[c] * m[0][c] : 0.f;
            }
        }
    }
    float2 cn[4];   // the next coil's sensitivities
    const int c0 = blockIdx.z * per_block, c1 = min(n_coils, c0 + per_block);
    if (coil != nullptr) row4(coil + (size_t)c0 * nv, cn);
    for (int cl = c0; cl < c1; ++cl) {
        float cr[4], ci[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            cr[c] = coil != nullptr ? cn[c].x : 1.f;
            ci[c] = coil != nullptr ? cn[c].y : 0.f;
        }
        if (coil != nullptr && cl + 1 < c1) row4(coil + (size_t)(cl + 1) * nv, cn);
#pragma unroll
        for (int k = 0; k < NC_XT; ++k) {
            float xr[4], xi[4];
            unsigned mx = 0u;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                xr[c] = cr[c] * ar[k][c] - ci[c] * ai[k][c];
                xi[c] = cr[c] * ai[k][c] + ci[c] * ar[k][c];
                mx = max(mx, max(mag(xr[c]), mag(xi[c])));
            }
            // A value that is not finite makes the row's (and so the TR's) sums so.
            const float sc = unbias(pow2_scale(wave_max(mx)), iy);
            if (k >= nt) continue;
            char* rec = X.at(cl * n_count + blockIdx.y * NC_XT + k);
            if (lane == 0) reinterpret_cast<float*>(rec + x_planes(ny, X.nx8))[iy] = 1.f / (sc * kPhaseScale);
            if (x0 < X.nx8) {
                unsigned o[4][2];
                split_h(sc * xr[0], sc * xr[1], o[0][0], o[1][0]);
                split_h(sc * xr[2], sc * xr[3], o[0][1], o[1][1]);
                split_h(sc * xi[0], sc * xi[1], o[2][0], o[3][0]);
                split_h(sc * xi[2], sc * xi[3], o[2][1], o[3][1]);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<uint2*>(rec + 2 * (((size_t)q * ny + iy) * X.nx8 + x0)) =
                        make_uint2(o[q][0], o[q][1]);
            }
        }
    }
}

// ------------------------------------------------------------------------
// Forward: a block of 8 waves per (TR, 128 samples); wave (ws, wr) owns 32
// samples and NT 16-row tiles of a pass of 32 NT image rows. K runs over the
// columns in steps of 32. Per step the block's Ex (4 columns-of-8 groups x 128
// samples, one sincos per group and the others by angle addition) is made by
// the vector units while the previous step multiplies, and X comes straight
// from memory to the other LDS buffer; both are kept in MFMA fragment order
// (1 KB per 16 x 32 fragment). P_re = Er Xr - Ei Xi, P_im = Er Xi + Ei Xr; the
// epilogue undoes the scales, applies Ey and sums the rows. Blocks are dealt
// so that the sample tiles of a TR share an XCD (X through one L2). Bound by
// the matrix pipe (three products of 2.0e11 flop at 224 x 224, 1120 spokes of
// 448: 0.8 of 2.5 PFLOP/s with the last sample tile half empty) and the LDS
// reads of its operands: 36 fragments per wave and step for 168 MFMA.
// mode 0: out = data - s (and FP64 partials of |out|^2); 1: out = -s; 2: s.
// ------------------------------------------------------------------------
constexpr int NC_MS = 128;   // samples per block

template <int NT>
__global__ __launch_bounds__(512) void nc_fwd_kernel(XStore X, const double* __restrict__ ax,
                                                     const double* __restrict__ ay, const float2* __restrict__ data,
                                                     float2* __restrict__ out, double* __restrict__ red, int mode,
                                                     int nx, int ny, int T, int n_first, int n_count, int n_coils,
                                                     int nk, int KT)
{
    __shared__ u4 As[4][NC_MS / 16][64];
    __shared__ u4 Bs[2][4][2 * NT][64];
    __shared__ float2 part[2][NC_MS];   // row sums per row wave
    __shared__ double rs[8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ws = wave & 3, wr = wave >> 2;
    const int slot = blockIdx.x >> 3;
    const int kt = slot % KT;
    const int rec = (slot / KT) * 8 + (blockIdx.x & 7);   // TR of the pass and coil
    if (rec >= n_count * n_coils) return;
    const int n = n_first + rec % n_count;
    const int k0 = kt * NC_MS, nx8 = X.nx8;
    // Phase generation: this thread's sample and group of 8 columns.
    const int gs = tid & (NC_MS - 1), gg = tid >> 7;
    const double ag = k0 + gs < nk ? ax[(size_t)n * nk + k0 + gs] : 0.0;
    float2 off[8];
#pragma unroll
    for (int m = 1; m < 8; ++m) off[m] = phase_of<true>(ag, m);
    u4 an[4];   // the next step's fragments of this thread
    auto make_a = [&](int s) {
        const int c0 = 32 * s + 8 * gg;
        float2 base = phase_of<false>(ag, c0 - nx / 2);
        base.x *= kPhaseScale;
        base.y *= kPhaseScale;
        float2 e[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            e[m] = m == 0 ? base : cmul(base, off[m]);
            if (c0 + m >= nx) e[m] = make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            unsigned h, l;
            split_h(e[2 * m].x, e[2 * m + 1].x, h, l);
            an[0][m] = h;
            an[1][m] = l;
            split_h(e[2 * m].y, e[2 * m + 1].y, h, l);
            an[2][m] = h;
            an[3][m] = l;
        }
    };
    u4* const aw = &As[0][gs >> 4][(gs & 15) + 16 * gg];
    const _Float16* Xn = reinterpret_cast<const _Float16*>(X.at(rec));
    const float* rinv = reinterpret_cast<const float*>(X.at(rec) + x_planes(ny, nx8));
    const int KS = (nx + 31) / 32, rows = 32 * NT;
    // X fragments of step s and row pass y0 to LDS: rows past ny read the last
    // one (their sums are dropped), columns past nx8 the first (their Ex is 0).
    auto load_b = [&](int y0, int s, int buf) {
        const int col = 32 * s + 8 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int f = wave + 8 * i;   // 8 NT fragments: plane f / (2 NT), row tile f % (2 NT)
            const int q = f / (2 * NT), t = f % (2 * NT);
            const int iy = min(y0 + 16 * t + (lane & 15), ny - 1);
            to_lds16(Xn + ((size_t)q * ny + iy) * nx8 + (col < nx8 ? col : 0), &Bs[buf][q][t][0]);
        }
    };
    const bool active = k0 + 32 * ws < nk;   // whole waves of samples past the end only stage
    const unsigned abase = lds_addr(&As[0][2 * ws][lane]);
    const unsigned bbase = lds_addr(&Bs[0][0][NT * wr][lane]);
    constexpr unsigned BBUF = sizeof(Bs[0]);

    for (int y0 = 0; y0 < ny; y0 += rows) {
        f4 pr[2][NT], pi[2][NT];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) pr[i][t] = pi[i][t] = f4{0.f, 0.f, 0.f, 0.f};
        load_b(y0, 0, 0);
        make_a(0);
        auto steps = [&](auto multiply) {
            for (int s = 0; s < KS; ++s) {
#pragma unroll
                for (int q = 0; q < 4; ++q) aw[q * (NC_MS / 16) * 64] = an[q];
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n s_barrier" ::: "memory");
                if (s + 1 < KS) {
                    load_b(y0, s + 1, (s + 1) & 1);
                    make_a(s + 1);
                }
                if constexpr (decltype(multiply)::value) {
                    u4 a[2][4];
                    read_frag4<(NC_MS / 16) * 1024>(a[0], abase);
                    read_frag4<(NC_MS / 16) * 1024>(a[1], abase + 1024);
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        u4 b[4];
                        read_frag4<2 * NT * 1024>(b, bbase + (s & 1) * BBUF + t * 1024);
                        const u4 nh = b[2] ^ 0x80008000u, nl = b[3] ^ 0x80008000u;   // -Xi
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            pr[i][t] = mma(a[i][0], b[0], pr[i][t]);
                            pi[i][t] = mma(a[i][0], b[2], pi[i][t]);
                            pr[i][t] = mma(a[i][2], nh, pr[i][t]);
                            pi[i][t] = mma(a[i][2], b[0], pi[i][t]);
                            pr[i][t] = mma(a[i][0], b[1], pr[i][t]);
                            pi[i][t] = mma(a[i][0], b[3], pi[i][t]);
                            pr[i][t] = mma(a[i][2], nl, pr[i][t]);
                            pi[i][t] = mma(a[i][2], b[1], pi[i][t]);
                            pr[i][t] = mma(a[i][1], b[0], pr[i][t]);
                            pi[i][t] = mma(a[i][1], b[2], pi[i][t]);
                            pr[i][t] = mma(a[i][3], nh, pr[i][t]);
                            pi[i][t] = mma(a[i][3], b[0], pi[i][t]);
                        }
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n s_barrier" ::: "memory");
            }
        };
        if (!active) {
            steps(std::false_type{});
            continue;
        }
        steps(std::true_type{});
        // s[k] += sum_iy Ey[k,iy] P[k,iy]: the lane's image row of tile t is
        // yl + 16 t, its phases one sincos and steps of 16 rows.
        const int yl = y0 + 16 * NT * wr + (lane & 15);
        float ri[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) ri[t] = yl + 16 * t < ny ? rinv[yl + 16 * t] : 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int kl = 32 * ws + 16 * i + 4 * (lane >> 4) + r;
                const double ayv = k0 + kl < nk ? ay[(size_t)n * nk + k0 + kl] : 0.0;
                float2 ey = phase_of<false>(ayv, yl - ny / 2), sum = make_float2(0.f, 0.f);
                const float2 st = phase_of<true>(ayv, 16);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (yl + 16 * t < ny) {
                        const float2 p = make_float2(ri[t] * pr[i][t][r], ri[t] * pi[i][t][r]);
                        sum.x += ey.x * p.x - ey.y * p.y;
                        sum.y += ey.x * p.y + ey.y * p.x;
                    }
                    if (t + 1 < NT) ey = cmul(ey, st);
                }
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) {
                    sum.x += __shfl_xor(sum.x, o);
                    sum.y += __shfl_xor(sum.y, o);
                }
                if ((lane & 15) == 0) {
                    if (y0 > 0) {
                        sum.x += part[wr][kl].x;
                        sum.y += part[wr][kl].y;
                    }
                    part[wr][kl] = sum;
                }
            }
    }
    __syncthreads();
    double sq = 0.0;
    if (tid < NC_MS && k0 + tid < nk) {
        const size_t idx = ((size_t)(rec / n_count) * T + n) * nk + k0 + tid;
        float2 v = make_float2(part[0][tid].x + part[1][tid].x, part[0][tid].y + part[1][tid].y);
        if (mode == 0) {
            const float2 d = data[idx];
            v = make_float2(d.x - v.x, d.y - v.y);
            sq = (double)v.x * v.x + (double)v.y * v.y;
        } else if (mode == 1) {
            v = make_float2(-v.x, -v.y);
        }
        out[idx] = v;
    }
    if (mode == 0) {
        for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
        if (lane == 0) rs[wave] = sq;
        __syncthreads();
        // (the other waves hold no samples)
        if (tid == 0) red[((size_t)(rec / n_count) * T + n) * KT + kt] = rs[0] + rs[1];
    }
}

// ------------------------------------------------------------------------
// The forward up to 128 columns, and with coils where passes of whole records
// would be short: the values stay FP32 (X[n][j] = i rho_j mu0 or i (rho_j
// sum_p v_p dm_p/dtheta_p + (v3 + i v4) mu0), one record per TR however many
// coils), and each forward block weights, scales and splits what it stages.
// With each row and TR goes its largest value's exponent, and with each row and
// coil that of its weights, from which the scale is made. A group of LX lanes
// takes an image row of XT TRs, lane l columns l + LX c, so rows of any width
// are read in whole segments and narrow ones share a wave.
// ------------------------------------------------------------------------
// Keys: |x| < 2^(b - 126) for the biased exponent b of a row's largest part
// (255: infinite or NaN); b(values) + b(coil weights) bounds the parts of
// their products by 2^(key - 251).
constexpr int kNoWeight = 126;   // of a weight of 1 that is not multiplied

// 2^e that brings values below 2^(key - 251) below 2^15 (e bounded so that
// 2^e and 2^-e / kPhaseScale stay normal numbers).
__device__ __forceinline__ int key_exp(int key) { return max(min(266 - key, 112), -126); }
__device__ __forceinline__ float key_scale(int key) { return __uint_as_float((unsigned)(key_exp(key) + 127) << 23); }
// 2^-e / kPhaseScale.
__device__ __forceinline__ float unscale(int key) { return __uint_as_float((unsigned)(127 - 14 - key_exp(key)) << 23); }
static_assert(kPhaseScale == 1 << 14, "unscale");

template <int NTRV, int XT, typename TT>
__global__ __launch_bounds__(256) void nc_value_kernel(const TT* __restrict__ trains, const float* __restrict__ theta,
                                                       const float* __restrict__ v, const uint8_t* __restrict__ mask,
                                                       const float2* __restrict__ coil, float2* __restrict__ X,
                                                       int* __restrict__ keys, int* __restrict__ ckeys, int nx,
                                                       int ny, int nv, int T, int C, int n_first, int n_end, int LX)
{
    const int xl = threadIdx.x % LX, iy = blockIdx.x * (256 / LX) + threadIdx.x / LX;
    const size_t plane = (size_t)T * nv;
    // Groups past the image repeat its last row, lanes past the row its last
    // column; neither is stored.
    const size_t jrow = (size_t)min(iy, ny - 1) * nx;
    auto row4 = [&](const auto* p, auto (&o)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) o[c] = p[jrow + min(xl + LX * c, nx - 1)];
    };
    float rr[4], ri[4], w[3][4], nr[4], ni[4];
    bool on[4];
    row4(theta + 3 * (size_t)nv, rr);
    row4(theta + 4 * (size_t)nv, ri);
    if constexpr (NTRV > 1) {
#pragma unroll
        for (int q = 0; q < NTRV - 1; ++q) row4(v + (size_t)q * nv, w[q]);
        row4(v + 3 * (size_t)nv, nr);
        row4(v + 4 * (size_t)nv, ni);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) on[c] = xl + LX * c < nx;
    if (mask != nullptr) {
        uint8_t mk[4];
        row4(mask, mk);
#pragma unroll
        for (int c = 0; c < 4; ++c) on[c] = on[c] && mk[c] != 0;
    }
    auto row_max = [&](unsigned a) {   // biased exponent of the row's largest
        for (int o = LX / 2; o > 0; o /= 2) a = max(a, (unsigned)__shfl_xor((int)a, o));
        return (int)(a >> 23);
    };
    if (coil != nullptr && blockIdx.y == 0)
        for (int q = 0; q < C; ++q) {
            float2 cw[4];
            row4(coil + (size_t)q * nv, cw);
            unsigned a = 0u;
#pragma unroll
            for (int c = 0; c < 4; ++c) a = max(a, max(mag(cw[c].x), mag(cw[c].y)));
            const int key = row_max(a);
            if (xl == 0 && iy < ny) ckeys[(size_t)q * ny + iy] = key;
        }
    const int n0 = n_first + blockIdx.y * XT;
    TT m[XT][NTRV][4];
#pragma unroll
    for (int k = 0; k < XT; ++k)
#pragma unroll
        for (int q = 0; q < NTRV; ++q) row4(trains + q * plane + (size_t)min(n0 + k, n_end - 1) * nv, m[k][q]);
#pragma unroll
    for (int k = 0; k < XT; ++k) {
        float2 x[4];
        unsigned a = 0u;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float t = 0.f;
            const float mu = (float)m[k][0][c];
#pragma unroll
            for (int q = 1; q < NTRV; ++q) t = fmaf(w[q - 1][c], (float)m[k][q][c], t);
            if constexpr (NTRV == 1)
                x[c] = make_float2(-ri[c] * mu, rr[c] * mu);
            else
                x[c] = make_float2(-(ri[c] * t + ni[c] * mu), rr[c] * t + nr[c] * mu);
            if (!on[c]) x[c] = make_float2(0.f, 0.f);   // whatever a masked voxel's trains hold
            a = max(a, max(mag(x[c].x), mag(x[c].y)));
        }
        const int n = n0 + k, key = row_max(a);
        if (iy >= ny || n >= n_end) continue;
        if (xl == 0) keys[(size_t)(n - n_first) * ny + iy] = key;
        float2* dst = X + (size_t)n * nv + jrow;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (xl + LX * c < nx) dst[xl + LX * c] = x[c];
    }
}

// ------------------------------------------------------------------------
// Forward from FP32 values: a block of 2 WS waves per (TR, coil, 32 WS
// samples); waves, tiles and products as above. Phases and staged values of a
// step are made by the vector units, held in registers and written to LDS in
// fragment order once the step before has been multiplied; the row phases of
// the sum come from a table. These blocks are short (one to four steps), so
// each piece of code stands once in the loop: a phase is some 50 instructions,
// and a first pass over the code costs as much as the work. (33 x 47, 4 coils,
// 1120 TRs: with the phases inlined at every use 94 us, now 60.)
// ------------------------------------------------------------------------
template <int NT, int WS, bool COIL>
__global__ __launch_bounds__(128 * WS) void nc_fwd_staged_kernel(
    const float2* __restrict__ X, const int* __restrict__ keys, const int* __restrict__ ckeys,
    const float2* __restrict__ coil,
    const double* __restrict__ ax, const double* __restrict__ ay, const float2* __restrict__ data,
    float2* __restrict__ out, double* __restrict__ red, int mode, int nx, int ny, int nv, int T, int C, int n_first,
    int n_end, int nk, int KT)
{
    constexpr int MS = 32 * WS, NTH = 128 * WS;
    constexpr int NI = (NT + WS - 1) / WS;   // pieces of 8 voxel values per thread and step
    constexpr int KP = 20;                   // pitch of the row phases: two samples' 16 rows in different banks
    __shared__ u4 As[4][MS / 16][64];        // after the last step: row phases [MS][KP]
    __shared__ u4 Bs[4][2 * NT][64];
    __shared__ float2 tab[8][MS];    // phases of 1, 2 and 4 columns, of 16, 1, 2, 16 NT (a row wave's) and 64 rows
    __shared__ float2 part[2][MS];   // row sums per row wave
    __shared__ double rs[2 * WS];
    static_assert(sizeof(As) >= KP * MS * sizeof(float2), "row phases");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ws = wave % WS, wr = wave / WS;
    const int slot = blockIdx.x >> 3;
    const int kt = slot % KT, c = slot / KT % C;
    const int n = n_first + slot / (KT * C) * 8 + (blockIdx.x & 7);
    if (n >= n_end) return;
    const int k0 = kt * MS;
    const float2* Xn = X + (size_t)n * nv;
    const float2* Cn = COIL ? coil + (size_t)c * nv : nullptr;
    const int* kn = keys + (size_t)(n - n_first) * ny;
    const int* kc = ckeys + (size_t)c * ny;
    auto row_key = [&](int iy) { return kn[iy] + (coil != nullptr ? kc[iy] : kNoWeight); };
    // Phase generation: this thread's sample and group of 8 columns (or of 4 rows).
    const int gs = tid % MS, gg = tid / MS;
    const bool sample = k0 + gs < nk;
    const double ag = sample ? ax[(size_t)n * nk + k0 + gs] : 0.0, bg = sample ? ay[(size_t)n * nk + k0 + gs] : 0.0;
    const int KS = (nx + 31) / 32, rows = 32 * NT;
    const bool active = k0 + 32 * ws < nk;   // whole waves of samples past the end only stage
    const unsigned abase = lds_addr(&As[0][2 * ws][lane]);
    const unsigned bbase = lds_addr(&Bs[0][NT * wr][lane]);
    u4* const aw = &As[0][gs >> 4][(gs & 15) + 16 * gg];
    float2* const eyt = reinterpret_cast<float2*>(&As[0][0][0]);

    for (int y0 = 0; y0 < ny; y0 += rows) {
        // Piece i: row tile f = e / 64 of the pass, fragment lane e % 64. Rows
        // past ny read the last one (their sums are dropped).
        int brow[NI];
        float bsc[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int e = tid + NTH * i;
            brow[i] = min(y0 + 16 * (e >> 6) + (e & 15), ny - 1);
            bsc[i] = unbias(key_scale(row_key(brow[i])), brow[i]);
        }
        const int yl = y0 + 16 * NT * wr + (lane & 15);   // the lane's image rows in the sums: yl + 16 t
        int rk[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) rk[t] = row_key(min(yl + 16 * t, ny - 1));
        f4 pr[2][NT], pi[2][NT];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) pr[i][t] = pi[i][t] = f4{0.f, 0.f, 0.f, 0.f};
        // Turn s makes step s's operands and multiplies step s - 1's.
#pragma unroll 1
        for (int s = 0; s <= KS; ++s) {
            u4 an[4], bn[NI][4];
            if (s < KS) {
                float2 x[NI][8], cw[NI][8];
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        const int e = tid + NTH * i, c0 = 32 * s + 8 * ((e >> 4) & 3);
                        if (NI * WS > NT && e >= 128 * NT) continue;
                        const float2* p = Xn + (size_t)brow[i] * nx + c0;
                        const float2* q = COIL ? Cn + (size_t)brow[i] * nx + c0 : nullptr;
                        if (c0 + 8 <= nx) {
                            struct __attribute__((packed, aligned(8))) V8 { float2 e[8]; };
                            const V8 t = *reinterpret_cast<const V8*>(p);
#pragma unroll
                            for (int m = 0; m < 8; ++m) x[i][m] = t.e[m];
                            if constexpr (COIL) {
                                const V8 u = *reinterpret_cast<const V8*>(q);
#pragma unroll
                                for (int m = 0; m < 8; ++m) cw[i][m] = u.e[m];
                            }
                        } else {
#pragma unroll
                            for (int m = 0; m < 8; ++m) {
                                x[i][m] = c0 + m < nx ? p[m] : make_float2(0.f, 0.f);
                                if constexpr (COIL) cw[i][m] = c0 + m < nx ? q[m] : make_float2(0.f, 0.f);
                            }
                        }
                    }
                if (y0 == 0 && s == 0) {
#pragma unroll 1
                    for (int h = 0; h < 2; ++h) {
                        const bool col = h == 0 && gg < 3;
                        tab[4 * h + gg][gs] = phase_of<true>(col ? ag : bg, h == 0 ? (col ? 1 << gg : 16) : gg < 2 ? 1 + gg : gg == 2 ? 16 * NT : 64);
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)\n s_barrier" ::: "memory");
                }
                const int c0 = 32 * s + 8 * gg;
                float2 base = phase_of<false>(ag, c0 - nx / 2);
                base.x *= kPhaseScale;
                base.y *= kPhaseScale;
                float2 off[8];
                off[1] = tab[0][gs];
                off[2] = tab[1][gs];
                off[4] = tab[2][gs];
                off[3] = cmul(off[1], off[2]);
                off[5] = cmul(off[4], off[1]);
                off[6] = cmul(off[4], off[2]);
                off[7] = cmul(off[4], off[3]);
                float2 e[8];
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    e[m] = m == 0 ? base : cmul(base, off[m]);
                    if (c0 + m >= nx) e[m] = make_float2(0.f, 0.f);
                }
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    unsigned h, l;
                    split_h(e[2 * m].x, e[2 * m + 1].x, h, l);
                    an[0][m] = h;
                    an[1][m] = l;
                    split_h(e[2 * m].y, e[2 * m + 1].y, h, l);
                    an[2][m] = h;
                    an[3][m] = l;
                }
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        float2 z[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            z[u] = x[i][2 * m + u];
                            if constexpr (COIL) z[u] = cmul(cw[i][2 * m + u], z[u]);
                            z[u].x *= bsc[i];
                            z[u].y *= bsc[i];
                        }
                        unsigned h, l;
                        split_h(z[0].x, z[1].x, h, l);
                        bn[i][0][m] = h;
                        bn[i][1][m] = l;
                        split_h(z[0].y, z[1].y, h, l);
                        bn[i][2][m] = h;
                        bn[i][3][m] = l;
                    }
            }
            if (s > 0) {
                if (active) {
                    u4 a[2][4];
                    read_frag4<(MS / 16) * 1024>(a[0], abase);
                    read_frag4<(MS / 16) * 1024>(a[1], abase + 1024);
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        u4 b[4];
                        read_frag4<2 * NT * 1024>(b, bbase + t * 1024);
                        const u4 nh = b[2] ^ 0x80008000u, nl = b[3] ^ 0x80008000u;   // -Xi
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            pr[i][t] = mma(a[i][0], b[0], pr[i][t]);
                            pi[i][t] = mma(a[i][0], b[2], pi[i][t]);
                            pr[i][t] = mma(a[i][2], nh, pr[i][t]);
                            pi[i][t] = mma(a[i][2], b[0], pi[i][t]);
                            pr[i][t] = mma(a[i][0], b[1], pr[i][t]);
                            pi[i][t] = mma(a[i][0], b[3], pi[i][t]);
                            pr[i][t] = mma(a[i][2], nl, pr[i][t]);
                            pi[i][t] = mma(a[i][2], b[1], pi[i][t]);
                            pr[i][t] = mma(a[i][1], b[0], pr[i][t]);
                            pi[i][t] = mma(a[i][1], b[2], pi[i][t]);
                            pr[i][t] = mma(a[i][3], nh, pr[i][t]);
                            pi[i][t] = mma(a[i][3], b[0], pi[i][t]);
                        }
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n s_barrier" ::: "memory");
            }
            if (s < KS) {
#pragma unroll
                for (int q = 0; q < 4; ++q) aw[q * (MS / 16) * 64] = an[q];
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const int e = tid + NTH * i;
                    if (NI * WS > NT && e >= 128 * NT) continue;
#pragma unroll
                    for (int q = 0; q < 4; ++q) Bs[q][e >> 6][e & 63] = bn[i][q];
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n s_barrier" ::: "memory");
            }
        }
        // Phases of the pass's first 16 rows per sample, 4 rows per thread.
        {
            const float2 e = phase_of<true>(bg, y0 + 4 * gg - ny / 2), r1 = tab[4][gs], r2 = tab[5][gs];
            float2* t = &eyt[KP * gs + 4 * gg];
            t[0] = e;
            t[1] = cmul(e, r1);
            t[2] = cmul(e, r2);
            t[3] = cmul(e, cmul(r1, r2));
        }
        __syncthreads();
        // s[k] += sum_iy Ey[k,iy] P[k,iy] over the lane's image rows.
        if (active) {
            float ri[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) ri[t] = unbias(unscale(rk[t]), yl + 16 * t);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int kl = 32 * ws + 16 * i + 4 * (lane >> 4) + r;
                    float2 ey = eyt[KP * kl + (lane & 15)], sum = make_float2(0.f, 0.f);
                    if (wr > 0) ey = cmul(ey, tab[6][kl]);
                    const float2 st = tab[3][kl];
                    float2 ey4 = ey;   // a step's error grows with each use: at most three
                    if constexpr (NT > 4) ey4 = cmul(ey, tab[7][kl]);
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        if (yl + 16 * t < ny) {
                            const float2 p = make_float2(ri[t] * pr[i][t][r], ri[t] * pi[i][t][r]);
                            sum.x += ey.x * p.x - ey.y * p.y;
                            sum.y += ey.x * p.y + ey.y * p.x;
                        }
                        if (t + 1 < NT) ey = t == 3 ? ey4 : cmul(ey, st);
                    }
                    sum.x = sum_row16(sum.x);
                    sum.y = sum_row16(sum.y);
                    if ((lane & 15) == 0) {
                        if (y0 > 0) {
                            sum.x += part[wr][kl].x;
                            sum.y += part[wr][kl].y;
                        }
                        part[wr][kl] = sum;
                    }
                }
        }
        if (y0 + rows < ny) __syncthreads();   // the next pass writes As
    }
    __syncthreads();
    double sq = 0.0;
    if (tid < MS && sample) {
        const size_t idx = ((size_t)c * T + n) * nk + k0 + tid;
        float2 v = make_float2(part[0][tid].x + part[1][tid].x, part[0][tid].y + part[1][tid].y);
        if (mode == 0) {
            const float2 d = data[idx];
            v = make_float2(d.x - v.x, d.y - v.y);
            sq = (double)v.x * v.x + (double)v.y * v.y;
        } else if (mode == 1) {
            v = make_float2(-v.x, -v.y);
        }
        out[idx] = v;
    }
    if (mode == 0) {
        for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
        if (lane == 0) rs[wave] = sq;
        __syncthreads();
        // (waves from 64 samples on hold none)
        if (tid == 0) red[((size_t)c * T + n) * KT + kt] = MS > 64 ? rs[0] + rs[1] : rs[0];
    }
}

// ------------------------------------------------------------------------
// Adjoint, V[n][j] = sum_c conj(C_c[j]) sum_k conj(E[n,k,j]) w_c[n,k]: a block
// of 8 waves per (TR, 128 columns, 32 NT rows); wave (ws, wr) owns 32 columns
// and NT 16-row tiles, K runs over the samples in steps of 32. Both operands
// are phases: H[k,ix] = conj(Ex) and G[k,iy] = conj(Ey) w (w scaled so that
// its largest value of the TR lies in [2^10, 2^11)). A thread makes one
// sample's values at 8 consecutive columns and 2 NT consecutive rows: two
// sincos, the others as products with the phases of 1 to 7 positions on, whose
// factors (1, 2 and 4 on) come from a table made a step ahead; it does so
// while the step before multiplies, holding the split values in registers.
// They lie in LDS as [plane][sample][position], written 16 bytes at a time
// and read as MFMA fragments by the transposing LDS load (each 16 lanes: 4
// samples x 16 positions). Bound by the matrix pipe and, nearly as long, the
// vector units that make and split the phases.
// ------------------------------------------------------------------------
constexpr int NCA_TX = 128;   // columns per block

typedef short s4 __attribute__((ext_vector_type(4)));

// Fragment (16 positions, 32 samples: lane l position l % 16, samples
// 8 (l / 16)..+7) from rows of ROW bytes per sample; `at` is this lane's
// address for samples 8 (l / 16) + (l % 16) / 4.
template <int ROW> __device__ __forceinline__ u4 read_tr(const char* at)
{
    typedef __attribute__((address_space(3))) s4* lp;
    const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(lptr)(char*)at);
    const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(lptr)(char*)(at + 4 * ROW));
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    return u4{x.x, x.y, y.x, y.y};
}

template <int NT>
__global__ __launch_bounds__(512) void nc_adj_kernel(const float2* __restrict__ coil, const double* __restrict__ ax,
                                                     const double* __restrict__ ay, const float2* __restrict__ w,
                                                     float2* __restrict__ V, int nx, int ny, int nv, int T, int nk,
                                                     int C, int ntx, int tiles)
{
    constexpr int NR = 2 * NT;                  // rows per thread, 32 NT per block
    constexpr int AROW = 2 * NCA_TX + 32;       // bytes per sample: 8 words past a multiple of 64 banks, so the
    constexpr int BROW = 64 * NT + 32;          // samples of a write or of a transposing read differ in banks
    __shared__ __attribute__((aligned(16))) char Hs[4][32][AROW];
    __shared__ __attribute__((aligned(16))) char Gs[4][32][BROW];
    __shared__ float2 tab[2][6][32];            // phases of 1, 2, 4 columns / rows per sample
    __shared__ unsigned wmax[8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ws = wave & 3, wr = wave >> 2;
    const int slot = blockIdx.x >> 3;
    const int tile = slot % tiles;
    const int n = (slot / tiles) * 8 + (blockIdx.x & 7);
    if (n >= T) return;
    const int x0 = (tile % ntx) * NCA_TX, y0 = (tile / ntx) * 32 * NT;
    const bool active = x0 + 32 * ws < nx;
    const int ks = tid & 31, pg = tid >> 5;     // this thread's sample of a step and group of positions
    const double* axn = ax + (size_t)n * nk;
    const double* ayn = ay + (size_t)n * nk;
    const int KS = (nk + 31) / 32;

    auto make_tab = [&](int s, int buf) {
        if (tid < 192) {
            const int k = 32 * s + (tid & 31), q = tid >> 5;   // q: x1 x2 x4 y1 y2 y4
            const double a = k < nk ? (q < 3 ? axn[k] : ayn[k]) : 0.0;
            tab[buf][q][tid & 31] = phase_of<false>(-a, 1 << (q % 3));
        }
    };
    for (int c = 0; c < C; ++c) {
        const float2* wn = w + ((size_t)c * T + n) * nk;
        // Scale of this TR's samples.
        unsigned mx = 0u;
        for (int k = tid; k < nk; k += 512) {
            const float2 v = wn[k];
            mx = max(mx, max(mag(v.x), mag(v.y)));
        }
        mx = wave_max(mx);
        __syncthreads();   // the previous coil's scale and tables have been read
        if (lane == 0) wmax[wave] = mx;
        make_tab(0, 0);
        make_tab(1, 1);
        __syncthreads();
        mx = wmax[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) mx = max(mx, wmax[i]);
        const float sc = unbias(pow2_scale(mx), n);

        unsigned hv[4][4], gv[4][NT];   // split values: [plane][pair of positions]
        auto make = [&](int s) {
            const int k = 32 * s + ks;
            const double ak = k < nk ? axn[k] : 0.0, bk = k < nk ? ayn[k] : 0.0;
            float2 wv = k < nk ? wn[k] : make_float2(0.f, 0.f);
            wv.x *= sc;
            wv.y *= sc;
            auto line = [&](float2 base, const float2 (&t)[8], auto& out, auto count, int first) {
                constexpr int N = decltype(count)::value;   // positions of this line, even
#pragma unroll
                for (int m = 0; m < N; m += 2) {
                    const float2 e0 = m == 0 ? base : cmul(base, t[m]), e1 = cmul(base, t[m + 1]);
                    split_h(e0.x, e1.x, out[0][first + m / 2], out[1][first + m / 2]);
                    split_h(e0.y, e1.y, out[2][first + m / 2], out[3][first + m / 2]);
                }
            };
            auto steps = [&](int q, float2 (&t)[8]) {
                t[1] = tab[s & 1][q][ks];
                t[2] = tab[s & 1][q + 1][ks];
                t[4] = tab[s & 1][q + 2][ks];
                t[3] = cmul(t[1], t[2]);
                t[5] = cmul(t[4], t[1]);
                t[6] = cmul(t[4], t[2]);
                t[7] = cmul(t[4], t[3]);
            };
            float2 t[8];
            steps(0, t);
            float2 base = phase_of<false>(-ak, x0 + 8 * pg - nx / 2);
            base.x *= kPhaseScale;
            base.y *= kPhaseScale;
            line(base, t, hv, std::integral_constant<int, 8>{}, 0);
            steps(3, t);
            base = cmul(phase_of<false>(-bk, y0 + NR * pg - ny / 2), wv);
            if constexpr (NR <= 8) {
                line(base, t, gv, std::integral_constant<int, NR>{}, 0);
            } else {
                line(base, t, gv, std::integral_constant<int, 8>{}, 0);
                line(cmul(base, cmul(t[4], t[4])), t, gv, std::integral_constant<int, NR - 8>{}, 4);
            }
        };
        f4 vr[2][NT], vi[2][NT];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) vr[i][t] = vi[i][t] = f4{0.f, 0.f, 0.f, 0.f};
        // This lane's part of a transposing read: sample 8 (l / 16) + (l % 16) / 4, positions 4 (l % 4)..+3.
        const int rk = 8 * (lane >> 4) + ((lane & 15) >> 2), rp = 4 * (lane & 3);
        const char* ha = &Hs[0][rk][2 * (32 * ws + rp)];
        const char* ga = &Gs[0][rk][2 * (16 * NT * wr + rp)];
        make(0);
        auto run = [&](auto multiply) {
            for (int s = 0; s < KS; ++s) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    *reinterpret_cast<u4*>(&Hs[q][ks][16 * pg]) = u4{hv[q][0], hv[q][1], hv[q][2], hv[q][3]};
#pragma unroll
                    for (int m = 0; m < NT; ++m) *reinterpret_cast<unsigned*>(&Gs[q][ks][4 * (NT * pg + m)]) = gv[q][m];
                }
                __syncthreads();
                if (s + 1 < KS) make(s + 1);
                if constexpr (decltype(multiply)::value) {
                    u4 h[2][4];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q) h[i][q] = read_tr<AROW>(ha + q * 32 * AROW + 32 * i);
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        u4 g[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) g[q] = read_tr<BROW>(ga + q * 32 * BROW + 32 * t);
                        const u4 nh = g[2] ^ 0x80008000u, nl = g[3] ^ 0x80008000u;   // -Gi
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            vr[i][t] = mma(h[i][0], g[0], vr[i][t]);
                            vi[i][t] = mma(h[i][0], g[2], vi[i][t]);
                            vr[i][t] = mma(h[i][2], nh, vr[i][t]);
                            vi[i][t] = mma(h[i][2], g[0], vi[i][t]);
                            vr[i][t] = mma(h[i][0], g[1], vr[i][t]);
                            vi[i][t] = mma(h[i][0], g[3], vi[i][t]);
                            vr[i][t] = mma(h[i][2], nl, vr[i][t]);
                            vi[i][t] = mma(h[i][2], g[1], vi[i][t]);
                            vr[i][t] = mma(h[i][1], g[0], vr[i][t]);
                            vi[i][t] = mma(h[i][1], g[2], vi[i][t]);
                            vr[i][t] = mma(h[i][3], nh, vr[i][t]);
                            vi[i][t] = mma(h[i][3], g[0], vi[i][t]);
                        }
                    }
                }
                __syncthreads();
                if (s + 2 < KS) make_tab(s + 2, s & 1);   // read after the next step's first barrier
            }
        };
        if (active) run(std::true_type{});
        else run(std::false_type{});

        if (!active) continue;
        const float inv = 1.f / (sc * kPhaseScale);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int iy = y0 + 16 * (NT * wr + t) + (lane & 15);
                const int ix = x0 + 32 * ws + 16 * i + 4 * (lane >> 4);
                if (iy >= ny) continue;
                const size_t j = (size_t)iy * nx + ix;
                float2* dst = V + (size_t)n * nv + j;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (ix + r >= nx) break;
                    float2 v = make_float2(inv * vr[i][t][r], inv * vi[i][t][r]);
                    if (coil != nullptr) {   // conj(C_c) v, summed over the coils
                        const float2 cc = coil[(size_t)c * nv + j + r];
                        v = make_float2(cc.x * v.x + cc.y * v.y, cc.x * v.y - cc.y * v.x);
                        if (c > 0) {
                            const float2 old = dst[r];
                            v.x += old.x;
                            v.y += old.y;
                        }
                    }
                    dst[r] = v;
                }
            }
    }
}

// ------------------------------------------------------------------------
// A_p[j] = sum_n mu_p[n,j] V[n][j] over the TRs of a chunk, two voxels per
// thread: chunk partials apart[chunk][2 p + (re, im)][j] with 8 planes per
// chunk (2 for the m train alone), the layout of the Cartesian adjoint, so the
// same gradient assembly follows. A streaming pass over V and the trains.
// ------------------------------------------------------------------------
template <int NTR, typename TT>
__global__ __launch_bounds__(256) void nc_acc_kernel(const TT* __restrict__ trains, const float2* __restrict__ V,
                                                     const uint8_t* __restrict__ mask, float* __restrict__ apart,
                                                     int nv, int T, int per)
{
    typedef TT V2 __attribute__((ext_vector_type(2), aligned(sizeof(TT))));
    typedef float F4 __attribute__((ext_vector_type(4), aligned(8)));
    constexpr int NB = 4;   // TRs whose loads are issued together
    // The last thread of an odd image takes its last two voxels and stores the
    // second one (one voxel: reads it twice).
    const int j0 = 2 * (blockIdx.x * 256 + threadIdx.x);
    if (j0 >= nv) return;
    const int j = min(j0, max(nv - 2, 0));
    const bool pair = nv > 1;
    const int n0 = blockIdx.y * per, n1 = min(T, n0 + per);
    const size_t plane = (size_t)T * nv;
    float acc[2][NTR][2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int p = 0; p < NTR; ++p) acc[e][p][0] = acc[e][p][1] = 0.f;
    for (int n = n0; n < n1; n += NB) {
        F4 v[NB];
        V2 m[NB][NTR];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const size_t at = (size_t)min(n + b, n1 - 1) * nv + j;
            if (pair) {
                v[b] = *reinterpret_cast<const F4*>(V + at);
#pragma unroll
                for (int p = 0; p < NTR; ++p) m[b][p] = *reinterpret_cast<const V2*>(trains + p * plane + at);
            } else {
                v[b] = F4{V[at].x, V[at].y, V[at].x, V[at].y};
#pragma unroll
                for (int p = 0; p < NTR; ++p) m[b][p] = V2{trains[p * plane + at], trains[p * plane + at]};
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (n + b >= n1) break;
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int p = 0; p < NTR; ++p) {
                    const float mu = (float)m[b][p][e];
                    acc[e][p][0] = fmaf(mu, v[b][2 * e], acc[e][p][0]);
                    acc[e][p][1] = fmaf(mu, v[b][2 * e + 1], acc[e][p][1]);
                }
        }
    }
    constexpr int planes = NTR == 1 ? 2 : 8;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        if (j + e < j0 || (e == 1 && !pair)) continue;
        const bool on = mask == nullptr || mask[j + e] != 0;
        float* dst = apart + (size_t)blockIdx.y * planes * nv + j + e;
#pragma unroll
        for (int p = 0; p < NTR; ++p)
#pragma unroll
            for (int k = 0; k < 2; ++k) dst[(size_t)(2 * p + k) * nv] = on ? acc[e][p][k] : 0.f;
    }
}

template <typename TT>
hipError_t x_launch(const Dims& d, int mode_y, const TT* trains, const float* theta, const float* v,
                    const uint8_t* mask, const float2* coil, const XStore& X, int n_first, int n_count, int n_coils,
                    hipStream_t s)
{
    // A block takes all coils of its TRs, or one where that leaves CUs idle.
    dim3 grid(ceil_div(d.ny, 4), ceil_div(n_count, NC_XT));
    const int per = (int)(grid.x * grid.y) < 512 ? 1 : n_coils;
    grid.z = ceil_div(n_coils, per);
#define NC_X(N)                                                                                                    \
    if (d.nx % 4 == 0)                                                                                            \
        nc_x_kernel<N, true, TT><<<grid, 256, 0, s>>>(trains, theta, v, mask, coil, X, d.nx, d.ny, d.nv, d.T,     \
                                                      n_first, n_count, n_coils, per);                            \
    else                                                                                                          \
        nc_x_kernel<N, false, TT><<<grid, 256, 0, s>>>(trains, theta, v, mask, coil, X, d.nx, d.ny, d.nv, d.T,    \
                                                       n_first, n_count, n_coils, per)
    switch (mode_y) {
    case 0: NC_X(1); break;
    case 1: NC_X(4); break;
    case 3: NC_X(3); break;
    default: return hipErrorInvalidValue;
    }
#undef NC_X
    return hipGetLastError();
}

template <typename TT>
hipError_t acc_launch(const Dims& d, int ntr, int chunks, const TT* trains, const float2* V, const uint8_t* mask,
                      float* apart, hipStream_t s)
{
    // Exactly `chunks` chunks (the count the gradient assembly sums), each
    // holding at least one TR.
    const int per = ceil_div(d.T, chunks);
    if (chunks < 1 || ceil_div(d.T, per) != chunks) return hipErrorInvalidValue;
    const dim3 grid(ceil_div(d.nv, 512), chunks);
    if (ntr == 1)
        nc_acc_kernel<1, TT><<<grid, 256, 0, s>>>(trains, V, mask, apart, d.nv, d.T, per);
    else if (ntr == 3)
        nc_acc_kernel<3, TT><<<grid, 256, 0, s>>>(trains, V, mask, apart, d.nv, d.T, per);
    else
        nc_acc_kernel<4, TT><<<grid, 256, 0, s>>>(trains, V, mask, apart, d.nv, d.T, per);
    return hipGetLastError();
}

// 16-row tiles per wave: 32 NT rows per pass (or block), at most 224, the
// fewest that divide the image's rows into equal passes.
int row_tiles(int ny) { return ceil_div(ny, 32 * ceil_div(ny, 224)); }

// How the forward's TRs and coils go in passes that the workspace holds: the
// main store (T nv 8 bytes; rows padded to 8 columns and the scales may leave
// a few TRs out) and the small one (nv 512 bytes).
struct Passes {
    XStore X;
    int coils, trs;   // per pass
};
Passes fwd_passes(const Dims& d, void* main_store, void* small)
{
    Passes p;
    p.X.nx8 = ceil_div(d.nx, 8) * 8;
    p.X.rec = x_planes(d.ny, p.X.nx8) + (size_t)(4 * d.ny + 15) / 16 * 16;
    p.X.a = static_cast<char*>(main_store);
    p.X.b = static_cast<char*>(small);
    p.X.split = (int)((size_t)d.T * d.nv * 8 / p.X.rec);
    const int cap = p.X.split + (int)((size_t)d.nv * 512 / p.X.rec);
    p.coils = std::min(d.C, cap);
    p.trs = std::min(d.T, cap / p.coils);
    return p;
}

int fwd_grid(int nk, int recs) { return 8 * ceil_div(nk, NC_MS) * ceil_div(recs, 8); }

// 16-row tiles per wave of the adjoint: as above while its blocks (one per TR,
// 128 columns and 32 NT rows) fill the 256 CUs, else fewer rows per block where
// that is faster. A block takes the time of its phases (as long as three row
// tiles) and of its tiles; two on a CU take 1.4 times one's time, more in
// proportion. J^H w in us, 64 TRs, the most rows / as chosen: 128 x 128, 4 coils,
// 128 samples 162 / 93; 24 x 200, 8 coils, 48 samples 257 / 118; 224 x 224, one
// coil, 448 samples 149 / 108; 250 TRs and more keep the most rows.
int adj_tiles(const Dims& d)
{
    int best = 0;
    long t_best = 0;
    for (int passes = ceil_div(d.ny, 224); passes <= ceil_div(d.ny, 32); ++passes) {
        const int nt = ceil_div(d.ny, 32 * passes);
        const int k = ceil_div(d.T * ceil_div(d.nx, NCA_TX) * ceil_div(d.ny, 32 * nt), 256);
        const long t = (3 + nt) * (k == 1 ? 10 : 7 * k);
        if (best == 0 || 10 * t < 9 * t_best) t_best = t, best = nt;
    }
    return best;
}

// How the forward takes a problem: values split once (`split`) or staged from
// FP32, sample waves per block, 16-row tiles per wave. J v in us, 4 coils, 1120
// TRs unless said, 1 / 2 / 4 sample waves staged / split:
//   split: its records are per TR and coil, T / n_coils TRs per launch, and its
//     rows take a wave each, whatever their width: 24 x 24, 48 samples 62 / 71 /
//     115 / 200; 101 x 90, 202 samples 838 / 742 / 620 / 704. From 129 columns on
//     the splitting that every staged block repeats costs more (224 x 224, 448
//     samples, one coil 1487 / 1155 / 1287 / 1016; 250 TRs 1505 / 1061 / 1061 /
//     828), unless its launches leave CUs idle (160 x 160, 160 samples, 64 TRs 120
//     / 99 / 115 / 127) or its rows fill a fraction of a block (200 x 24, 200
//     samples, 250 TRs 120 / 153 / 155 / 194). Just below, with coils, it needs
//     full launches (128 x 128, 2 coils, 256 samples, 560 TRs 257 by four, 235).
//   one wave: few rows or samples (above; 24 x 200, 24 samples 157 / 187 / 304).
//   two or four: the one that pads rows and samples to less; in between two for
//     one coil (128 x 128, 128 samples 238 / 179 / 188), and with coils (whose
//     blocks hold at most 32 rows per wave) four from two row passes of two on
//     (128 x 128, 256 samples, 250 TRs 339 / 250 / 220; 64 x 64 242 / 182 / 212).
struct FwdPlan {
    bool split;
    int ws, nt, kt;   // kt: sample tiles
};
FwdPlan fwd_plan(const Dims& d)
{
    auto tiles = [&](int most) { return ceil_div(d.ny, 32 * ceil_div(d.ny, most)); };
    auto padded = [&](int ws, int most) {   // samples times rows, the last tiles' padding counted
        return (long)ceil_div(d.nk, 32 * ws) * ws * ceil_div(d.ny, 32 * tiles(most)) * tiles(most);
    };
    FwdPlan p;
    const int kt4 = ceil_div(d.nk, NC_MS), fill = d.T * kt4;   // blocks of a launch of the split form, with coils
    p.split = d.nx > 128 ? d.C == 1 || (d.ny > 32 && fill >= 256)
                         : d.nx > 112 && d.ny > 112 && d.C > 1 && kt4 > 1 && fill >= 1024;
    if (p.split)
        p.ws = 4;
    else if (d.ny <= 32 || (d.nk <= 32 && (d.C > 1 || d.ny <= 64)))
        p.ws = 1;
    else if (d.C > 1)
        p.ws = d.ny > 64 && padded(4, 128) <= padded(2, 64) ? 4 : 2;
    else
        p.ws = 10 * padded(4, 224) < 9 * padded(2, 128) ? 4 : 2;
    if (ceil_div(d.nk, 32 * p.ws) > d.nx) p.ws = 4;   // the room for the partial sums of f
    p.nt = p.split ? row_tiles(d.ny) : tiles(d.C > 1 ? 32 * p.ws : p.ws == 4 ? 224 : 64 * p.ws);
    p.kt = ceil_div(d.nk, 32 * p.ws);
    return p;
}

template <typename TT>
hipError_t value_launch(const Dims& d, int mode_y, const TT* trains, const float* theta, const float* v,
                        const uint8_t* mask, const float2* coil, float2* X, int* keys, int* ckeys, int n_first,
                        int n_end, hipStream_t s)
{
    int LX = 1;
    while (4 * LX < d.nx) LX *= 2;
    // One TR per group while four leave CUs idle.
    const int gx = ceil_div(d.ny, 256 / LX), nt = n_end - n_first;
    const bool few = gx * ceil_div(nt, 4) < 1024;
    const dim3 grid(gx, few ? nt : ceil_div(nt, 4));
#define NC_V2(N, XT)                                                                                               \
    nc_value_kernel<N, XT, TT><<<grid, 256, 0, s>>>(trains, theta, v, mask, coil, X, keys, ckeys, d.nx, d.ny,      \
                                                    d.nv, d.T, d.C, n_first, n_end, LX)
#define NC_V(N)                                                                                                    \
    if (few) NC_V2(N, 1);                                                                                         \
    else NC_V2(N, 4)
    switch (mode_y) {
    case 0: NC_V(1); break;
    case 1: NC_V(4); break;
    case 3: NC_V(3); break;
    default: return hipErrorInvalidValue;
    }
#undef NC_V
#undef NC_V2
    return hipGetLastError();
}

template <int WS, bool COIL>
hipError_t staged_launch(const Dims& d, const FwdPlan& p, const float2* X, const int* keys, const int* ckeys,
                         const float2* coil, const double* ax, const double* ay, const float2* data, float2* out,
                         double* red, int mode_x, int n_first, int n_end, hipStream_t s)
{
    constexpr int MOST = COIL ? WS : WS == 4 ? 7 : 2 * WS;   // of 16-row tiles per wave
    const int grid = 8 * p.kt * d.C * ceil_div(n_end - n_first, 8);
#define NC_FWD(N)                                                                                                  \
    if constexpr (N <= MOST)                                                                                      \
        if (p.nt == N) {                                                                                          \
            nc_fwd_staged_kernel<N, WS, COIL><<<grid, 128 * WS, 0, s>>>(X, keys, ckeys, coil, ax, ay, data, out,   \
                                                                        red, mode_x, d.nx, d.ny, d.nv, d.T, d.C,   \
                                                                        n_first, n_end, d.nk, p.kt);               \
            return hipGetLastError();                                                                             \
        }
    NC_FWD(1) NC_FWD(2) NC_FWD(3) NC_FWD(4) NC_FWD(5) NC_FWD(6) NC_FWD(7)
#undef NC_FWD
    return hipErrorInvalidValue;
}

}  // namespace

int nc_adj_chunks(const Dims& d)
{
    // Enough blocks (512 voxels each) to fill the chip with the streaming pass
    // over V and the trains, with partial sums kept modest (chunks x 8 floats
    // per voxel, at most 32 chunks and, for narrow images, 512 per 32 x 64
    // voxels).
    const int tiles = ceil_div(d.nx, 32) * ceil_div(d.ny, 64);
    return std::min({ceil_div(1024, ceil_div(d.nv, 512)), ceil_div(512, tiles), 32, d.T});
}

int nc_fwd_blocks(const Dims& d) { return d.C * d.T * fwd_plan(d).kt; }

hipError_t launch_nc_fwd(const Dims& d, int enc, int mode_y, int mode_x, const void* trains, bool f16,
                         const float* theta, const float* v, const float2* coil, const uint8_t* mask,
                         const double* ax, const double* ay, void* X, void* small, const float2* data, float2* out,
                         double* red, int* nred, hipStream_t s)
{
    if (d.nx > 256 || (enc != 0 && enc != 1)) return hipErrorInvalidValue;
    const FwdPlan plan = fwd_plan(d);
    if (nred) *nred = nc_fwd_blocks(d);
    if (!plan.split) {
        float2* const Xv = static_cast<float2*>(X);
        int* const keys = static_cast<int*>(small);
        const int trs = std::min(d.T, 128 * d.nx - d.C);   // TRs whose keys fit beside the coils'
        int* const ckeys = keys + (size_t)trs * d.ny;
        for (int n = 0; n < d.T; n += trs) {
            const int end = std::min(d.T, n + trs);
            hipError_t e = f16 ? value_launch(d, mode_y, static_cast<const _Float16*>(trains), theta, v, mask, coil, Xv,
                                              keys, ckeys, n, end, s)
                               : value_launch(d, mode_y, static_cast<const float*>(trains), theta, v, mask, coil, Xv,
                                              keys, ckeys, n, end, s);
            if (e != hipSuccess) return e;
#define NC_FWD2(W)                                                                                                 \
    (coil != nullptr ? staged_launch<W, true>(d, plan, Xv, keys, ckeys, coil, ax, ay, data, out, red, mode_x, n, end, s) \
                     : staged_launch<W, false>(d, plan, Xv, keys, ckeys, coil, ax, ay, data, out, red, mode_x, n, end, s))
            e = plan.ws == 1 ? NC_FWD2(1) : plan.ws == 2 ? NC_FWD2(2) : NC_FWD2(4);
#undef NC_FWD2
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const Passes p = fwd_passes(d, X, small);
    const int KT = plan.kt, nt = plan.nt;
    for (int c = 0; c < d.C; c += p.coils) {
        const int nc = std::min(p.coils, d.C - c);
        const float2* cc = coil == nullptr ? nullptr : coil + (size_t)c * d.nv;
        const size_t at = (size_t)c * d.T * d.nk;
        for (int n = 0; n < d.T; n += p.trs) {
            const int cnt = std::min(p.trs, d.T - n);
            hipError_t e = f16 ? x_launch(d, mode_y, static_cast<const _Float16*>(trains), theta, v, mask, cc, p.X, n,
                                          cnt, nc, s)
                               : x_launch(d, mode_y, static_cast<const float*>(trains), theta, v, mask, cc, p.X, n,
                                          cnt, nc, s);
            if (e != hipSuccess) return e;
            const int grid = fwd_grid(d.nk, cnt * nc);
#define NC_FWD(N)                                                                                                  \
    case N:                                                                                                       \
        nc_fwd_kernel<N><<<grid, 512, 0, s>>>(p.X, ax, ay, data == nullptr ? nullptr : data + at, out + at,       \
                                              red == nullptr ? nullptr : red + (size_t)c * d.T * KT, mode_x, d.nx, d.ny, d.T, n,  \
                                              cnt, nc, d.nk, KT);                                                 \
        break;
            switch (nt) {
                NC_FWD(1) NC_FWD(2) NC_FWD(3) NC_FWD(4) NC_FWD(5) NC_FWD(6) NC_FWD(7)
            default: return hipErrorInvalidValue;
            }
#undef NC_FWD
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t launch_nc_adj(const Dims& d, int enc, int ntr, int chunks, const void* trains, bool f16,
                         const float2* coil, const uint8_t* mask, const double* ax, const double* ay,
                         const float2* w, float2* V, float* apart, hipStream_t s)
{
    if (enc != 0 && enc != 1) return hipErrorInvalidValue;
    const int ntx = ceil_div(d.nx, NCA_TX), nt = adj_tiles(d);
    const int tiles = ntx * ceil_div(d.ny, 32 * nt);
    const unsigned grid = 8u * tiles * ceil_div(d.T, 8);
#define NC_ADJ(N)                                                                                                  \
    case N: nc_adj_kernel<N><<<grid, 512, 0, s>>>(coil, ax, ay, w, V, d.nx, d.ny, d.nv, d.T, d.nk, d.C, ntx, tiles); break;
    switch (nt) {
        NC_ADJ(1) NC_ADJ(2) NC_ADJ(3) NC_ADJ(4) NC_ADJ(5) NC_ADJ(6) NC_ADJ(7)
    default: return hipErrorInvalidValue;
    }
#undef NC_ADJ
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return f16 ? acc_launch(d, ntr, chunks, static_cast<const _Float16*>(trains), V, mask, apart, s)
               : acc_launch(d, ntr, chunks, static_cast<const float*>(trains), V, mask, apart, s);
}

}  // namespace mrstat

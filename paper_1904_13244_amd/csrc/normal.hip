// The CG product q = Re(J^H J d) of a Cartesian single-coil context in one
// pass over the trains. The readout phases satisfy Ex^H Ex = n_read I on the
// library's grid ((k - nk/2)(ix - nx/2)/nk with nk >= nx: a geometric sum over
// whole periods), so between J d and J^H the x-stage is a factor,
//     W[n,ix] = (Ex^H (-Ex U))[n,ix] = -n_read U[n,ix],
// and the product falls apart into image columns: per TR and column
//     U = sum_iy Ey[n,iy] i (rho a + nu mu_0),  a = v0 mu_1 + v1 mu_2 + v2 mu_3,
//     A_p[j] += mu_p[n,j] conj(Ey[n,iy]) W.
// A block that holds all rows of a few columns can therefore use each train
// value for both halves while it is in registers.
#include "mrstat_internal.h"

#include <algorithm>

namespace mrstat {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int NX = 16;   // image columns per block

// Four adjacent columns of a train row; rows start anywhere (nx need not be a
// multiple of 4), so the vectors are aligned to their elements only.
template <typename TT> struct TrainVec;
template <> struct TrainVec<float> { typedef float T __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct TrainVec<_Float16> { typedef _Float16 T __attribute__((ext_vector_type(4), aligned(2))); };
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// a + b after exchanging the upper 32 lanes of a with the lower 32 of b: the
// lower half of the wave holds the two halves' sum of a, the upper that of b.
__device__ __forceinline__ float fold32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The same for 16-lane rows: even rows hold the sum of a over a row pair, odd
// rows that of b.
__device__ __forceinline__ float fold16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int ROR> __device__ __forceinline__ float add_ror(float x)
{
    return x + __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + ROR, 0xf, 0xf, false));
}

// ------------------------------------------------------------------------
// Block: NTHR threads hold all rows of NX columns (4 adjacent columns and R
// rows per thread: rows rg + RS r) for a chunk of TRs, with the voxels'
// weights and the 2 NTR running sums per voxel in registers. D TRs of trains
// are in flight or in use at a time. Per TR: U is summed over a thread's rows,
// over the wave by lane swaps and over the waves through LDS (one barrier, D
// buffers), then every thread adds the TR to its sums and loads the TR D
// ahead. Each train byte is read once per product, where J d and J^H read it
// twice. Bound by the L1's line look-ups: a 64-byte (FP32) or 32-byte (FP16)
// row segment per tile costs one each, so both types take about 1.7 us per TR
// and block even with the trains in L2. Measured (four trains; the y-stages,
// x-GEMMs and partial sums it replaces): 224 x 224, 1120 TRs FP32 213 us (368),
// FP16 182 us (206); 128 x 128, 1024 TRs, three trains FP32 34 us (94).
// ------------------------------------------------------------------------
template <int NTR, int R, int NTHR, int D, typename TT>
__global__ __launch_bounds__(NTHR) void normal_kernel(
    const TT* __restrict__ trains, const float* __restrict__ theta, const float* __restrict__ v,
    const uint8_t* __restrict__ mask, const float2* __restrict__ eytab, float* __restrict__ apart, int nx, int ny,
    int nv, int T, int per, int chunks, int tiles, float neg_nk)
{
    typedef typename TrainVec<TT>::T V;
    constexpr int LX = NX / 4, RS = NTHR / LX, NW = NTHR / 64;
    static_assert(NW == 2 || NW == 4 || NW == 8, "sum over the waves");
    static_assert(D >= 2, "a buffer is rewritten D barriers after it was read");
    __shared__ __attribute__((aligned(16))) float sums[D][NW][2 * NX];
    // rho and the direction's nu per voxel, read back per TR: in registers
    // they would spill, and a spill's reload waits for every train load.
    __shared__ f4 wts[4][R][NTHR];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lx = tid % LX, rg = tid / LX;
    // With a multiple of 8 chunks, all column tiles of a chunk go to one XCD
    // (blocks are dealt to the 8 XCDs in turn), whose L2 then serves the parts
    // of a 128-byte line that neighbouring tiles read.
    int chunk, tile;
    if (chunks % 8 == 0) {
        const int g = blockIdx.x / (8 * tiles), rem = blockIdx.x % (8 * tiles);
        chunk = 8 * g + rem % 8;
        tile = rem / 8;
    } else {
        chunk = blockIdx.x / tiles;
        tile = blockIdx.x % tiles;
    }
    const int n0 = chunk * per, n1 = min(T, n0 + per);
    // A thread past the last whole group of 4 columns takes the last 4 of the
    // row (nx >= 4) and stores those that no other thread has.
    const int x0 = tile * NX + 4 * lx;
    const int xs = min(x0, nx - 4);
    const size_t plane = (size_t)T * nv;

    // Rows past the image read its last row with zero weights.
    unsigned jr[R], er[R];
    float v0[R][4], v1[R][4], v2[R][4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int iy = rg + RS * r;
        er[r] = min(iy, ny - 1);
        jr[r] = er[r] * nx + xs;
        f4 wt[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const unsigned j = jr[r] + c;
            const bool on = iy < ny && (mask == nullptr || mask[j] != 0);
            wt[0][c] = on ? theta[3 * (size_t)nv + j] : 0.f;
            wt[1][c] = on ? theta[4 * (size_t)nv + j] : 0.f;
            wt[2][c] = on ? v[3 * (size_t)nv + j] : 0.f;
            wt[3][c] = on ? v[4 * (size_t)nv + j] : 0.f;
            v0[r][c] = on ? v[j] : 0.f;
            v1[r][c] = on ? v[(size_t)nv + j] : 0.f;
            v2[r][c] = NTR == 4 && on ? v[2 * (size_t)nv + j] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) wts[k][r][tid] = wt[k];
    }
    float acc[R][4][NTR][2];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int p = 0; p < NTR; ++p) acc[r][c][p][0] = acc[r][c][p][1] = 0.f;

    struct Stage {
        V m[R][NTR];
        float2 ey[R];
    };
    // TRs past the chunk read its last one.
    auto load = [&](Stage& t, int n) {
        const int nn = min(n, n1 - 1);
        const TT* base = trains + (size_t)nn * nv;
        const float2* erow = eytab + (size_t)nn * ny;
#pragma unroll
        for (int p = 0; p < NTR; ++p) {
            const char* row = reinterpret_cast<const char*>(base + p * plane);
#pragma unroll
            for (int r = 0; r < R; ++r) t.m[r][p] = *reinterpret_cast<const V*>(row + jr[r] * (unsigned)sizeof(TT));
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            t.ey[r] = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(erow) + er[r] * 8u);
    };
    auto process = [&](Stage& t, int n, int buf) {
        if (n >= n1)   // a zero phase: no contribution
#pragma unroll
            for (int r = 0; r < R; ++r) t.ey[r] = make_float2(0.f, 0.f);
        float u[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) u[i] = 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const f4 pr = wts[0][r][tid], pi = wts[1][r][tid], qr = wts[2][r][tid], qi = wts[3][r][tid];
            const float2 e = t.ey[r];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float mu = (float)t.m[r][0][c];
                float a = v0[r][c] * (float)t.m[r][1][c];
                a = fmaf(v1[r][c], (float)t.m[r][2][c], a);
                if constexpr (NTR == 4) a = fmaf(v2[r][c], (float)t.m[r][3][c], a);
                // x = i (rho a + nu mu) = -xr + i xi
                const float xr = fmaf(pi[c], a, qi[c] * mu), xi = fmaf(pr[c], a, qr[c] * mu);
                u[2 * c] = fmaf(-e.x, xr, fmaf(-e.y, xi, u[2 * c]));
                u[2 * c + 1] = fmaf(e.x, xi, fmaf(-e.y, xr, u[2 * c + 1]));
            }
        }
        // The lanes of one column group differ in bits 2 to 5. Wave halves
        // keep columns 0-1 / 2-3, odd rows of 16 lanes the second of the two.
        float t4[4], s2[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) t4[i] = fold32(u[i], u[i + 4]);
#pragma unroll
        for (int i = 0; i < 2; ++i) s2[i] = add_ror<4>(add_ror<8>(fold16(t4[i], t4[i + 2])));
        if ((lane & 12) == 0)
            *reinterpret_cast<float2*>(&sums[buf][wave][8 * lx + 2 * ((lane >> 4) & 1) + 4 * (lane >> 5)]) =
                make_float2(s2[0], s2[1]);
        __syncthreads();
        if constexpr (sizeof(TT) == 2) {
            // Keep the packed halves, not their conversions, across the sum.
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int p = 0; p < NTR; ++p) asm volatile("" : "+v"(t.m[r][p]));
        }
        float w[8];
        const f4* src = reinterpret_cast<const f4*>(&sums[buf][(lane >> 2) % NW][8 * lx]);
        const f4 lo = src[0], hi = src[1];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float s = i < 4 ? lo[i & 3] : hi[i & 3];
            if constexpr (NW >= 4) s = add_ror<8>(s);
            s = add_ror<4>(s);
            if constexpr (NW == 8) s = fold16(s, s);
            w[i] = neg_nk * s;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float2 e = t.ey[r];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float vr = fmaf(e.x, w[2 * c], e.y * w[2 * c + 1]);
                const float vi = fmaf(e.x, w[2 * c + 1], -e.y * w[2 * c]);
#pragma unroll
                for (int p = 0; p < NTR; ++p) {
                    const float mu = (float)t.m[r][p][c];
                    acc[r][c][p][0] = fmaf(mu, vr, acc[r][c][p][0]);
                    acc[r][c][p][1] = fmaf(mu, vi, acc[r][c][p][1]);
                }
            }
        }
    };

    Stage st[D];
#pragma unroll
    for (int i = 0; i < D; ++i) load(st[i], n0 + i);
    for (int n = n0; n < n1; n += D)
#pragma unroll
        for (int i = 0; i < D; ++i) {
            process(st[i], n + i, i);
            load(st[i], n + i + D);
        }

    float* dst = apart + (size_t)chunk * 8 * nv;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (rg + RS * r >= ny) continue;
#pragma unroll
        for (int p = 0; p < NTR; ++p)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                float* o = dst + (size_t)(2 * p + k) * nv + jr[r];
                if (xs == x0)
                    *reinterpret_cast<f4u*>(o) =
                        f4u{acc[r][0][p][k], acc[r][1][p][k], acc[r][2][p][k], acc[r][3][p][k]};
                else
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (xs + c >= x0) o[c] = acc[r][c][p][k];
            }
    }
}

template <int R, int NTHR, typename TT>
hipError_t launch_shape(const Dims& d, int chunks, int ntr, const TT* trains, const float* theta, const float* v,
                        const uint8_t* mask, const float2* eytab, float* apart, hipStream_t s)
{
    constexpr int D = sizeof(TT) == 2 && R == 1 ? 3 : 2;
    const int per = ceil_div(d.T, chunks), tiles = ceil_div(d.nx, NX);
    if (ntr == 4)
        normal_kernel<4, R, NTHR, D, TT><<<chunks * tiles, NTHR, 0, s>>>(
            trains, theta, v, mask, eytab, apart, d.nx, d.ny, d.nv, d.T, per, chunks, tiles, -(float)d.nk);
    else
        normal_kernel<3, R, NTHR, D, TT><<<chunks * tiles, NTHR, 0, s>>>(
            trains, theta, v, mask, eytab, apart, d.nx, d.ny, d.nv, d.T, per, chunks, tiles, -(float)d.nk);
    return hipGetLastError();
}

// 4 NTHR / NX rows per step: the smallest block that holds all rows, and from
// 129 rows on two of them per thread.
template <typename TT>
hipError_t launch_typed(const Dims& d, int chunks, int ntr, const TT* trains, const float* theta, const float* v,
                        const uint8_t* mask, const float2* eytab, float* apart, hipStream_t s)
{
    if (d.ny <= 32) return launch_shape<1, 128>(d, chunks, ntr, trains, theta, v, mask, eytab, apart, s);
    if (d.ny <= 64) return launch_shape<1, 256>(d, chunks, ntr, trains, theta, v, mask, eytab, apart, s);
    if (d.ny <= 128) return launch_shape<1, 512>(d, chunks, ntr, trains, theta, v, mask, eytab, apart, s);
    return launch_shape<2, 512>(d, chunks, ntr, trains, theta, v, mask, eytab, apart, s);
}

}  // namespace

int normal_chunks(const Dims& d)
{
    if (d.C != 1 || d.nx < 4 || d.ny > 256 || d.T < 8) return 0;
    const int tiles = ceil_div(d.nx, NX);
    int ch = std::min({ceil_div(256, tiles), 32, d.T / 8});
    if (ch >= 8) ch -= ch % 8;
    ch = std::max(ch, 1);
    return ceil_div(d.T, ceil_div(d.T, ch));
}

hipError_t launch_normal(const Dims& d, int ntr, const void* trains, bool f16, const float* theta, const float* v,
                         const uint8_t* mask, const float2* eytab, float* apart, hipStream_t s)
{
    const int chunks = normal_chunks(d);
    if (chunks == 0 || (ntr != 3 && ntr != 4)) return hipErrorInvalidValue;
    if (f16)
        return launch_typed(d, chunks, ntr, static_cast<const _Float16*>(trains), theta, v, mask, eytab, apart, s);
    return launch_typed(d, chunks, ntr, static_cast<const float*>(trains), theta, v, mask, eytab, apart, s);
}

}  // namespace mrstat

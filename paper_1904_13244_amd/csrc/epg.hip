// EPG linearisation kernel: one voxel per group of L lanes, the K states of
// the voxel split over the group (S = Kcap / L consecutive orders per lane),
// value and NTAN tangent state vectors in registers (NTAN = 3: ln T1, ln T2,
// B1; 2: ln T1, ln T2 only, for fits with B1 held fixed, whose Jacobian has
// no B1 column; 0: value only).
//
// Model: gradient-spoiled transient-state sequence; per TR an instantaneous RF
// pulse of angle B1 * alpha_n about an axis at RF phase phi_n in {0, pi},
// relaxation to TE, readout of F+_0 demodulated by the RF phase, relaxation to
// TR, spoiler shift of all orders by one (truncated at K). Tangents in ln T1,
// ln T2 and B1 follow the forward-mode recursion of Supporting Information S2
// (each update differentiated, zero initial tangents, sin/cos/exp of a TR
// computed once and reused by value and tangents).
//
// Real form: with phi_n in {0, pi} and no off-resonance every F state stays
// purely imaginary and every Z state real, so the kernel carries
// f = Im F+, g = Im F-, z = Z (3 reals per order instead of 6). With
// sg = cos(phi_n) = +-1 and a = B1 alpha_n, the RF operator is
//     f' = c^2 f + s^2 g - sg sin(a) z
//     g' = s^2 f + c^2 g + sg sin(a) z
//     z' = (sg/2) sin(a) (f - g) + cos(a) z          (c, s = cos, sin of a/2)
// and the relaxation over a whole TR (E1, E2, regrowth 1 - E1 of Z_0) is
// folded into its coefficients; the readout uses the unrelaxed RF output at
// order 0 times E2(TE). Recorded value: Im m = sg E2(TE) f_0.
#include "mrstat_internal.h"

#include <algorithm>

namespace mrstat {
namespace {

// sin and cos of half the flip angle b alpha, b = B1 / 2 pi: the product and its
// reduction to half turns in FP64 (full rate here, and far fewer temporaries than
// the general FP32 reduction, which would spill states); what the FP32 half turns
// leave out turns the result: errors around half a turn up to 2e-7 instead of 4e-7,
// for 0 to 3% of the time (up to 8% with 2 tangents of 8 orders per lane, which spill).
__device__ __forceinline__ void half_sines(double b, float alpha, float& sn, float& cs)
{
    const double t = b * (double)alpha, r = t - 2.0 * rint(0.5 * t);
    const float h = (float)r, low = (float)((r - (double)h) * 3.14159265358979323846);
    float s0, c0;
    sincospif(h, &s0, &c0);
    sn = fmaf(c0, low, s0);
    cs = fmaf(-s0, low, c0);
}

// Spoiler shift of one state vector: order k of F+ takes order k-1, order k
// of F- takes order k+1, F-_{K-1} = 0, and the new F+_0 = conj(F-_0), which
// is -g_0 in the real form. Orders are spread over the L lanes of a group.
template <int S, int L>
__device__ __forceinline__ void shift_orders(float (&f)[S], float (&g)[S], bool lead, bool last)
{
    float up = 0.f, dn = 0.f;
    if constexpr (L > 1) {
        up = __shfl_up(f[S - 1], 1, L);
        dn = __shfl_down(g[0], 1, L);
    }
#pragma unroll
    for (int i = S - 1; i >= 1; --i) f[i] = f[i - 1];
#pragma unroll
    for (int i = 0; i < S - 1; ++i) g[i] = g[i + 1];
    g[S - 1] = last ? 0.f : dn;
    f[0] = lead ? -g[0] : up;
}

template <int S>
__device__ __forceinline__ void clear_above(float (&f)[S], int base, int K)
{
#pragma unroll
    for (int i = 0; i < S; ++i)
        if (base + i >= K) f[i] = 0.f;
}

// LIST: the group handles voxel idx[vox] for vox < *count (the other voxels'
// outputs are left untouched); whole blocks past the list exit at once.
// TT: element type of the stored trains (float, or _Float16 rounded to
// nearest from the FP32 recursion).
//
// Bound by the vector units: an order's update is 34 operations (value 7,
// ln T1 8, ln T2 9, B1 10): with w = f - g and p = E2 (s^2 w + sg sin(a) z) the
// rotation is f' = E2 f - p, g' = E2 g + p, and the B1 tangent takes the
// rotation's generator, alpha sg (-z, z, w/2), before it is rotated itself.
// The lane moves stay shuffles through LDS, a unit that is idle here: as DPP
// moves they take vector slots and waits (3 tangents 2.03 ms instead of 1.78).
// 224^2 voxels, 32 orders, 1120 TRs, 2 lanes: 1.78 ms with 3 tangents and
// 0.45 ms for values in launches that follow one another, 1.91 and 0.49 inside
// GN steps (coefficients c^2, s^2 and their derivatives for every row, sines per
// lane, one TR per turn: 1.98 to 2.13 and 0.52); 128^2 with 2 tangents, at the
// lanes chosen below, 0.44 and 0.21 ms in GN steps (1.24 and 0.52 with 2 lanes).
//
// FP16 trains keep the row products with c^2 and s^2 (PLAIN): their values and
// gradients carry the rounding of the trains, to which a changed FP32 recursion
// adds its own (a gradient's norm moved by up to 2e-6); 2.39 ms with 3 tangents.
// Waves per SIMD that the states (3 S (1 + NTAN) registers) leave room for; PLAIN
// is faster without that bound (256^2, 32 orders, 256 TRs, 3 tangents 605 and 573
// us) except where its states then spill (24 orders on 2 lanes, 842 and 575 us).
constexpr int epg_waves(int s, int ntan, bool plain)
{
    if (plain) return s == 16 && ntan == 3 ? 2 : 1;
    return 3 * s * (1 + ntan) > 130 ? 2 : 3 * s * (1 + ntan) > 84 ? 3 : 4;
}

// TRs per turn of the loop, whose shifts then need no register moves; the
// largest states leave no room for a second copy.
constexpr int epg_unroll(int s, int l, int ntan) { return 3 * s * (1 + ntan) > 150 ? 1 : l >= 4 && 3 * s * (1 + ntan) <= 50 ? 4 : 2; }

template <int S, int L, int NTAN, bool MASKED, bool LIST, typename TT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(epg_waves(S, NTAN, sizeof(TT) == 2)))) void
epg_kernel(const float* __restrict__ theta, const float2* __restrict__ seq, TT* __restrict__ out, int nv, int T, int K,
           SeqTimes st, const int* __restrict__ idx, const int* __restrict__ count)
{
    const int gt = blockIdx.x * blockDim.x + threadIdx.x;
    const int vox = gt / L;
    const int l = gt % L;
    int j;
    bool valid;
    if constexpr (LIST) {
        const int cnt = *count;
        if ((int)(blockIdx.x * blockDim.x / L) >= cnt) return;   // uniform per block
        valid = vox < cnt;
        j = idx[valid ? vox : cnt - 1];
    } else {
        valid = vox < nv;
        j = valid ? vox : nv - 1;   // keep every lane active for the lane moves
    }
    const bool lead = (l == 0), last = (l == L - 1);
    const bool store = valid && lead;
    const int base = l * S;

    const float lnT1 = theta[j], lnT2 = theta[nv + j], B1 = theta[2 * nv + j];
    const float rT1 = expf(-lnT1), rT2 = expf(-lnT2);   // 1/T1, 1/T2
    const float tau1 = st.tr * rT1, tau2 = st.tr * rT2, tau2e = st.te * rT2;
    const float E1 = expf(-tau1), E1m = expm1f(-tau1), E2 = expf(-tau2);
    const float R1 = lead ? -E1m : 0.f;                 // regrowth of Z_0 only
    const float dR1 = lead ? tau1 * E1 : 0.f;           // -d(1-E1)/dlnT1
    const float E2e = expf(-tau2e);
    const float taui = st.tinv * rT1;
    const float E1i = expf(-taui), R1i = -expm1f(-taui);

    constexpr bool TANG = NTAN > 0, TB1 = NTAN == 3;
    // z + (E1 cos(a) - 1) z instead of E1 cos(a) z halves the trains' error at
    // 128 TRs (1.2e-6 to 0.66e-6; at 1120 TRs 1.5e-6 to 1.25e-6) for nothing up
    // to 8 orders per lane; with 16 it costs 6 to 11% (an FMA that reads three
    // registers takes 3 cycles, a product 2), and the product stays.
    constexpr bool FINE = S <= 8;
    constexpr bool PLAIN = sizeof(TT) == 2;
    float f[S], g[S], z[S];
    float f1[S], g1[S], z1[S];   // d/d ln T1
    float f2[S], g2[S], z2[S];   // d/d ln T2
    float f3[S], g3[S], z3[S];   // d/d B1
#pragma unroll
    for (int i = 0; i < S; ++i) {
        f[i] = g[i] = z[i] = 0.f;
        if constexpr (TANG) {
            f1[i] = g1[i] = z1[i] = 0.f;
            f2[i] = g2[i] = z2[i] = 0.f;
        }
        if constexpr (TB1) f3[i] = g3[i] = z3[i] = 0.f;
    }
    // Ideal inversion of the equilibrium Z_0 = 1, then relaxation over t_inv.
    if (lead) {
        z[0] = R1i - E1i;
        if constexpr (TANG) z1[0] = -2.f * taui * E1i;
    }

    const size_t plane = (size_t)T * nv;
    TT* o0 = out + j;
    auto put = [&](int q, int n, float x) {
        if (store) o0[q * plane + (size_t)n * nv] = (TT)x;
    };
    // One TR: sh, ch are sin and cos of half its flip angle B1 alpha.
    auto tr = [&](int n, float alpha, float sg, float sh, float ch) {
        const float s2 = sh * sh, sa = 2.f * sh * ch;
        const float sgsa = sg * sa;
        const float ke = sg * E2e;
        // Coefficients with the TR relaxation folded in.
        const float B = E2 * s2, Cc = E2 * sgsa, D = 0.5f * E1 * sgsa;
        if constexpr (PLAIN) {
            const float c2 = ch * ch, ca = (ch - sh) * (ch + sh);
            const float A = E2 * c2, G = E1 * ca;
            // B1 derivatives of the coefficients (d a / d B1 = alpha): dA = -dB.
            const float dA = -0.5f * E2 * alpha * sa, dC = E2 * alpha * sg * ca;
            const float dD = 0.5f * E1 * alpha * sg * ca, dG = -E1 * alpha * sa;
            const float rp = fmaf(c2, f[0], fmaf(s2, g[0], -sgsa * z[0]));
            put(0, n, ke * rp);
            if constexpr (TANG) {
                put(1, n, ke * fmaf(c2, f1[0], fmaf(s2, g1[0], -sgsa * z1[0])));
                put(2, n, ke * fmaf(tau2e, rp, fmaf(c2, f2[0], fmaf(s2, g2[0], -sgsa * z2[0]))));
            }
            if constexpr (TB1) {
                const float drp = fmaf(-0.5f * sa, f[0] - g[0], -sg * ca * z[0]);
                put(3, n, ke * fmaf(c2, f3[0], fmaf(s2, g3[0], fmaf(alpha, drp, -sgsa * z3[0]))));
            }
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const float w = f[i] - g[i], Cz = Cc * z[i];
                const float nf = fmaf(A, f[i], fmaf(B, g[i], -Cz));
                const float ng = fmaf(B, f[i], fmaf(A, g[i], Cz));
                const float nz = fmaf(D, w, G * z[i]);
                if constexpr (TANG) {
                    {
                        const float w1 = f1[i] - g1[i], Cz1 = Cc * z1[i];
                        const float a = fmaf(A, f1[i], fmaf(B, g1[i], -Cz1));
                        g1[i] = fmaf(B, f1[i], fmaf(A, g1[i], Cz1));
                        f1[i] = a;
                        z1[i] = fmaf(D, w1, fmaf(G, z1[i], tau1 * nz));
                    }
                    {
                        const float w2 = f2[i] - g2[i], Cz2 = Cc * z2[i];
                        const float a = fmaf(A, f2[i], fmaf(B, g2[i], fmaf(tau2, nf, -Cz2)));
                        g2[i] = fmaf(B, f2[i], fmaf(A, g2[i], fmaf(tau2, ng, Cz2)));
                        f2[i] = a;
                        z2[i] = fmaf(D, w2, G * z2[i]);
                    }
                }
                if constexpr (TB1) {
                    const float w3 = f3[i] - g3[i], Cz3 = Cc * z3[i];
                    const float t3 = fmaf(dA, w, -dC * z[i]);
                    const float a = fmaf(A, f3[i], fmaf(B, g3[i], t3 - Cz3));
                    g3[i] = fmaf(B, f3[i], fmaf(A, g3[i], Cz3 - t3));
                    f3[i] = a;
                    z3[i] = fmaf(D, w3, fmaf(G, z3[i], fmaf(dD, w, dG * z[i])));
                }
                f[i] = nf, g[i] = ng, z[i] = nz;
            }
        } else {
            const float Gm = fmaf(-2.f * E1, s2, E1m);   // E1 cos(a) - 1
            const float G = FINE ? 1.f + Gm : E1 * ((ch - sh) * (ch + sh));
            // Readout at TE from the unrelaxed RF output of order 0.
            const float rp = f[0] - fmaf(s2, f[0] - g[0], sgsa * z[0]);
            put(0, n, ke * rp);
            if constexpr (TANG) {
                const float rp1 = f1[0] - fmaf(s2, f1[0] - g1[0], sgsa * z1[0]);
                const float rp2 = f2[0] - fmaf(s2, f2[0] - g2[0], sgsa * z2[0]);
                put(1, n, ke * rp1);
                put(2, n, ke * fmaf(tau2e, rp, rp2));
            }
            const float as = alpha * sg, hs = 0.5f * as;
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const float w = f[i] - g[i];
                if constexpr (TB1) {   // the generator of the rotation, then the rotation itself
                    f3[i] = fmaf(-as, z[i], f3[i]);
                    g3[i] = fmaf(as, z[i], g3[i]);
                    z3[i] = fmaf(hs, w, z3[i]);
                    const float w3 = f3[i] - g3[i];
                    if (i == 0) put(3, n, ke * (f3[0] - fmaf(s2, w3, sgsa * z3[0])));
                    const float p3 = fmaf(B, w3, Cc * z3[i]);
                    f3[i] = fmaf(E2, f3[i], -p3);
                    g3[i] = fmaf(E2, g3[i], p3);
                    z3[i] = fmaf(D, w3, G * z3[i]);
                }
                const float p = fmaf(B, w, Cc * z[i]);
                f[i] = fmaf(E2, f[i], -p);
                g[i] = fmaf(E2, g[i], p);
                z[i] = fmaf(D, w, FINE ? fmaf(Gm, z[i], z[i]) : G * z[i]);
                if constexpr (TANG) {
                    {   // ln T1: only E1 (Z rows) depends on T1
                        const float w1 = f1[i] - g1[i];
                        const float p1 = fmaf(B, w1, Cc * z1[i]);
                        f1[i] = fmaf(E2, f1[i], -p1);
                        g1[i] = fmaf(E2, g1[i], p1);
                        z1[i] = fmaf(D, w1, fmaf(G, z1[i], tau1 * z[i]));
                    }
                    {   // ln T2: only E2 (F rows) depends on T2
                        const float w2 = f2[i] - g2[i];
                        const float p2 = fmaf(B, w2, Cc * z2[i]);
                        f2[i] = fmaf(E2, f2[i], fmaf(tau2, f[i], -p2));
                        g2[i] = fmaf(E2, g2[i], fmaf(tau2, g[i], p2));
                        z2[i] = fmaf(D, w2, G * z2[i]);
                    }
                }
            }
        }
        z[0] += R1;
        if constexpr (TANG) z1[0] -= dR1;

        shift_orders<S, L>(f, g, lead, last);
        if constexpr (MASKED) clear_above<S>(f, base, K);
        if constexpr (TANG) {
            shift_orders<S, L>(f1, g1, lead, last);
            shift_orders<S, L>(f2, g2, lead, last);
            if constexpr (MASKED) {
                clear_above<S>(f1, base, K);
                clear_above<S>(f2, base, K);
            }
        }
        if constexpr (TB1) {
            shift_orders<S, L>(f3, g3, lead, last);
            if constexpr (MASKED) clear_above<S>(f3, base, K);
        }
    };
    if constexpr (PLAIN) {
        for (int n = 0; n < T; ++n) {
            const float2 q = seq[n];
            float sh, ch;
            sincosf(0.5f * (B1 * q.x), &sh, &ch);
            tr(n, q.x, q.y, sh, ch);
        }
        return;
    }
    // U TRs at a time. Lane l of the group makes the sines of TR l mod U (one
    // lane: of all U), for the next U TRs while these ones run.
    constexpr int U = epg_unroll(S, L, NTAN), NS = L == 1 ? U : 1;
    static_assert(U <= L || L == 1, "one lane for each TR's sines");
    const double turns = (double)B1 * 0.15915494309189533577;   // B1 / 2 pi
    float s0[NS], c0[NS];
    float2 q[U];
    auto load = [&](int n) {
#pragma unroll
        for (int k = 0; k < U; ++k) q[k] = seq[min(n + k, T - 1)];
    };
    auto sines = [&]() {
        if constexpr (NS == U) {
#pragma unroll
            for (int k = 0; k < U; ++k) half_sines(turns, q[k].x, s0[k], c0[k]);
        } else {
            float a = l & 1 ? q[1].x : q[0].x;
            if constexpr (U == 4) a = l & 2 ? (l & 1 ? q[3].x : q[2].x) : a;
            half_sines(turns, a, s0[0], c0[0]);
        }
    };
    float sh[U], ch[U], al[U], sg[U];
    auto take = [&]() {   // the next U TRs become the present ones
#pragma unroll
        for (int k = 0; k < U; ++k) al[k] = q[k].x, sg[k] = q[k].y;
        if constexpr (NS == U) {
#pragma unroll
            for (int k = 0; k < U; ++k) sh[k] = s0[k], ch[k] = c0[k];
        } else {
            sh[0] = __shfl(s0[0], 0, L), sh[1] = __shfl(s0[0], 1, L);
            ch[0] = __shfl(c0[0], 0, L), ch[1] = __shfl(c0[0], 1, L);
            if constexpr (U == 4) {
                sh[2] = __shfl(s0[0], 2, L), sh[3] = __shfl(s0[0], 3, L);
                ch[2] = __shfl(c0[0], 2, L), ch[3] = __shfl(c0[0], 3, L);
            }
        }
    };
    load(0);
    if constexpr (U > 1) sines();
    int n = 0;
    for (; n + U <= T; n += U) {
        if constexpr (U == 1) sines();   // no registers to make the next ones early
        take();
        load(n + U);
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (U > 1 && k == U / 2) sines();
            tr(n + k, al[k], sg[k], sh[k], ch[k]);
        }
    }
    if constexpr (U > 1) {
        take();
#pragma unroll
        for (int k = 0; k < U - 1; ++k)
            if (n + k < T) tr(n + k, al[k], sg[k], sh[k], ch[k]);
    }
}

// FP16 values at 16 orders per lane, the products of PLAIN in a kernel of their
// own: 224^2 voxels, 256 TRs, 32 orders on 2 lanes 131 us (137 as a form of
// epg_kernel), 64 orders on 4 lanes at 160^2 131 (140).
template <int L, bool MASKED, bool LIST>
__global__ __launch_bounds__(256) void epg_half_value_kernel(const float* __restrict__ theta,
                                                             const float2* __restrict__ seq,
                                                             _Float16* __restrict__ out, int nv, int T, int K,
                                                             SeqTimes st, const int* __restrict__ idx,
                                                             const int* __restrict__ count)
{
    constexpr int S = 16;
    const int gt = blockIdx.x * blockDim.x + threadIdx.x;
    const int vox = gt / L;
    const int l = gt % L;
    int j;
    bool valid;
    if constexpr (LIST) {
        const int cnt = *count;
        if ((int)(blockIdx.x * blockDim.x / L) >= cnt) return;   // uniform per block
        valid = vox < cnt;
        j = idx[valid ? vox : cnt - 1];
    } else {
        valid = vox < nv;
        j = valid ? vox : nv - 1;   // keep every lane active for the lane moves
    }
    const bool lead = (l == 0), last = (l == L - 1);
    const bool store = valid && lead;
    const int base = l * S;

    const float lnT1 = theta[j], lnT2 = theta[nv + j], B1 = theta[2 * nv + j];
    const float rT1 = expf(-lnT1), rT2 = expf(-lnT2);   // 1/T1, 1/T2
    const float tau1 = st.tr * rT1, tau2 = st.tr * rT2, tau2e = st.te * rT2;
    const float E1 = expf(-tau1), E2 = expf(-tau2);
    const float R1 = lead ? -expm1f(-tau1) : 0.f;       // regrowth of Z_0 only
    const float E2e = expf(-tau2e);
    const float taui = st.tinv * rT1;
    const float E1i = expf(-taui), R1i = -expm1f(-taui);

    float f[S], g[S], z[S];
#pragma unroll
    for (int i = 0; i < S; ++i) f[i] = g[i] = z[i] = 0.f;
    if (lead) z[0] = R1i - E1i;   // ideal inversion, then relaxation over t_inv

    _Float16* o0 = out + j;
    for (int n = 0; n < T; ++n) {
        const float2 sq = seq[n];
        const float alpha = sq.x, sg = sq.y;
        float sh, ch;
        sincosf(0.5f * (B1 * alpha), &sh, &ch);
        const float c2 = ch * ch, s2 = sh * sh;
        const float sa = 2.f * sh * ch, ca = (ch - sh) * (ch + sh);
        const float sgsa = sg * sa;
        const float A = E2 * c2, B = E2 * s2, Cc = E2 * sgsa;
        const float D = 0.5f * E1 * sgsa, G = E1 * ca;
        {
            const float rp = fmaf(c2, f[0], fmaf(s2, g[0], -sgsa * z[0]));
            const float ke = sg * E2e;
            if (store) o0[(size_t)n * nv] = (_Float16)(ke * rp);
        }
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const float w = f[i] - g[i];
            const float Cz = Cc * z[i];
            const float nf = fmaf(A, f[i], fmaf(B, g[i], -Cz));
            const float ng = fmaf(B, f[i], fmaf(A, g[i], Cz));
            z[i] = fmaf(D, w, G * z[i]);
            f[i] = nf; g[i] = ng;
        }
        z[0] += R1;
        shift_orders<S, L>(f, g, lead, last);
        if constexpr (MASKED) clear_above<S>(f, base, K);
    }
}

template <int S, int L, int NTAN, bool LIST, typename TT>
hipError_t launch_sl(const Dims& d, SeqTimes st, const float* theta, const float2* seq, TT* out,
                     const int* idx, const int* count, hipStream_t s)
{
    const long threads = (long)d.nv * L;
    const int block = 256;
    const int grid = (int)((threads + block - 1) / block);
    auto run = [&](auto kernel) { kernel<<<grid, block, 0, s>>>(theta, seq, out, d.nv, d.T, d.K, st, idx, count); };
    const bool whole = d.K == S * L;
    if constexpr (S == 16 && NTAN == 0 && sizeof(TT) == 2) {
        if (whole) run(&epg_half_value_kernel<L, false, LIST>);
        else run(&epg_half_value_kernel<L, true, LIST>);
    } else {
        if (whole) run(&epg_kernel<S, L, NTAN, false, LIST, TT>);
        else run(&epg_kernel<S, L, NTAN, true, LIST, TT>);
    }
    return hipGetLastError();
}

// Lanes per voxel where the caller left them open: those with the least orders
// per lane S times waves per SIMD w (of 256 CUs x 4), both with what comes on
// top. A lane's time has a part that does not shrink with its orders (the sines;
// for values, which leave little else, more, and with FP32 trains shared by four
// lanes or more); two waves on a SIMD take 1.4 times one's time (one alone issues
// a vector operation in 4 cycles, two together one in 2), more in proportion; 16
// orders leave room for fewer waves. Near ties go to fewer lanes. Measured over
// 256 TRs, us with 1 / 2 / 4 / 8 lanes, FP32 trains with 3 tangents; values; FP16
// trains with 3 tangents; values:
//   K 8   96^2    179  150  107;   71  68  48;   233 181 143;   85  82  69
//         256^2   188  178  194;   72  79  74;   237 221 260;   87  83 105
//         320^2   220  294  305;   78 115 110;   301 362 404;   91 121 155
//   K 16  128^2   324  219  134  123;   93  84  56  52;   388 267 188 162;  121  91  77  69
//         200^2   329  246  217  230;   94  92  71  85;   394 342 296 309;  121  96 101 120
//         320^2   379  454  439  537;  106 145 136 189;   513 607 585 704;  134 157 187 262
//   K 32  144^2        365  255  216;      112  70  72;       431 342 300;      122 106 100
//         224^2        418  458  433;      117 115 134;       559 600 579;      137 160 186
//         320^2        806  737  777;      206 189 237;      1071 987 1032;     236 256 324
//   K 64  200^2             716  540;           143 141;            885 721;          195 196
//         256^2             821  838;           179 215;           1077 1107;         246 291
int auto_lanes(const Dims& d, int ntan, bool f16)
{
    const int most = d.K <= 8 ? 4 : 8, orders = d.K <= 8 ? 8 : d.K <= 16 ? 16 : d.K <= 32 ? 32 : 64;
    int best = 0;
    double t_best = 0.0;
    for (int l = std::max(1, orders / 16); l <= most; l *= 2) {
        const int s = orders / l, w = (int)(((long)d.nv * l + 65535) / 65536);
        const double top = ntan > 0 ? 1.8 : f16 ? 5.2 : l < 4 ? 7.5 : 4.5;
        const double full = s < 16 || ntan == 0 ? 0.0 : ntan == 3 ? 1.6 : 1.3;
        const double t = (s + top + full) * (w > 1 ? w : ntan > 0 ? 1.45 : 1.6);
        if (best == 0 || t < 0.98 * t_best) t_best = t, best = l;
    }
    return best;
}

template <int NTAN, bool LIST, typename TT>
hipError_t launch_any(const Dims& d, SeqTimes st, const float* theta, const float2* seq,
                      TT* out, int lanes, const int* idx, const int* count, hipStream_t s)
{
    if (lanes == 0) lanes = auto_lanes(d, NTAN, sizeof(TT) == 2);
    const int K = d.K;
#define SL(S_, L_) launch_sl<S_, L_, NTAN, LIST, TT>(d, st, theta, seq, out, idx, count, s)
    if (K <= 8) {
        if (lanes == 2) return SL(4, 2);
        if (lanes == 4) return SL(2, 4);
        return SL(8, 1);
    }
    if (K <= 16) {
        if (lanes == 1) return SL(16, 1);
        if (lanes == 4) return SL(4, 4);
        if (lanes == 8) return SL(2, 8);
        return SL(8, 2);
    }
    if (K <= 32) {
        if (lanes == 4) return SL(8, 4);
        if (lanes == 8) return SL(4, 8);
        return SL(16, 2);
    }
    if (K <= 64) {
        if (lanes == 8) return SL(8, 8);
        return SL(16, 4);
    }
#undef SL
    return hipErrorInvalidValue;
}

// Appends to idx every voxel (in the mask) whose (ln T1, ln T2, B1) lies
// outside [lo, hi] or is not finite; *count must be 0 on entry. One atomic per
// wave; the order of the list is unspecified (each voxel is simulated alone).
__global__ __launch_bounds__(256) void box_compact_kernel(const float* __restrict__ theta, int nv,
                                                          float lo0, float lo1, float lo2, float hi0,
                                                          float hi1, float hi2,
                                                          const uint8_t* __restrict__ mask,
                                                          int* __restrict__ idx, int* __restrict__ count)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    bool out = false;
    if (j < nv && (!mask || mask[j])) {
        const float a = theta[j], b = theta[nv + j], c = theta[2 * nv + j];
        const bool in = (a >= lo0 && a <= hi0) && (b >= lo1 && b <= hi1) && (c >= lo2 && c <= hi2);
        out = !in;   // NaN compares false, so it falls back as well
    }
    const uint64_t bal = __ballot(out);
    if (bal == 0) return;
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (lane == __ffsll((unsigned long long)bal) - 1) base = atomicAdd(count, __popcll(bal));
    base = __shfl(base, __ffsll((unsigned long long)bal) - 1);
    if (out) idx[base + __popcll(bal & ((1ull << lane) - 1ull))] = j;
}

__global__ void zero_int_kernel(int* p) { *p = 0; }

__global__ void half_to_float_kernel(const _Float16* __restrict__ in, float* __restrict__ out, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (float)in[i];
}

}  // namespace

template <bool LIST, typename TT>
hipError_t launch_ntan(const Dims& d, SeqTimes st, const float* theta, const float2* seq, TT* out,
                       int ntan, int lanes, const int* idx, const int* count, hipStream_t s)
{
    switch (ntan) {
        case 0: return launch_any<0, LIST>(d, st, theta, seq, out, lanes, idx, count, s);
        case 2: return launch_any<2, LIST>(d, st, theta, seq, out, lanes, idx, count, s);
        case 3: return launch_any<3, LIST>(d, st, theta, seq, out, lanes, idx, count, s);
        default: return hipErrorInvalidValue;
    }
}

template <bool LIST>
hipError_t launch_typed(const Dims& d, SeqTimes st, const float* theta, const float2* seq, void* out,
                        int ntan, int lanes, bool f16, const int* idx, const int* count,
                        hipStream_t s)
{
    if (f16)
        return launch_ntan<LIST>(d, st, theta, seq, static_cast<_Float16*>(out), ntan, lanes, idx, count, s);
    return launch_ntan<LIST>(d, st, theta, seq, static_cast<float*>(out), ntan, lanes, idx, count, s);
}

hipError_t launch_epg(const Dims& d, SeqTimes st, const float* theta, const float2* seq,
                      void* out, int ntan, int lanes, bool f16, hipStream_t s)
{
    return launch_typed<false>(d, st, theta, seq, out, ntan, lanes, f16, nullptr, nullptr, s);
}

hipError_t launch_epg_list(const Dims& d, SeqTimes st, const float* theta, const float2* seq,
                           void* out, int ntan, int lanes, bool f16, const int* idx,
                           const int* count, hipStream_t s)
{
    return launch_typed<true>(d, st, theta, seq, out, ntan, lanes, f16, idx, count, s);
}

hipError_t launch_trains_to_f32(const void* in, bool f16, float* out, size_t n, hipStream_t s)
{
    if (!f16) return hipMemcpyAsync(out, in, n * sizeof(float), hipMemcpyDeviceToDevice, s);
    half_to_float_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(static_cast<const _Float16*>(in),
                                                                   out, n);
    return hipGetLastError();
}

hipError_t launch_box_compact(const Dims& d, const float* theta, const float* lo, const float* hi,
                              const uint8_t* mask, int* idx, int* count, hipStream_t s)
{
    zero_int_kernel<<<1, 1, 0, s>>>(count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    box_compact_kernel<<<ceil_div(d.nv, 256), 256, 0, s>>>(theta, d.nv, lo[0], lo[1], lo[2], hi[0], hi[1],
                                                           hi[2], mask, idx, count);
    return hipGetLastError();
}

}  // namespace mrstat

// Constrained linear fitting of the cheap potential on gfx950 (Methods,
// "Constrained potential fitting").
//
// The cheap potential is linear in its free spline coefficients u, so a
// configuration's energy and forces are A u for a design matrix A. Three
// kernels build and solve the fit:
//  - k_fit_design: one wavefront per atom i produces the derivatives of F_i
//    (three rows) and of the site energy E_i by every parameter as small dense
//    products over i's interactions, on the FP64 matrix cores. Interactions
//    are produced up to 64 at a time (one per lane) as records in LDS, then
//    contracted four at a time, so each output element is a sum in a fixed
//    order (no atomics). F_i collects the pairs of i, the triplets centred on
//    i, and the triplets centred on a neighbour j in which i is a leg (the
//    other leg from j's 3-body list, built beforehand by k_fit_list3).
//  - k_fit_gram_partial / k_fit_gram_reduce: G = A^T diag(w) A and
//    b = A^T diag(w) y. Each workgroup stages 32 rows at a time in LDS and
//    every thread accumulates 4 x 4 blocks of the upper triangle; partials of
//    fixed row chunks are summed in chunk order.
//  - k_fit_search: one workgroup runs the whole lambda search (G_H and b_H
//    come from the Gram kernels just before): the normal
//    equations (G_S + lam G_H + ridge I) c = b_S + lam b_H solved by a
//    Cholesky factorisation held packed in LDS, the hard residual
//    sum_h w_h (A_H c - y_H)_h^2 from the hard rows, decades of lam until the residual
//    is at most alpha, then interval bisection until it is within tol of
//    alpha. Every loop has a fixed bound.
// Everything is FP64 whatever the context's force precision.
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace mlmix {

constexpr int kFitWave = 64;

// Orders one wavefront's LDS writes before its later LDS reads.
__device__ __forceinline__ void fit_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- B-splines

// The four non-zero clamped uniform cubic B-splines at x (0 <= x < top) and
// their derivatives, by the Cox-de Boor triangle on the span holding x. The
// recursion runs in knot units u = x / h (B-splines do not change when x and
// the knots are scaled together), where the knot differences are 1, 2 or 3 and
// those of the derivative are the last stage's, so no division is left; ih =
// 1/h = (npts - 1)/top. The functions are B_first .. B_first+3.
__device__ __forceinline__ void fit_bspline(double x, int npts, double ih, int &first, double N[4],
                                            double dN[4])
{
    const double u = x * ih;
    const double k0 = fmin(fmax(floor(u), 0.0), (double)(npts - 2)), top = (double)(npts - 1);
    // knots K_mu-2 .. K_mu+3 (K_mu = k0, clamped at both ends)
    const double km2 = fmax(k0 - 2.0, 0.0), km1 = fmax(k0 - 1.0, 0.0), k1 = k0 + 1.0;
    const double k2 = fmin(k0 + 2.0, top), k3 = fmin(k0 + 3.0, top);
    const double l1 = u - k0, l2 = u - km1, l3 = u - km2, r1 = k1 - u, r2 = k2 - u, r3 = k3 - u;
    auto inv2 = [](double d) { return 1.5 - 0.5 * d; };  // d = 1, 2
    auto inv3 = [](double d) { return d == 3.0 ? 1.0 / 3.0 : 1.5 - 0.5 * d; };
    // degree 1: r1, l1 (the span is one knot wide); degree 2
    const double a0 = r1 * inv2(k1 - km1), a1 = l1 * inv2(k2 - k0);
    const double b0 = r1 * a0, b1 = l2 * a0 + r2 * a1, b2 = l1 * a1;
    // degree 3
    const double c0 = b0 * inv3(k1 - km2), c1 = b1 * inv3(k2 - km1), c2 = b2 * inv3(k3 - k0);
    N[0] = r1 * c0;
    N[1] = l3 * c0 + r2 * c1;
    N[2] = l2 * c1 + r3 * c2;
    N[3] = l1 * c2;
    const double h3 = 3.0 * ih;
    dN[0] = h3 * -c0;
    dN[1] = h3 * (c0 - c1);
    dN[2] = h3 * (c1 - c2);
    dN[3] = h3 * c2;
    first = (int)k0;
}

// d = xj - xi (minimum image), returns |d|^2
__device__ __forceinline__ double fit_fold(const double xi[3], const double xj[3], const Box &b,
                                           double d[3])
{
#pragma clang fp contract(off)
    for (int k = 0; k < 3; ++k) {
        double dx = xj[k] - xi[k];
        if (b.per[k]) {
            const double hh = 0.5 * b.L[k];
            dx = dx > hh ? dx - b.L[k] : (dx < -hh ? dx + b.L[k] : dx);
        }
        d[k] = dx;
    }
    double r2 = d[0] * d[0];
    r2 = r2 + d[1] * d[1];
    r2 = r2 + d[2] * d[2];
    return r2;
}

__device__ __forceinline__ double fit_disp(const double *__restrict__ pos, int n, int i, int j,
                                           const Box &b, double d[3])
{
    const double xi[3] = {pos[i], pos[n + i], pos[2 * n + i]};
    const double xj[3] = {pos[j], pos[n + j], pos[2 * n + j]};
    return fit_fold(xi, xj, b, d);
}

// ------------------------------------------------------------ design rows

struct FitShape {
    int ns, nk2, nk3, nd, n2cols;  // n2cols: 2-body columns (all species pairs)
    double rc2, rc3;
    double ih2, ih3, ih3c;         // knots per A: 2-body, 3-body legs, third side
};

// 2-body column k decoded: species pair a <= b, spline p.
struct FitCol {
    int a, b, p;
};

__device__ __forceinline__ FitCol fit_decode2(const FitShape &sh, int k)
{
    FitCol c{-1, -1, 0};
    if (k >= sh.n2cols)
        return c;
    const int nf2 = sh.nk2 - 1;  // nb2 - 3
    int pair = k / nf2;
    c.p = k - pair * nf2;
    for (int za = 0; za < sh.ns; ++za) {
        const int row = sh.ns - za;
        if (pair < row) {
            c.a = za;
            c.b = za + pair;
            break;
        }
        pair -= row;
    }
    return c;
}

// Entry of the list of i's neighbours inside the 3-body cutoff, the leg
// functions that are fitted written out densely (at most four: FitDims), with
// a zero that selections of no function read.
struct FitLeg {
    int j, z;
    double d[3], u[3], B[5], dB[5];  // d = x_j - x_i, u = d / |d|
};

// One configuration of a batched design launch (everything per workspace).
struct FitCfgDev {
    int n, cap;
    const int *nbr, *cnt;
    const double *pos;
    const int32_t *species;
    double *rows, *erow;
    int *l3, *l3cnt, *hdr;
    Box box;
};
// Configurations of one launch, passed by value as kernel arguments; the
// workgroup of global atom b belongs to the configuration whose atom range
// [atom0[c], atom0[c+1]) holds b.
struct FitBatch {
    int ncfg, ld;
    int atom0[kFitBatch + 1];
    FitCfgDev c[kFitBatch];
};

static_assert(sizeof(FitBatch) + 64 <= 4096, "design launch arguments exceed 4 KB");

__device__ __forceinline__ int fit_cfg_of(const FitBatch &B, int b)
{
    // one bound per lane instead of a chain of dependent reads (kFitBatch <= 64)
    const int l = threadIdx.x & 63;
    return __popcll(__ballot(l + 1 < B.ncfg && B.atom0[min(l + 1, kFitBatch)] <= b));
}

constexpr int kFitRec = 64;   // triplet records per batch
constexpr int kFitLegs = 32;  // 3-body neighbours per atom in the design kernel

// Sizes of the 3-body part for NF3 fitted functions per leg (knots - 1) and CG
// groups of four columns (species x third-side function). The limit of
// kFitMaxParams columns leaves NF3 = 3 (one or two species) and 4 (one): five
// functions alone would take 15 x 8 = 120 columns.
template <int NF3, int CG>
struct FitDims {
    static constexpr int NPQ = NF3 * (NF3 + 1) / 2, NB3 = NF3 + 3;
    // record of a leg triplet: the other leg's functions (four), the weights
    // 1 and the third side's direction, the third-side functions and their
    // derivatives; of a centred one: the third-side functions. Odd strides:
    // neither the lanes' row writes nor the column reads conflict.
    static constexpr int B = 0, W = 4, C = 8, E = C + NB3, RS = (E + NB3) | 1, RC = NB3 | 1;
};
__host__ __device__ inline int fit_pair_stride(int nf2) { return (2 * nf2 + 3) | 1; }

// Value of the lane with the same lane / 16 and lane % 4 in block BLK of the
// four blocks (lane / 4 % 4): a block of a 4x4x4 result as the right operand of
// another 4x4x4 step, for all of its blocks.
template <int BLK>
__device__ __forceinline__ double fit_from_block(double v)
{
    constexpr int pat = (4 * BLK) << 5 | 0x13;  // swizzle: keep lane bits 0, 1, 4; set the block
    union {
        double d;
        int w[2];
    } x{v};
    x.w[0] = __builtin_amdgcn_ds_swizzle(x.w[0], pat);
    x.w[1] = __builtin_amdgcn_ds_swizzle(x.w[1], pat);
    return x.d;
}

// Design rows of one atom per wavefront, as small dense products on the FP64
// matrix cores in 4x4x4 steps of four blocks (16 cycles; the dimensions here
// are about 4 and 7, where a 16x16x4 step would be mostly padding).
// 2-body: 4 rows (components, energy) x 16 columns per step over the pairs.
// 3-body, leg pair (p1, p2), third side s, per 3-body neighbour j of i with leg
// functions a_j and direction u_j (b_jk: the other leg's functions):
//   centred on i:  T[p][s]    = sum_k b_ik[p] C_jk[s]
//                  E  += a_j T / 2,  F_q += u_jq a'_j T    (symmetrised over p1, p2)
//   centred on j:  T[p][s]    = sum_k b_jk[p] C_ik[s],
//                  T_q[p][s]  = sum_k b_jk[p] w_ikq C'_ik[s]
//                  F_q += u_jq a'_j T + a_j T_q
// so the sums over the records have four functions p as rows (the four blocks:
// T and T_q, or four column groups of T), and the leg pairs appear once per j.
// Bound by the FP64 vector work of building the records (splines, square
// roots, reciprocals), which all 64 lanes share, and its latency.
// 41,000 atoms, 81 columns: 3,053 -> 689 us.
template <int NF3, int CG>
__global__ void __launch_bounds__(kFitWave) k_fit_design(FitBatch Bt, FitShape sh, int rb2)
{
    using FD = FitDims<NF3, CG>;
    constexpr int NPQ = FD::NPQ, NB3 = FD::NB3, RS = FD::RS;
    constexpr bool three = NF3 > 0;
    extern __shared__ double rec[];
    __shared__ FitLeg leg[three ? kFitLegs : 1];
    __shared__ int legpre[kFitLegs + 1];
    __shared__ int rz[kFitWave];
    const int cfg = fit_cfg_of(Bt, blockIdx.x);
    const FitCfgDev &Cf = Bt.c[cfg];
    const int n = Cf.n, cap = Cf.cap, ld = Bt.ld;
    const int *__restrict__ nbr = Cf.nbr;
    const int *__restrict__ cnt = Cf.cnt;
    const double *__restrict__ pos = Cf.pos;
    const int32_t *__restrict__ species = Cf.species;
    double *__restrict__ rows = Cf.rows;
    double *__restrict__ erow = Cf.erow;
    const int *__restrict__ l3 = Cf.l3;
    const int *__restrict__ l3cnt = Cf.l3cnt;
    int *__restrict__ hdr = Cf.hdr;
    const Box box = Cf.box;
    const int i = blockIdx.x - Bt.atom0[cfg];
    const int lane = threadIdx.x;
    if (i >= n)
        return;  // uniform: one wavefront per workgroup
    const int kg = lane >> 4, l16 = lane & 15;  // inner index of a step; row or column
    const int nf2 = sh.nk2 - 1, rs2 = fit_pair_stride(nf2);
    const int zi = sp_clamp(species[i], sh.ns);
    const double rc2sq = sh.rc2 * sh.rc2, rc3sq = sh.rc3 * sh.rc3;
    const int ci = cnt[i] < cap ? cnt[i] : cap;

    // ---- 1. pairs of i (2-body columns), and the list of its 3-body legs
    constexpr int T2 = (kFitMaxParams + 15) / 16;
    const int nt2 = (sh.n2cols + 15) / 16;
    double acc2[T2];
    int need[T2], col2[T2];  // this lane's column 16 t + l16: partner species, spline
#pragma unroll
    for (int t = 0; t < T2; ++t) {
        acc2[t] = 0.0;
        need[t] = -2;
        col2[t] = 0;
        if (t < nt2) {
            const FitCol c = fit_decode2(sh, 16 * t + l16);
            need[t] = c.a == zi ? c.b : (c.b == zi ? c.a : -2);
            col2[t] = c.p;
        }
    }
    int m = 0;  // legs
    for (int base = 0; base < ci; base += rb2) {
        const int slot = base + lane;
        bool in2 = false, in3 = false;
        double d[3] = {0.0, 0.0, 0.0}, r2 = 0.0;
        int j = -1;
        if (lane < rb2 && slot < ci) {
            j = nbr[(size_t)i * cap + slot];
            if (j >= 0 && j < n) {
                r2 = fit_disp(pos, n, i, j, box, d);
                in2 = r2 < rc2sq;
                in3 = three && r2 < rc3sq;
            }
        }
        const unsigned long long m2 = __ballot(in2), m3 = __ballot(in3);
        const int nv = __popcll(m2), nv4 = (nv + 3) & ~3;
        const double r = sqrt(r2);
        if (in2) {
            const int at = __popcll(m2 & ((1ull << lane) - 1ull));
            double *q = rec + at * rs2;
            int fb;
            double Bw[4], dBw[4];
            fit_bspline(r, sh.nk2, sh.ih2, fb, Bw, dBw);
            for (int k = 0; k < 2 * nf2; ++k)
                q[k] = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (fb + k < nf2) {
                    q[fb + k] = Bw[k];
                    q[nf2 + fb + k] = dBw[k];
                }
            const double ir = 1.0 / r;
            for (int k = 0; k < 3; ++k)
                q[2 * nf2 + k] = d[k] * ir;
            rz[at] = sp_clamp(species[j], sh.ns);
        }
        if (lane >= nv && lane < nv4) {  // rows that pad the inner dimension
            for (int k = 0; k < rs2; ++k)
                rec[lane * rs2 + k] = 0.0;
            rz[lane] = -1;
        }
        if constexpr (three) {
            const int at = m + __popcll(m3 & ((1ull << lane) - 1ull));
            if (in3) {
                if (at < kFitLegs) {
                    FitLeg &G = leg[at];
                    G.j = j;
                    G.z = sp_clamp(species[j], sh.ns);
                    const double ir = 1.0 / r;
                    for (int k = 0; k < 3; ++k) {
                        G.d[k] = d[k];
                        G.u[k] = d[k] * ir;
                    }
                    int f;
                    double B[4], dB[4];
                    fit_bspline(r, NF3 + 1, sh.ih3, f, B, dB);
#pragma unroll
                    for (int k = 0; k < 5; ++k) {
                        G.B[k] = 0.0;
                        G.dB[k] = 0.0;
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (f + k < NF3) {
                            G.B[f + k] = B[k];
                            G.dB[f + k] = dB[k];
                        }
                } else {
                    atomicOr(&hdr[H_STATUS], MLMIX_STATUS_TRIPLET_OVERFLOW);
                }
            }
            m = min(m + __popcll(m3), kFitLegs);
        }
        fit_wave_sync();
        const int row = lane & 3;
        for (int k0 = 0; k0 < nv4; k0 += 16) {
            // four steps, their operands read first (masked steps add zeros)
            const double *q[4];
            int zr[4];
            double av[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int s = min(k0 + 4 * v, nv4 - 4) + kg;
                q[v] = rec + s * rs2;
                zr[v] = k0 + 4 * v < nv4 ? rz[s] : -1;
                av[v] = row < 3 ? q[v][2 * nf2 + row] : 0.0;
            }
            const double ae = row == 3 ? 0.5 : 0.0;
#pragma unroll
            for (int t = 0; t < T2; ++t)
                if (t < nt2) {
                    double bd[4], bv[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        bd[v] = q[v][nf2 + col2[t]];
                        bv[v] = q[v][col2[t]];
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const bool on = zr[v] == need[t];
                        acc2[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[v], on ? bd[v] : 0.0, acc2[t], 0, 0, 0);
                        acc2[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(ae, on ? bv[v] : 0.0, acc2[t], 0, 0, 0);
                    }
                }
        }
        fit_wave_sync();
    }
    // lane holds [row kg (component, or energy)][column 16 t + l16]
#pragma unroll
    for (int t = 0; t < T2; ++t) {
        const int c = 16 * t + l16;
        if (c < sh.n2cols) {
            if (kg < 3)
                rows[(size_t)(1 + (size_t)kg * n + i) * ld + c] = acc2[t];
            else
                erow[(size_t)c * n + i] = acc2[t];
        }
    }

    if constexpr (three) {
        const int l4 = lane & 3, blk = (lane >> 2) & 3;
        // rows of the leg-pair products: (p1, p2) = row l16, inner index p =
        // kg; gi selects the leg function that meets T[p] there (4: none)
        int gi = 4;
        {
            int idx = 0;
#pragma unroll
            for (int p1 = 0; p1 < NF3; ++p1)
#pragma unroll
                for (int p2 = p1; p2 < NF3; ++p2, ++idx)
                    if (idx == l16)
                        gi = kg == p2 ? p1 : (kg == p1 ? p2 : 4);
        }
        // columns c = (species, third side): 4 g + l4 of the results, and 4 blk
        // + l4 where the blocks are the column groups
        int cz[CG], cs[CG];
#pragma unroll
        for (int g = 0; g < CG; ++g) {
            const int c = 4 * g + l4;
            cz[g] = c < sh.ns * NB3 ? c / NB3 : -2;
            cs[g] = c % NB3;
        }
        const int cb = 4 * blk + l4;
        const bool onb = cb < sh.ns * NB3 && cb / NB3 == zi;
        const int csb = cb % NB3;
        double accF[3][CG], accE[CG];
#pragma unroll
        for (int g = 0; g < CG; ++g) {
            accE[g] = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q)
                accF[q][g] = 0.0;
        }

        // ---- 2. triplets centred on i: for each leg a the other legs b (a
        // multiple of four slots per a; unused ones hold zeros)
        const int mp = (m + 3) & ~3;
        {
            double tc = 0.0;
            int a = 0, end = mp;
            auto flush = [&]() {
                const FitLeg &G = leg[a];
                const double ga = 0.5 * G.B[gi], gd = G.dB[gi];  // T counts a pair twice
                double t[CG];
                t[0] = fit_from_block<0>(tc);
                if constexpr (CG > 1)
                    t[1] = fit_from_block<1>(tc);
                if constexpr (CG > 2)
                    t[2] = fit_from_block<2>(tc);
#pragma unroll
                for (int g = 0; g < CG; ++g) {
                    accE[g] = __builtin_amdgcn_mfma_f64_4x4x4f64(ga, t[g], accE[g], 0, 0, 0);
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        accF[q][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(gd * G.u[q], t[g], accF[q][g], 0, 0, 0);
                }
                tc = 0.0;
                ++a;
                end += mp;
            };
            const int total = m * mp;
            for (int base = 0; base < total; base += kFitRec) {
                const int nr = min(kFitRec, total - base);
                if (lane < nr) {
                    const int ra = (base + lane) / mp, rb = base + lane - ra * mp;
                    double *q = rec + lane * FD::RC;
#pragma unroll
                    for (int k = 0; k < NB3; ++k)
                        q[k] = 0.0;
                    if (rb < m && rb != ra) {
                        double dd[3];
                        for (int k = 0; k < 3; ++k)
                            dd[k] = leg[rb].d[k] - leg[ra].d[k];
                        const double r = sqrt(dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2]);
                        int f;
                        double N[4], dN[4];
                        fit_bspline(r, NF3 + 1, sh.ih3c, f, N, dN);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            q[f + k] = N[k];
                    }
                }
                fit_wave_sync();
                // up to four steps of one leg at a time, their operands read
                // before the first (masked steps add zeros)
                for (int k0 = 0; k0 < nr;) {
                    if (base + k0 == end)
                        flush();
                    const int ns4 = min(min(16, nr - k0), end - base - k0);
                    double av[4], bv[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int s = min(k0 + 4 * v, nr - 4) + kg;
                        av[v] = leg[min(base + s - (end - mp), m - 1)].B[l4];
                        bv[v] = rec[s * FD::RC + csb];
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        tc = __builtin_amdgcn_mfma_f64_4x4x4f64(av[v], onb && 4 * v < ns4 ? bv[v] : 0.0, tc, 0, 0, 0);
                    k0 += ns4;
                }
                fit_wave_sync();
            }
            if (m > 0)
                flush();
        }

        // ---- 3. triplets centred on a 3-body neighbour j with i as one leg:
        // the other leg k runs over j's own 3-body list (k != i), again a
        // multiple of four slots per j
        const int own = lane < m ? l3cnt[leg[lane].j] : 0, pad = (own + 3) & ~3;
        int pre = pad;
        for (int o = 1; o < kFitLegs; o <<= 1) {
            const int v = __shfl_up(pre, o);
            pre += lane >= o ? v : 0;
        }
        if (lane < m) {
            legpre[lane] = pre - pad;
            rz[lane] = own;
        }
        const int total = __shfl(pre, kFitLegs - 1);
        if (lane == 0)
            legpre[m] = total;
        fit_wave_sync();
        {
            double t[CG];
#pragma unroll
            for (int g = 0; g < CG; ++g)
                t[g] = 0.0;
            int a = 0, end = m > 0 ? legpre[1] : 0;
            int fb[CG];  // this lane's right operand: C (block 0) or its derivative
#pragma unroll
            for (int g = 0; g < CG; ++g)
                fb[g] = (blk == 0 ? FD::C : FD::E) + cs[g];
            auto flush = [&]() {
                const FitLeg &G = leg[a];
                const double ga = G.B[gi], gd = G.dB[gi];
#pragma unroll
                for (int g = 0; g < CG; ++g) {
                    const double t0 = fit_from_block<0>(t[g]);
                    const double tq[3] = {fit_from_block<1>(t[g]), fit_from_block<2>(t[g]),
                                          fit_from_block<3>(t[g])};
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        accF[q][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(gd * G.u[q], t0, accF[q][g], 0, 0, 0);
                        accF[q][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(ga, tq[q], accF[q][g], 0, 0, 0);
                    }
                    t[g] = 0.0;
                }
                ++a;
                end = legpre[min(a + 1, m)];
            };
            // the partner of a slot and both positions are read a batch ahead
            int ra = 0, k = -1;
            double xj[3], xk[3];
            auto fetch = [&](int tt) {
                ra = 0;  // the last leg whose slots start at or before tt
                k = -1;
                if (tt >= total)
                    return;
                for (int w = kFitLegs / 2; w > 0; w >>= 1)
                    if (ra + w < m && legpre[ra + w] <= tt)
                        ra += w;
                const int j = leg[ra].j, idx = tt - legpre[ra];
                if (idx < rz[ra])
                    k = l3[(size_t)j * kMaxTriplet + idx];
                const int kc = k >= 0 && k < n ? k : j;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    xj[c] = pos[c * n + j];
                    xk[c] = pos[c * n + kc];
                }
            };
            fetch(lane);
            for (int base = 0; base < total; base += kFitRec) {
                const int nr = min(kFitRec, total - base);
                if (lane < nr) {
                    const FitLeg &Ga = leg[ra];
                    double *q = rec + lane * RS;
#pragma unroll
                    for (int c = 0; c < RS; ++c)
                        q[c] = 0.0;
                    if (k >= 0 && k < n && k != i) {
                        double djk[3];
                        const double r2jk = fit_fold(xj, xk, box, djk);
                        if (r2jk < rc3sq) {
                            double d3[3];
                            for (int c = 0; c < 3; ++c)
                                d3[c] = Ga.d[c] + djk[c];
                            const double r3 = sqrt(d3[0] * d3[0] + d3[1] * d3[1] + d3[2] * d3[2]);
                            int f;
                            double N[4], dN[4];
                            fit_bspline(r3, NF3 + 1, sh.ih3c, f, N, dN);
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                q[FD::C + f + c] = N[c];
                                q[FD::E + f + c] = dN[c];
                            }
                            fit_bspline(sqrt(r2jk), NF3 + 1, sh.ih3, f, N, dN);
#pragma unroll
                            for (int c = 0; c < 4; ++c)
                                if (f + c < NF3)
                                    q[FD::B + f + c] = N[c];
                            const double ir3 = 1.0 / r3;
                            q[FD::W] = 1.0;
#pragma unroll
                            for (int c = 0; c < 3; ++c)
                                q[FD::W + 1 + c] = d3[c] * ir3;
                        }
                    }
                }
                fetch(base + kFitRec + lane);
                fit_wave_sync();
                for (int k0 = 0; k0 < nr;) {
                    while (base + k0 >= end)
                        flush();
                    const int ns4 = min(min(16, nr - k0), end - base - k0);
                    const int zj = leg[a].z;
                    double av[4], bv[4][CG];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const double *q = rec + (min(k0 + 4 * v, nr - 4) + kg) * RS;
                        av[v] = q[FD::B + l4] * q[FD::W + blk];
#pragma unroll
                        for (int g = 0; g < CG; ++g)
                            bv[v][g] = q[fb[g]];
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int g = 0; g < CG; ++g)
                            t[g] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                av[v], cz[g] == zj && 4 * v < ns4 ? bv[v][g] : 0.0, t[g], 0, 0, 0);
                    k0 += ns4;
                }
                fit_wave_sync();
            }
            if (a < m)
                flush();
        }
        // lane holds [row 4 blk + kg = leg pair][column 4 g + l4]
        const int pq = 4 * blk + kg;
#pragma unroll
        for (int g = 0; g < CG; ++g) {
            if (cz[g] < 0 || pq >= NPQ)
                continue;
            const int c = sh.n2cols + (cz[g] * NPQ + pq) * NB3 + cs[g];
#pragma unroll
            for (int q = 0; q < 3; ++q)
                rows[(size_t)(1 + (size_t)q * n + i) * ld + c] = accF[q][g];
            erow[(size_t)c * n + i] = accE[g];
        }
    }
}

// Every atom's neighbours inside the 3-body cutoff, in row order (at most
// kMaxTriplet; more sets MLMIX_STATUS_TRIPLET_OVERFLOW).
__global__ void __launch_bounds__(kFitWave) k_fit_list3(FitBatch Bt, double rc3sq)
{
    const int cfg = fit_cfg_of(Bt, blockIdx.x);
    const FitCfgDev &Cf = Bt.c[cfg];
    const int n = Cf.n, cap = Cf.cap;
    const int *__restrict__ nbr = Cf.nbr;
    const int *__restrict__ cnt = Cf.cnt;
    const double *__restrict__ pos = Cf.pos;
    int *__restrict__ l3 = Cf.l3;
    int *__restrict__ l3cnt = Cf.l3cnt;
    int *__restrict__ hdr = Cf.hdr;
    const Box box = Cf.box;
    const int i = blockIdx.x - Bt.atom0[cfg];
    const int lane = threadIdx.x;
    if (i >= n)
        return;
    const int ci = cnt[i] < cap ? cnt[i] : cap;
    int m = 0;
    for (int base = 0; base < ci; base += kFitWave) {
        const int slot = base + lane;
        bool in3 = false;
        int j = -1;
        if (slot < ci) {
            j = nbr[(size_t)i * cap + slot];
            if (j >= 0 && j < n) {
                double d[3];
                in3 = fit_disp(pos, n, i, j, box, d) < rc3sq;
            }
        }
        const unsigned long long b = __ballot(in3);
        const int at3 = m + __popcll(b & ((1ull << lane) - 1ull));
        if (in3) {
            if (at3 < kMaxTriplet)
                l3[(size_t)i * kMaxTriplet + at3] = j;
            else
                atomicOr(&hdr[H_STATUS], MLMIX_STATUS_TRIPLET_OVERFLOW);
        }
        m += __popcll(b);
    }
    if (lane == 0)
        l3cnt[i] = m < kMaxTriplet ? m : kMaxTriplet;
}

// rows[0][k] = sum_i erow[k][i], one workgroup per (column, configuration),
// fixed order
__global__ void __launch_bounds__(256) k_fit_erow_sum(FitBatch Bt)
{
    __shared__ double sh[256];
    const int k = blockIdx.x;
    const FitCfgDev &Cf = Bt.c[blockIdx.y];
    const int n = Cf.n;
    const double *__restrict__ erow = Cf.erow;
    double *__restrict__ rows = Cf.rows;
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256)
        s += erow[(size_t)k * n + i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        rows[k] = sh[0];
}

void launch_fit_design(hipStream_t s, const Ctx &c, const FitCfgHost *cfg, int ncfg, int ld, int nd)
{
    FitShape sh;
    sh.ns = c.m.ns;
    sh.nk2 = c.d.uf3_n_knots2;
    sh.nk3 = c.d.uf3_n_knots3;
    sh.nd = nd;
    sh.n2cols = sh.ns * (sh.ns + 1) / 2 * (sh.nk2 - 1);
    sh.rc2 = c.d.uf3_rcut2;
    sh.rc3 = c.d.uf3_rcut3;
    sh.ih2 = (double)(sh.nk2 - 1) / sh.rc2;
    sh.ih3 = sh.nk3 > 1 ? (double)(sh.nk3 - 1) / sh.rc3 : 0.0;
    sh.ih3c = sh.nk3 > 1 ? (double)(sh.nk3 - 1) / (2.0 * sh.rc3) : 0.0;
    for (int c0 = 0; c0 < ncfg; c0 += kFitBatch) {
        FitBatch Bt{};
        Bt.ld = ld;
        int atoms = 0;
        for (int q = 0; q < kFitBatch && c0 + q < ncfg; ++q) {
            const FitCfgHost &h = cfg[c0 + q];
            const WsLayout &L = h.L;
            if (L.n == 0)
                continue;
            FitCfgDev &d = Bt.c[Bt.ncfg];
            d.n = L.n;
            d.cap = L.cap;
            d.nbr = at<int>(h.ws, L.nbr);
            d.cnt = at<int>(h.ws, L.cnt);
            d.pos = h.pos;
            d.species = h.species;
            d.rows = h.rows;
            d.erow = at<double>(h.ws, L.g);
            d.l3 = reinterpret_cast<int *>(d.erow + (size_t)nd * L.n);
            d.l3cnt = d.l3 + (size_t)kMaxTriplet * L.n;
            d.hdr = at<int>(h.ws, L.hdr);
            d.box = h.box;
            Bt.atom0[Bt.ncfg] = atoms;
            atoms += L.n;
            ++Bt.ncfg;
        }
        if (Bt.ncfg == 0)
            continue;
        Bt.atom0[Bt.ncfg] = atoms;
        if (sh.nk3 > 1)
            k_fit_list3<<<atoms, kFitWave, 0, s>>>(Bt, sh.rc3 * sh.rc3);
        auto go = [&](auto nf, auto cg) {
            using FD = FitDims<decltype(nf)::value, decltype(cg)::value>;
            const size_t rs2 = fit_pair_stride(sh.nk2 - 1) * sizeof(double);
            // pair records per batch: 64 unless many knots make them long
            const int rb2 = rs2 * 64 <= 32 * 1024 ? 64 : (rs2 * 32 <= 32 * 1024 ? 32 : 16);
            size_t lds = rs2 * rb2;
            if (sh.nk3 > 1)
                lds = std::max(lds, (size_t)kFitRec * FD::RS * sizeof(double));
            k_fit_design<decltype(nf)::value, decltype(cg)::value><<<atoms, kFitWave, lds, s>>>(Bt, sh, rb2);
        };
        if (sh.nk3 <= 1)
            go(std::integral_constant<int, 0>(), std::integral_constant<int, 1>());
        else if (sh.nk3 == 5)
            go(std::integral_constant<int, 4>(), std::integral_constant<int, 2>());
        else if (sh.ns == 1)
            go(std::integral_constant<int, 3>(), std::integral_constant<int, 2>());
        else
            go(std::integral_constant<int, 3>(), std::integral_constant<int, 3>());
        k_fit_erow_sum<<<dim3(nd, Bt.ncfg), 256, 0, s>>>(Bt);
    }
}

// ------------------------------------------------------------------ Gram

constexpr int kGramRows = 32;  // rows staged per LDS pass

__host__ __device__ inline int fit_nblk(int nd) { return (nd + 3) / 4; }

// Upper-triangle 4x4 block index t -> (bi, bj), bi <= bj, row by row.
__device__ __forceinline__ void fit_blk(int t, int nb, int &bi, int &bj)
{
    bi = 0;
    while (t >= nb - bi) {
        t -= nb - bi;
        ++bi;
    }
    bj = bi + t;
}

__global__ void __launch_bounds__(256)
    k_fit_gram_partial(long long nrows, int nd, int ld, const double *__restrict__ A,
                       const double *__restrict__ y, const double *__restrict__ w,
                       long long chunk, double *__restrict__ part)
{
    const int nb = fit_nblk(nd), nd4 = nb * 4;
    const int nblk = nb * (nb + 1) / 2;
    __shared__ double tile[kGramRows][kFitMaxParams + 4];
    __shared__ double wy[kGramRows][2];
    const long long r0 = (long long)blockIdx.x * chunk;
    long long r1 = r0 + chunk;
    if (r1 > nrows)
        r1 = nrows;
    constexpr int kPer = (kFitMaxParams / 4) * (kFitMaxParams / 4 + 1) / 2 / 256 + 1;
    double acc[kPer][16];
    int bis[kPer], bjs[kPer];
    for (int u = 0; u < kPer; ++u) {
        const int t = threadIdx.x + 256 * u;
        bis[u] = -1;
        if (t < nblk)
            fit_blk(t, nb, bis[u], bjs[u]);
        for (int e = 0; e < 16; ++e)
            acc[u][e] = 0.0;
    }
    double bacc[4] = {0.0, 0.0, 0.0, 0.0};
    for (long long rb = r0; rb < r1; rb += kGramRows) {
        const int nr = (int)(r1 - rb < kGramRows ? r1 - rb : kGramRows);
        for (int e = threadIdx.x; e < kGramRows * nd4; e += 256) {
            const int r = e / nd4, k = e - r * nd4;
            tile[r][k] = (r < nr && k < nd) ? A[(size_t)(rb + r) * ld + k] : 0.0;
        }
        if ((int)threadIdx.x < kGramRows) {
            const int r = threadIdx.x;
            wy[r][0] = r < nr ? (w ? w[rb + r] : 1.0) : 0.0;
            wy[r][1] = r < nr ? (y ? y[rb + r] : 0.0) : 0.0;
        }
        __syncthreads();
        for (int r = 0; r < nr; ++r) {
            const double wr = wy[r][0];
            for (int u = 0; u < kPer; ++u) {
                if (bis[u] < 0)
                    continue;
                double ai[4], aj[4];
                for (int q = 0; q < 4; ++q) {
                    ai[q] = wr * tile[r][4 * bis[u] + q];
                    aj[q] = tile[r][4 * bjs[u] + q];
                }
                for (int p = 0; p < 4; ++p)
                    for (int q = 0; q < 4; ++q)
                        acc[u][4 * p + q] += ai[p] * aj[q];
            }
            if ((int)threadIdx.x < nb) {
                const double wyr = wr * wy[r][1];
                for (int q = 0; q < 4; ++q)
                    bacc[q] += wyr * tile[r][4 * threadIdx.x + q];
            }
        }
        __syncthreads();
    }
    double *out = part + (size_t)blockIdx.x * ((size_t)nblk * 16 + nd4);
    for (int u = 0; u < kPer; ++u) {
        const int t = threadIdx.x + 256 * u;
        if (t < nblk)
            for (int e = 0; e < 16; ++e)
                out[(size_t)t * 16 + e] = acc[u][e];
    }
    if ((int)threadIdx.x < nb)
        for (int q = 0; q < 4; ++q)
            out[(size_t)nblk * 16 + 4 * threadIdx.x + q] = bacc[q];
}

// G[k][l] += sum over chunks (both triangles written), b[k] += likewise
__global__ void __launch_bounds__(256) k_fit_gram_reduce(int nd, int nparts,
                                                         const double *__restrict__ part,
                                                         double *__restrict__ G,
                                                         double *__restrict__ bvec)
{
    const int nb = fit_nblk(nd), nd4 = nb * 4;
    const int nblk = nb * (nb + 1) / 2;
    const size_t stride = (size_t)nblk * 16 + nd4;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= nblk * 16 + nd4)
        return;
    // eight running sums (partial p goes to sum p mod 8) keep eight loads in
    // flight; they are combined in a fixed order
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int p = 0;
    for (; p + 8 <= nparts; p += 8)
        for (int q = 0; q < 8; ++q)
            acc[q] += part[(size_t)(p + q) * stride + e];
    for (int q = 0; p < nparts; ++p, ++q)
        acc[q] += part[(size_t)p * stride + e];
    const double s = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    if (e < nblk * 16) {
        int bi, bj;
        fit_blk(e / 16, nb, bi, bj);
        const int k = 4 * bi + (e % 16) / 4, l = 4 * bj + (e % 4);
        if (k < nd && l < nd) {
            if (bi != bj || k <= l) {
                G[(size_t)k * nd + l] += s;
                if (k != l)
                    G[(size_t)l * nd + k] += s;
            }
        }
    } else {
        const int k = e - nblk * 16;
        if (k < nd)
            bvec[k] += s;
    }
}

size_t fit_gram_parts(long long nrows, long long &chunk)
{
    long long parts = (nrows + 255) / 256;
    parts = parts < 1 ? 1 : (parts > 512 ? 512 : parts);
    chunk = (nrows + parts - 1) / parts;
    chunk = (chunk + kGramRows - 1) / kGramRows * kGramRows;
    if (chunk < kGramRows)
        chunk = kGramRows;
    parts = (nrows + chunk - 1) / chunk;
    return (size_t)(parts < 1 ? 1 : parts);
}

size_t fit_gram_part_bytes(int nd, size_t parts)
{
    const int nb = fit_nblk(nd);
    return parts * ((size_t)nb * (nb + 1) / 2 * 16 + (size_t)nb * 4) * sizeof(double);
}

void launch_fit_gram(hipStream_t s, long long nrows, int nd, int ld, const double *A,
                     const double *y, const double *w, double *G, double *b, double *part)
{
    if (nrows <= 0)
        return;
    long long chunk = 0;
    const size_t parts = fit_gram_parts(nrows, chunk);
    k_fit_gram_partial<<<(unsigned)parts, 256, 0, s>>>(nrows, nd, ld, A, y, w, chunk, part);
    const int nb = fit_nblk(nd);
    const int ne = nb * (nb + 1) / 2 * 16 + nb * 4;
    k_fit_gram_reduce<<<(ne + 255) / 256, 256, 0, s>>>(nd, (int)parts, part, G, b);
}

// ---------------------------------------------------------------- search

struct FitSearchArgs {
    int nd, nh, ldh;
    const double *GS, *bS, *AH, *yH, *wH;
    double alpha, tol, lam0, ridge;
    int max_decades, max_bisect;
    const double *GH, *bH;  // A_H^T W A_H and A_H^T W y_H (built before the search)
    double *c, *info;
};

typedef double fit_d4 __attribute__((ext_vector_type(4)));

// v of lane l (the same l on every lane)
__device__ __forceinline__ double fit_readlane(double v, int l)
{
    union {
        double d;
        int w[2];
    } x{v};
    x.w[0] = __builtin_amdgcn_readlane(x.w[0], l);
    x.w[1] = __builtin_amdgcn_readlane(x.w[1], l);
    return x.d;
}

// 1/sqrt(t) for t > 0: the hardware estimate and two Newton steps
__device__ __forceinline__ double fit_rsqrt(double t)
{
    double y = __builtin_amdgcn_rsq(t);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const double e = fma(-t * y, y, 1.0);
        y = fma(y * e, fma(e, 0.375, 0.5), y);
    }
    return y;
}

__device__ __forceinline__ double fit_wave_sum(double v)
{
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o);
    return v;
}

__global__ void __launch_bounds__(256) k_fit_search(FitSearchArgs a)
{
    // packed lower triangle of M plus the right-hand side as an extra row nd
    // (factorising that row performs the forward substitution)
    constexpr int kPacked = (kFitMaxParams + 1) * (kFitMaxParams + 2) / 2;
    // (sixteen entries past its end are read and not used, the last written
    // by lanes with nothing to store: the masked accesses need no branch)
    constexpr int kDump = kPacked + 16;
    __shared__ double Lp[kDump + 1];
    __shared__ double cur[kFitMaxParams], keep[kFitMaxParams], rdg[kFitMaxParams];
    __shared__ double red[4];
    __shared__ int fail;
    const int nd = a.nd, tid = threadIdx.x;
    auto P = [](int r, int c2) { return r * (r + 1) / 2 + c2; };  // r >= c2
    const int wv = tid >> 6, ln = tid & 63, kg = ln >> 4, l16 = ln & 15;
    // this thread's entries of the packed triangle: offset in the square
    // matrices, bit 16 on the diagonal
    constexpr int kOwn = (kFitMaxParams * (kFitMaxParams + 1) / 2 + 255) / 256;
    int own[kOwn];
#pragma unroll
    for (int u = 0; u < kOwn; ++u) {
        const int e = min(tid + 256 * u, nd * (nd + 1) / 2 - 1);
        int r = (int)((sqrtf(8.0f * (float)e + 1.0f) - 1.0f) * 0.5f);
        while (r * (r + 1) / 2 > e)
            --r;
        while ((r + 1) * (r + 2) / 2 <= e)
            ++r;
        const int c2 = e - r * (r + 1) / 2;
        own[u] = (r * nd + c2) | (r == c2 ? 1 << 16 : 0);
    }
    // one solve at lam: cur = c(lam); returns the hard residual (or -1 when
    // the factorisation meets a non-positive pivot)
    auto solve = [&](double lam) -> double {
        double gs[kOwn], gh[kOwn];
#pragma unroll
        for (int u = 0; u < kOwn; ++u) {  // every load in flight before the first use
            const int e = own[u] & 0xffff;
            gs[u] = a.GS[e];
            gh[u] = a.GH[e];
        }
#pragma unroll
        for (int u = 0; u < kOwn; ++u)
            if (tid + 256 * u < nd * (nd + 1) / 2)
                Lp[tid + 256 * u] = gs[u] + lam * gh[u] + (own[u] >> 16 ? a.ridge : 0.0);
        if (tid < nd)
            Lp[P(nd, tid)] = a.bS[tid] + lam * a.bH[tid];
        if (tid == 0)
            fail = 0;
        __syncthreads();
        // Cholesky in panels of 16 columns, row nd (the right-hand side) carried
        // along. Within a panel every lane holds one row's 16 entries: lanes
        // 0 .. 15 of each wavefront the diagonal block (all four the same),
        // the others 48 rows below it, so that a column needs no barrier: its
        // pivot and multipliers are read from the block's lanes. The trailing
        // matrix then takes 16x16x4 FP64 matrix steps. (One column at a time
        // with two barriers each: 115 us per solve at 81 parameters; panels:
        // 33 us.)
        for (int k0 = 0; k0 < nd; k0 += 16) {
            const int nbk = min(16, nd - k0);
            const int row = ln < 16 ? k0 + ln : k0 + ln + 48 * wv;
            const bool live = row <= nd;
            double *Lr = Lp + P(min(row, nd), 0) + k0;
            double x[16];
#pragma unroll
            for (int c = 0; c < 16; ++c)
                x[c] = Lr[c];
#pragma unroll
            for (int c = 0; c < 16; ++c)
                x[c] = live && c < nbk && k0 + c <= row ? x[c] : 0.0;
            double rj = 1.0;  // lane j: 1/L_jj of column k0 + j
            bool bad = false;
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (j < nbk) {  // uniform
                    const double tj = fit_readlane(x[j], j);
                    const double r = tj > 0.0 ? fit_rsqrt(tj) : 1.0;
                    const double l = x[j] * r;
                    x[j] = l;
#pragma unroll
                    for (int c = j + 1; c < 16; ++c)
                        x[c] -= l * fit_readlane(l, c);
                    rj = ln == j ? r : rj;
                    bad = bad || !(tj > 0.0);
                }
            if (tid < nbk)
                rdg[k0 + tid] = rj;
            if (tid == 0 && bad)
                fail = 1;
            __syncthreads();  // every wavefront has read its rows
            const bool keeps = live && (ln >= 16 || wv == 0);
#pragma unroll
            for (int c = 0; c < 16; ++c)
                *(keeps && c < nbk && k0 + c < row ? Lr + c : Lp + kDump) = x[c];
            __syncthreads();
            const int t0 = k0 + 16, nt = t0 <= nd ? (nd - t0) / 16 + 1 : 0;
            for (int t = wv, ti = 0, tj = wv; t < nt * (nt + 1) / 2; t += 4, tj += 4) {
                while (tj > ti) {  // tile (ti, tj), tj <= ti, row by row
                    tj -= ti + 1;
                    ++ti;
                }
                const int i0 = t0 + 16 * ti, j0 = t0 + 16 * tj;
                const int ia = i0 + l16, jb = j0 + l16;
                const double *La = Lp + P(min(ia, nd), 0) + k0 + kg;
                const double *Lb = Lp + P(min(jb, nd), 0) + k0 + kg;
                double av[4], bv[4], cv[4];
                double *Lc[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + 4 * u + kg;
                    Lc[u] = i <= nd && jb < nd && jb <= i ? Lp + P(i, jb) : Lp + kDump;
                    av[u] = La[4 * u];
                    bv[u] = Lb[4 * u];
                    cv[u] = *Lc[u];
                }
                fit_d4 acc = {cv[0], cv[1], cv[2], cv[3]};
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[u], bv[u], acc, 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    *Lc[u] = acc[u];
            }
            __syncthreads();
        }
        // row nd now holds x with L x = b; L^T c = x by wavefront 0, column
        // by column (c_j = x_j / L_jj, then x_k -= L_jk c_j for k < j): x and
        // 1/L_jj in registers, four rows of L read ahead of their columns
        if (wv == 0) {
            const int lo = min(ln, nd - 1), hi = min(ln + 64, nd - 1);
            double x0 = Lp[P(nd, lo)], x1 = Lp[P(nd, hi)];
            const double d0 = rdg[lo], d1 = rdg[hi];
            double c0 = 0.0, c1 = 0.0;
            for (int j0 = nd - 1; j0 >= 64; j0 -= 4) {  // columns 64 and up
                double l0[4], l1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double *Lj = Lp + P(max(j0 - u, 64), 0);
                    l0[u] = Lj[ln];
                    l1[u] = Lj[min(ln + 64, max(j0 - u, 64))];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 - u, jl = max(j - 64, 0);
                    const double v = fit_readlane(x1, jl) * fit_readlane(d1, jl);
                    const double cj = j >= 64 ? v : 0.0;
                    c1 = ln + 64 == j ? cj : c1;
                    x0 -= l0[u] * cj;
                    x1 -= ln + 64 < j ? l1[u] * cj : 0.0;
                }
            }
            for (int j0 = min(nd, 64) - 1; j0 >= 0; j0 -= 4) {
                double l0[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    l0[u] = Lp[P(max(j0 - u, 0), min(ln, max(j0 - u, 0)))];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 - u, jl = max(j, 0);
                    const double v = fit_readlane(x0, jl) * fit_readlane(d0, jl);
                    const double cj = j >= 0 ? v : 0.0;
                    c0 = ln == j ? cj : c0;
                    x0 -= ln < j ? l0[u] * cj : 0.0;
                }
            }
            if (ln < nd)
                cur[ln] = c0;
            if (ln + 64 < nd)
                cur[ln + 64] = c1;
        }
        __syncthreads();
        // hard residual: A_H c for 16 rows per wavefront and pass as 4x4x4 FP64
        // matrix steps (every column of the right operand is c), a pass's loads
        // eight steps ahead
        double part = 0.0;
        for (int h0 = 16 * wv; h0 < a.nh; h0 += 64) {
            const double *src = a.AH + (size_t)min(h0 + l16, a.nh - 1) * a.ldh;
            double r = 0.0;
            for (int k0 = 0; k0 < nd; k0 += 32) {
                double av[8], cv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int k = k0 + 4 * u + kg;
                    av[u] = src[min(k, nd - 1)];
                    cv[u] = k < nd ? cur[k] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    r = __builtin_amdgcn_mfma_f64_4x4x4f64(av[u], cv[u], r, 0, 0, 0);
            }
            // lane holds row 4 (lane / 4 % 4) + kg (the same in four columns)
            const int h = h0 + 4 * ((ln >> 2) & 3) + kg;
            if ((ln & 3) == 0 && h < a.nh) {
                const double d = r - a.yH[h];
                part += (a.wH ? a.wH[h] : 1.0) * d * d;
            }
        }
        const double ps = fit_wave_sum(part);
        if (ln == 0)
            red[wv] = ps;
        __syncthreads();
        const double res = (red[0] + red[1]) + (red[2] + red[3]);
        __syncthreads();
        return fail ? -1.0 : res;
    };
    auto save = [&]() {
        if (tid < nd)
            keep[tid] = cur[tid];
        __syncthreads();
    };

    // the search as one loop around one solve (its code is long: a copy per
    // call site would not fit the instruction cache): the first lambda, decades
    // until the residual is at most alpha, then bisection
    int nsolve = 0, status = 0, dec = 0, it = 0;
    bool bisect = false;
    double lam = a.lam0, lam_lo = lam, out_lam = lam, out_res = 0.0, best_res = 0.0, best_lam = lam;
    double lo = lam, hi = lam, r_hi = 0.0;
    for (;;) {
        const double res = solve(lam);
        ++nsolve;
        if (!bisect) {
            if (nsolve == 1 || (res >= 0.0 && res < best_res)) {
                best_res = res;
                best_lam = lam;
                save();
            }
            if (res > a.alpha && dec < a.max_decades) {
                lam_lo = lam;
                lam *= 10.0;
                ++dec;
                continue;
            }
            out_lam = best_lam;
            out_res = best_res;
            if (res < 0.0 || res > a.alpha) {
                status = res < 0.0 ? 3 : 1;
                break;
            }
            if (dec == 0)
                break;
            // lo fails, hi passes (keep holds c(hi))
            lo = lam_lo;
            hi = lam;
            r_hi = res;
            save();
            bisect = true;
        } else {
            if (res < 0.0) {
                status = 3;
            } else if (res <= a.alpha) {
                hi = lam;
                r_hi = res;
                save();
            } else {
                lo = lam;
            }
            ++it;
        }
        out_lam = hi;
        out_res = r_hi;
        lam_lo = lo;
        if (status == 3 || a.alpha - r_hi < a.tol)
            break;
        if (it == a.max_bisect) {
            status = 2;
            break;
        }
        lam = 0.5 * (lo + hi);
    }
    if (tid < nd)
        a.c[tid] = keep[tid];
    if (tid == 0) {
        a.info[0] = out_lam;
        a.info[1] = out_res;
        a.info[2] = (double)nsolve;
        a.info[3] = (double)status;
        a.info[4] = lam_lo;
        a.info[5] = (double)dec;
    }
}

void launch_fit_search(hipStream_t s, int nd, int nh, int ldh, const double *GS, const double *bS,
                       const double *AH, const double *yH, const double *wH, double alpha,
                       double tol, double lam0, double ridge, int max_decades, int max_bisect,
                       double *c, double *info, double *scratch)
{
    // G_H, b_H by the Gram kernels (zeroed by a fill kernel first), then the
    // search in one workgroup
    double *GH = scratch, *bH = scratch + (size_t)nd * nd, *part = bH + nd;
    launch_fill_f64(s, GH, 0.0, (size_t)nd * nd + nd);
    launch_fit_gram(s, nh, nd, ldh, AH, yH, wH, GH, bH, part);
    FitSearchArgs a{nd, nh, ldh, GS, bS, AH, yH, wH, alpha, tol, lam0, ridge, max_decades, max_bisect,
                    GH, bH, c, info};
    k_fit_search<<<1, 256, 0, s>>>(a);
}

}  // namespace mlmix

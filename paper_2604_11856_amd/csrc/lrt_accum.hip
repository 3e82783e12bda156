// gfx950 kernels of the line-by-line path (arXiv 2604.11856): populations,
// line setups and the line-to-grid accumulation.
//
//   thermo      per (cell, species): partition function, ln(N/Q), Doppler
//               coefficient; per cell: beta's, Lorentz HWHM, line-skip bound
//               (Sec. 2.1 Boltzmann populations, Sec. 2.2.1 widths); the
//               QSS-CR populations of selected species come from lrt_cr.hip
//               and enter the line setup as departures from Boltzmann
//   ranges      per (cell, tile): index range of the nu0-sorted lines that
//               can reach the tile
//   scale       per cell: power-of-two scale of the single-precision eta/kappa
//   accum_*     per (cell, tile): stage per-(cell, line) setups in LDS (FP64),
//               then every lane accumulates the Whiting-Voigt profile of each
//               staged line at its own grid points (Sec. 2.2.1)
//   count       per (cell, candidate line): in-window and core term counts
//   serve       serving kernel: profiles + march of request chunks, one
//               workgroup per item, and the composition of finished tiles
// The march of the path and its reductions live in lrt_march.hip.
//
// Everything is output-stationary: each output element has one owner, so no
// atomics touch eta, kappa, I or the flux; sums run in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <climits>
#include <cstdint>
#include <cmath>
#include <type_traits>

#include "lrt_device.h"
#include "lrt_internal.h"
#include "lrt_math.h"
#include "lrt_nodes.h"

namespace lrt {

namespace {


// ---------------------------------------------------------------------------
// a1: partition functions and per-cell constants (FP64)
// ---------------------------------------------------------------------------

// van der Waals HWHM (cm^-1) of the lines of atom s in cell c: the printed
// lambda^2 [6.65e-29 N_s (2T/M_s)^0.5 + 2.925e-29 N_o (2T/M_o)^0.5] nm times
// 1e7/lambda^2; N_o, M_o over the other species but electrons (M < 0.01).
__device__ double vdw_width(const DevSpecies &sp, const DevCells &cells, int c, int s)
{
    const int S = cells.n_species;
    const double Ttr = cells.T_tr[c];
    double No = 0.0, NMo = 0.0;
    for (int t = 0; t < S; ++t) {
        if (t == s || sp.mass[t] < 0.01) continue;
        const double n = cells.N[(int64_t)c * S + t];
        No += n;
        NMo += n * sp.mass[t];
    }
    double w = 6.65e-29 * cells.N[(int64_t)c * S + s] * sqrt(2.0 * Ttr / sp.mass[s]);
    if (No > 0.0) w += 2.925e-29 * No * sqrt(2.0 * Ttr / (NMo / No));
    return 1e7 * w;
}

// Per-cell constants and, per (cell, species), the Doppler coefficient and
// ln(N/Q) with Q the partition function of an atom (Sec. 2.1, electronic
// levels) or a molecule (Sec. 2.1 molecular Boltzmann relation: Q = sum_e g_e
// e^{-beta_v T_e} sum_v e^{-beta_v G_v} sum_J (2J+1) e^{-beta_tr (B_v J(J+1) -
// D_v J^2(J+1)^2)}).  One wave per (cell, species): lane l takes levels l (mod
// 64), or of every (e, v) the J = l (mod 64), then the lanes are summed in a
// fixed butterfly order.  Where all vibrational levels of a state have the same
// rotational constants (a rigid rotor) the vibrational and the rotational sum
// factor.  Bound by the exponentials' instructions: 32,768 cells with four
// molecules of 50 levels and 152 J each took 3.54 ms with a rotational sum per
// level and the library's exponential, 0.28 ms so (1.28 where the constants
// differ); on 8 cells of two atoms, an atom's levels one after the other and the
// molecules in a launch of their own, 7.8 us, 4.8 so.
__global__ __launch_bounds__(64) void thermo_kernel(DevSpecies sp, DevCells cells, DevWidths wd, double M_min,
                                                    uint64_t mask, CellConst *cc, CellSpecies *cs)
{
    const int S = cells.n_species;
    const int64_t t = blockIdx.x;
    const int c = (int)(t / S), s = (int)(t % S);
    const int lane = threadIdx.x;
    const double Tv = cells.T_v[c], Ttr = cells.T_tr[c];
    const double bv = kC2 / Tv, br = kC2 / Ttr;
    const int kind = sp.kind[s];
    double Q = 0.0;
    if (kind == 1) {
        for (int64_t j = sp.lev_off[s] + lane; j < sp.lev_off[s + 1]; j += 64)
            Q += sp.lev_g[j] * exp_any(-bv * sp.lev_E[j]);
    } else if (kind == 2) {
        // this lane's part of the rotational sum of constants (B, D)
        auto rotational = [&](double B, double D, int Jmax) {
            double qr = 0.0;
            for (int J = lane; J <= Jmax; J += 64) {
                const double jj = (double)J * (J + 1.0);
                qr += (2.0 * J + 1.0) * exp_any(-br * (B * jj - D * jj * jj));
            }
            return qr;
        };
        for (int64_t e = sp.el_off[s]; e < sp.el_off[s + 1]; ++e) {
            const int Jmax = sp.el_Jmax[e];
            const int64_t v0 = sp.vib_off[e], v1 = sp.vib_off[e + 1];
            double qvr = 0.0;
            // every level with the first one's constants: the two sums factor
            const double B0 = sp.vib_B[v0], D0 = sp.vib_D[v0];
            bool same = true;
            for (int64_t v = v0 + lane; v < v1; v += 64) same = same && sp.vib_B[v] == B0 && sp.vib_D[v] == D0;
            if (__all(same)) {
                for (int64_t v = v0 + lane; v < v1; v += 64) qvr += exp_any(-bv * sp.vib_G[v]);
                for (int o = 32; o > 0; o >>= 1) qvr += __shfl_xor(qvr, o);
                qvr *= rotational(B0, D0, Jmax);
            } else {
                for (int64_t v = v0; v < v1; ++v)
                    qvr += exp_any(-bv * sp.vib_G[v]) * rotational(sp.vib_B[v], sp.vib_D[v], Jmax);
            }
            Q += sp.el_g[e] * exp_any(-bv * sp.el_T[e]) * qvr;
        }
    }
    if (kind == 1 || kind == 2)
        for (int o = 32; o > 0; o >>= 1) Q += __shfl_xor(Q, o);
    if (lane == 0) {
        const double N = cells.N[(int64_t)c * S + s];
        CellSpecies o;
        // species outside a non-zero mask carry no lines (bit s of mask)
        o.lnNQ = (species_on(mask, s) && kind != 0 && N > 0.0 && Q > 0.0) ? log(N) - log(Q) : -INFINITY;
        o.dop = 7.16233e-7 / 2.0 * sqrt(Ttr / sp.mass[s]);
        o.gW = (wd.E_ion && kind == 1 && wd.E_ion[s] > 0.0) ? vdw_width(sp, cells, c, s) : 0.0;
        cs[t] = o;
    }
    if (s == 0 && lane == 1) {
        CellConst k;
        k.beta_v = bv;
        k.beta_tr = br;
        k.gL = 1e-16 * cells.n_e[c] * pow(Tv / 1e4, 0.33);
        // Voigt HWHM <= gL + gG, gG = dop(M) nu0 <= dop(M_min) nu0; widened.
        // gL of any line <= gN_max + gS_max gL(c) + the largest van der Waals width.
        double gWmax = 0.0;
        if (wd.E_ion)
            for (int s2 = 0; s2 < S; ++s2)
                if (sp.kind[s2] == 1 && wd.E_ion[s2] > 0.0) gWmax = fmax(gWmax, vdw_width(sp, cells, c, s2));
        k.cand_G = 100.0 * (wd.gN_max + wd.gS_max * k.gL + gWmax) * (1.0 + 1e-6);
        k.cand_A = 100.0 * (7.16233e-7 / 2.0) * sqrt(Ttr / M_min) * (1.0 + 1e-6);
        cc[c] = k;
    }
}

// ---------------------------------------------------------------------------
// a2: one (cell, line) pair in FP64
// ---------------------------------------------------------------------------

struct PairF64 {
    double se, sk;        // eta and kappa per unit profile shape (strength * norm)
    double inv2g, r;      // 1 / (2 gamma_V), gamma_L / gamma_V
    int32_t klo, khi;     // inclusive window, klo > khi when empty
    int32_t kclo, kchi;   // core: points with |nu_k - nu0| <= kCoreHalfWidth gamma_V
};

// Half-width of the single-precision core in units of gamma_V, where the
// profile's two exponential terms are evaluated.  Beyond it x = |dnu|/(2
// gamma_V) > 6, and with the staged normalisation s = max(r, 2^-40) the
// exponential part (1-r)/s e^{-2.772 x^2} + 0.016 r(1-r)/s e^{-0.4 x^2.25}
// is below 5.1e-32 + 2.7e-12, while the rational part 1/(1+4x^2) -
// 0.016(1-r)/(1+0.1 x^2.25) is at least 4.48e-3 (both ratios fall with x):
// the omitted part is below 2^-30 of the term, under a quarter of the
// single-precision rounding of the term itself.  (At 25 gamma_V both
// exponentials are exactly zero in single precision; the narrower core
// halves the terms that evaluate them.)
constexpr double kCoreHalfWidth = 12.0;

// The cell's row of ln departures from Boltzmann (QSS-CR populations), or
// NULL when no line has levels.
__device__ __forceinline__ const double *cr_row(const DevLines &L, int c)
{
    return L.lev ? L.lnd + (int64_t)c * L.lnd_stride : nullptr;
}

// a[i0 + t], i0 the same for the whole wave: a scalar base and a 32-bit offset.
template <typename T>
__device__ __forceinline__ T line_at(const T *a, int64_t i0, uint32_t t)
{
    return *(const T *)((const char *)(a + i0) + t * (uint32_t)sizeof(T));
}

// The line list's pointers and a cell's constants, read again (scalar loads) for
// every round of setups: held across the kernel they do not fit in the scalar
// registers beside the masks, and come back from spills by one vector
// instruction per register (stagnation line 343 -> 330 ms, one served request
// 2.25 -> 2.12 ms; the double-precision kernel 89 -> 64 VGPRs).  DevLines is the
// first argument of the kernels that use lines_arg.
template <typename T>
__device__ __forceinline__ const T &reread(const T *p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    auto q = (const __attribute__((address_space(4))) T *)(((uint64_t)hi << 32) | lo);
    asm volatile("" : "+s"(q));
    return *(const T *)q;
}
__device__ __forceinline__ const DevLines &lines_arg()
{
    auto q = (const __attribute__((address_space(4))) DevLines *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(q));
    return *(const DevLines *)q;
}

__device__ __forceinline__ bool pair_setup(const DevLines &L, const DevGrid &g, const CellConst &k,
                                           const CellSpecies *csc, const double *lnd_c, int64_t i0, uint32_t t,
                                           PairF64 &p)
{
    const int s = line_at(L.species, i0, t);
    const CellSpecies q = csc[s];
    if (!(q.lnNQ > -INFINITY)) {
        p.klo = p.kclo = 1;
        p.khi = p.kchi = 0;
        p.se = p.sk = p.inv2g = p.r = 0.0;
        return false;
    }
    const double nu0 = line_at(L.nu0, i0, t);
    const double Eu_ev = line_at(L.Eu_ev, i0, t), Eu_rot = line_at(L.Eu_rot, i0, t);
    const double El_ev = line_at(L.El_ev, i0, t), El_rot = line_at(L.El_rot, i0, t);
    const double base = q.lnNQ + line_at(L.lngu, i0, t);
    // N_u = N g_u e^{-E_u}/Q, and N_l g_u/g_l = N_u e^{x} with x the line's
    // reduced energy, so N_l (g_u/g_l)(1 - e^{-x}) = N_u (e^{x} - 1)
    const double lnNu = base - k.beta_v * Eu_ev - k.beta_tr * Eu_rot;
    const double x = k.beta_v * (Eu_ev - El_ev) + k.beta_tr * (Eu_rot - El_rot);
    const int32_t lv = lnd_c ? line_at(L.lev, i0, t) : -1;
    double Nu, Nlx;
    if (lv < 0) {
        if (fabs(lnNu) < 700.0 && fabs(x) < 700.0) {
            const ExpParts e = exp_parts(lnNu);
            Nu = exp_of(e);
            Nlx = Nu * expm1_of(exp_parts(x));
        } else {
            // (the two-factor form only while N_u e^{x} stays representable)
            Nu = exp_any(lnNu);
            Nlx = (lnNu > -700.0 && x < 700.0) ? Nu * expm1_any(x) : exp_any(lnNu + x) * (-expm1_any(-x));
        }
    } else {
        // QSS-CR populations: both levels carry their departure from
        // Boltzmann, N_u = e^{lu}, N_l g_u/g_l = e^{ll}, and the absorption
        // takes N_l g_u/g_l - N_u (negative for an inverted pair)
        const double lu = lnNu + lnd_c[lv & 0xffff];
        const double ll = lnNu + x + lnd_c[lv >> 16];
        Nu = exp_any(lu);
        Nlx = (ll >= lu) ? (ll > -INFINITY ? exp_any(ll) * -expm1_any(lu - ll) : 0.0) : Nu * expm1_any(ll - lu);
    }
    const double Seta = line_at(L.seta0, i0, t) * Nu;
    const double Skap = line_at(L.skap0, i0, t) * Nlx;
    // widths (Sec. 2.2.1): Doppler, Lorentz, Voigt (Olivero fit)
    const double gG = q.dop * nu0;
    const double gL = line_at(L.gN, i0, t) + line_at(L.gS, i0, t) * k.gL + q.gW;
    const double gV = voigt_hwhm(gL, gG, rcp_f64(gL + gG));
    const double inv_gV = rcp_f64(gV);
    const double r = gL * inv_gV;
    const double norm = 0.5 * inv_gV * rcp_f64(1.065 + 0.447 * r + 0.058 * r * r);
    // window |nu_k - nu0| <= 100 gamma_V; rounding-exact operation order.  The
    // product by 1/h gives the same bound as the division unless it lies within
    // its own rounding (below 1e-6 on grids of up to 2^31 points) of an integer.
    const double W = __dmul_rn(100.0, gV);
    const double dlo = __dsub_rn(__dsub_rn(nu0, W), g.nu_min), dhi = __dsub_rn(__dadd_rn(nu0, W), g.nu_min);
    const double qlo = dlo * g.inv_h, qhi = dhi * g.inv_h;
    double lo = ceil(qlo), hi = floor(qhi);
    if (fabs(qlo - rint(qlo)) < 1e-5 || fabs(qhi - rint(qhi)) < 1e-5) {
        lo = ceil(__ddiv_rn(dlo, g.h));
        hi = floor(__ddiv_rn(dhi, g.h));
    }
    lo = fmax(lo, 0.0);
    hi = fmin(hi, (double)(g.n_points - 1));
    if (lo > hi) {
        p.klo = 1;
        p.khi = 0;
    } else {
        p.klo = (int32_t)lo;
        p.khi = (int32_t)hi;
    }
    {
        // core: a superset of the points within kCoreHalfWidth gamma_V (one point of
        // margin on each side covers the rounding of the product by 1/h)
        const double Wc = kCoreHalfWidth * gV;
        double clo = fmax(ceil((nu0 - Wc - g.nu_min) * g.inv_h) - 1.0, lo);
        double chi = fmin(floor((nu0 + Wc - g.nu_min) * g.inv_h) + 1.0, hi);
        if (clo > chi) {
            p.kclo = 1;
            p.kchi = 0;
        } else {
            p.kclo = (int32_t)clo;
            p.kchi = (int32_t)chi;
        }
    }
    p.se = Seta * norm;
    p.sk = Skap * norm;
    p.inv2g = 0.5 * inv_gV;
    p.r = r;
    return p.klo <= p.khi;
}

// ---------------------------------------------------------------------------
// atomic continuum (Sec. 2.2.1 bound-free and free-free)
// ---------------------------------------------------------------------------

constexpr double kElectronMass = 9.1093837015e-28;   // g

// Per cell: prefix sums over the sorted thresholds of the bound-free
// absorption and emission weights (times nu_thr^3), the two free-free
// coefficients, and ln upper bounds of eta_c and kappa_c over [nu_lo, nu_hi]
// for the power-of-two scale.
__global__ void cont_cells_kernel(const ContThr *thr, int32_t n_thr, const ContRec *rec,
                                  int32_t n_rec, DevCells cells, const CellSpecies *cs, DevCR cr,
                                  uint64_t species_mask, double nu_lo, double nu_hi, double *cum,
                                  double *ff, double *lnb)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cells.n_cells) return;
    const int ns = cells.n_species;
    const double T = cells.T_v[c], ne = cells.n_e[c];
    // Saha-Boltzmann volume (h^2 / (2 pi m_e k T))^{3/2}
    const double V = pow(kPlanck * kPlanck / (2.0 * kPi * kElectronMass * kBoltz * T), 1.5);
    double *cA = cum + (int64_t)c * 2 * (n_thr + 1), *cB = cA + (n_thr + 1);
    double a = 0.0, b = 0.0, ka = 0.0, eb = 0.0;
    cA[0] = cB[0] = 0.0;
    const double twohc2 = 1e-7 * 2.0 * kPlanck * kLight * kLight;
    for (int j = 0; j < n_thr; ++j) {
        const ContThr t = thr[j];
        const ContRec r = rec[t.rec];
        if (!species_on(species_mask, r.species)) {   // a species outside the mask radiates nothing
            cA[j + 1] = a;
            cB[j + 1] = b;
            continue;
        }
        const double Np = cells.N[(int64_t)c * ns + r.ion];
        const int slot = cr.n > 0 ? cr.slot[r.species] : -1;
        // absorption from the level: its QSS-CR population, else Boltzmann
        const double aj = slot >= 0 ? cr.pop[((int64_t)c * cr.n + slot) * cr.LS + t.lev] * t.s3
                                    : exp(cs[(int64_t)c * ns + r.species].lnNQ) * t.g * exp(-kC2 * t.E / T) * t.s3;
        const double bj = Np * ne * V * t.g / (2.0 * r.Q_ion) * t.s3;   // without e^{c2 nu_j / T}
        a += aj;
        b += bj * exp(kC2 * t.nu / T);
        cA[j + 1] = a;
        cB[j + 1] = b;
        // bounds: at nu >= max(nu_j, nu_lo), aj / nu^3 <= aj / max(nu_j, nu_lo)^3 and
        // B(nu) bj e^{c2 nu_j/T} / nu^3 <= 2hc^2 bj / (1 - e^{-c2 max(nu_j, nu_lo)/T})
        const double nm = fmax(t.nu, nu_lo);
        ka += aj / (nm * nm * nm);
        eb += twohc2 * bj / -expm1(-kC2 * nm / T);
    }
    double f0 = 0.0, f1 = 0.0;
    for (int q = 0; q < n_rec; ++q) {
        const ContRec r = rec[q];
        if (!species_on(species_mask, r.species)) continue;
        const double w = cells.N[(int64_t)c * ns + r.ion] * ne * 1e-40 * r.z4inv;
        f0 += w * (r.peach[0] + r.peach[1] * exp(-r.peach[2] * T));
        f1 += w * (r.peach[3] + r.peach[4] * exp(-r.peach[5] * T) + r.peach[6] * exp(-r.peach[7] * T));
    }
    ff[2 * c + 0] = f0;
    ff[2 * c + 1] = f1;
    // free-free falls with nu on the grid; its emission carries the Planck
    // factor, whose maximum over [nu_lo, nu_hi] is at nu_p = 2.8214 T / c2 or
    // the nearer end
    const double inv3 = 1.0 / (nu_lo * nu_lo * nu_lo);
    const double kff = (fabs(f0) * kNuH / nu_lo + fabs(f1)) * kNuH * kNuH * kNuH * inv3;
    const double nu_p = fmin(fmax(2.8214393721220787 * T / kC2, nu_lo), nu_hi);
    const double km = ka + kff, em = eb + planck_f64(nu_p, T) * kff;
    lnb[2 * c + 0] = em > 0.0 ? log(em) : -INFINITY;
    lnb[2 * c + 1] = km > 0.0 ? log(km) : -INFINITY;
}

// Continuum eta and kappa of cell c at nu (double precision).
__device__ __forceinline__ void continuum_point(const DevCont &ct, int c, double nu, double &eta,
                                                double &kap)
{
    int lo = 0, hi = ct.n_thr;   // m = number of thresholds <= nu
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ct.thr[mid].nu <= nu) lo = mid + 1; else hi = mid;
    }
    const double *cA = ct.cum + (int64_t)c * 2 * (ct.n_thr + 1);
    const double inv3 = 1.0 / (nu * nu * nu);
    const double kff = (ct.ff[2 * c] * (kNuH / nu) + ct.ff[2 * c + 1]) * (kNuH * kNuH * kNuH) * inv3;
    kap = cA[lo] * inv3 + kff;
    eta = planck_f64(nu, ct.T_v[c]) * (cA[ct.n_thr + 1 + lo] * inv3 + kff);
}

// ---------------------------------------------------------------------------
// candidate line ranges per (cell, tile)
// ---------------------------------------------------------------------------

__device__ __forceinline__ int64_t lower_bound_dev(const double *a, int64_t n, double v)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t m = lo + ((hi - lo) >> 1);
        if (a[m] < v) lo = m + 1; else hi = m;
    }
    return lo;
}

__global__ void ranges_kernel(DevLines L, DevGrid g, const CellConst *cc, int32_t n_cells,
                              int32_t k_first, int32_t n_band, int32_t tile_points,
                              int32_t n_tiles, int2 *ranges)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n_cells * n_tiles) return;
    const int c = (int)(t / n_tiles), tile = (int)(t % n_tiles);
    const CellConst k = cc[c];
    const int32_t ka = k_first + tile * tile_points;
    const int32_t kb = ka + min(k_first + n_band - ka, tile_points) - 1;
    const double nu_a = g.nu_min + (double)ka * g.h - g.h;
    const double nu_b = g.nu_min + (double)kb * g.h + g.h;
    double lo = (nu_a - k.cand_G) / (1.0 + k.cand_A);
    double hi = (nu_b + k.cand_G) / (1.0 - k.cand_A);
    // Within those the window is at most the Voigt width of the largest Lorentz
    // width and the Doppler width at the last of their centres (the fit grows
    // with both), up to 18 % less than the sum of the two.
    if (hi > 0.0) {
        const double W = voigt_hwhm(k.cand_G, k.cand_A * hi, 1.0 / (k.cand_G + k.cand_A * hi));
        lo = fmax(lo, nu_a - W);
        hi = fmin(hi, nu_b + W);
    }
    int2 r;
    r.x = (int)lower_bound_dev(L.nu0, L.n, lo);
    r.y = (int)lower_bound_dev(L.nu0, L.n, hi);
    ranges[t] = r;
}

// ---------------------------------------------------------------------------
// per-cell power-of-two scale for the single-precision form
// ---------------------------------------------------------------------------

// Per-cell scale from the level-energy bins: the cell's waves take the
// largest upper bound of ln(eta peak) and ln(|kappa peak|) over the bins.
// Peak of line i: strength * norm with norm = 1/(2 gV (1.065 + ...)) and
// gV >= 0.9 gG (the Voigt width is at least the Doppler one; 0.9 leaves room
// for the fit), gG = dop_s nu0; |kappa| <= skap0 max(N_u, N_l g_u/g_l).  The
// bound exceeds the true peak by a modest factor (bin width, Lorentz part of
// the width), which the power-of-two scale absorbs.
// kWaves waves per cell: four while the cells alone leave the chip idle, else one.
// The species' part of the bound is taken once per cell (LDS, up to
// kScaleSpecies species), so a bin costs two multiply-adds and two maxima; bound
// by the bins' loads.  32,768 cells of the 1M-line list 1.71 -> 1.04 ms, 190 cells
// 240 -> 63 us.
constexpr int kScaleSpecies = 64;
template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) void scale_bound_kernel(DevBins B, const CellConst *cc,
                                                                  const CellSpecies *cs, const double *cont_lnb,
                                                                  int32_t n_cells, int32_t n_species, int32_t *escale)
{
    __shared__ double v0[kScaleSpecies];
    __shared__ double part[kWaves][2];
    const int c = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const CellConst k = cc[c];
    const double ln_norm = -log(2.0 * 1.065 * 0.9);
    auto species_part = [&](int s) {
        const CellSpecies q = cs[(int64_t)c * n_species + s];
        return q.lnNQ > -INFINITY ? q.lnNQ + ln_norm - log(q.dop) : -INFINITY;
    };
    if ((int)threadIdx.x < min(n_species, kScaleSpecies)) v0[threadIdx.x] = species_part(threadIdx.x);
    __syncthreads();
    double ve = -INFINITY, vk = -INFINITY;
    const double *lnd_c = B.lev_off ? B.lnd + (int64_t)c * B.lnd_stride : nullptr;
    // a spectral window: line centres that can reach it (as ranges_kernel)
    double ca = -INFINITY, cb = INFINITY;
    if (B.nu_lo) {
        ca = (B.win_a - k.cand_G) / (1.0 + k.cand_A);
        cb = (B.win_b + k.cand_G) / (1.0 - k.cand_A);
    }
    for (int b = threadIdx.x; b < B.n; b += 64 * kWaves) {
        if (B.nu_lo && (B.nu_hi[b] < ca || B.nu_lo[b] > cb)) continue;
        const int s = B.species[b];
        const double v1 = s < kScaleSpecies ? v0[s] : species_part(s);
        if (!(v1 > -INFINITY)) continue;
        double v = v1 - k.beta_v * B.Ev[b] - k.beta_tr * B.Er[b];
        if (lnd_c) {
            // QSS-CR: the largest departure from Boltzmann among the bin's levels
            double d = -INFINITY;
            for (int32_t j = B.lev_off[b]; j < B.lev_off[b + 1]; ++j) {
                const int32_t o = B.lev[j];
                d = fmax(d, o < 0 ? 0.0 : lnd_c[o]);
            }
            v += d;
        }
        ve = fmax(ve, B.a_eta[b] + v);
        vk = fmax(vk, B.a_kap[b] + v);
    }
    for (int o = 32; o > 0; o >>= 1) {
        ve = fmax(ve, __shfl_xor(ve, o));
        vk = fmax(vk, __shfl_xor(vk, o));
    }
    if constexpr (kWaves > 1) {
        if (lane == 0) {
            part[threadIdx.x >> 6][0] = ve;
            part[threadIdx.x >> 6][1] = vk;
        }
        __syncthreads();
        for (int w = 0; w < kWaves; ++w) {
            ve = fmax(ve, part[w][0]);
            vk = fmax(vk, part[w][1]);
        }
    }
    if (cont_lnb) {   // the atomic continuum's own bound
        ve = fmax(ve, cont_lnb[2 * c + 0]);
        vk = fmax(vk, cont_lnb[2 * c + 1]);
    }
    if (threadIdx.x == 0) {
        // peak < 2^e; stay unscaled while e is within 2^+-60
        const double v2[2] = {ve, vk};
        for (int j = 0; j < 2; ++j) {
            int e = 0;
            if (v2[j] > -INFINITY) {
                const double t = ceil(v2[j] * kLog2e) + 1.0;
                e = (int)fmax(-2000.0, fmin(2000.0, t));
                if (e >= -60 && e <= 60) e = 0;
            }
            escale[2 * c + j] = e;
        }
    }
}

// ---------------------------------------------------------------------------
// a3: line-to-grid accumulation
// ---------------------------------------------------------------------------

// Single-precision line record staged in LDS.  Grid indices inside the
// kernel are relative to the tile start, so every float index is a small
// exact integer whatever the grid size.
struct __align__(16) RecPos {
    float k0f, hg, fg, qw;          // centre index (tile-relative), h/gV, frac0/gV, 0.016 r (1-r) / s
};
struct __align__(16) RecAmp {
    float se, sk, qg;               // strengths times s and the cell's scale; (1-r) / s
    uint32_t edges;                 // window, tile-relative, clamped to the tile: klo | (khi + 1) << 16 (edge masks)
};
// Double-precision line record: x = |(k - k0) h2 - f2| with h2 = h/(2 gamma_V),
// f2 = frac0/(2 gamma_V) and the tile-relative index k.
struct __align__(16) RecPos64 {
    double k0, h2, f2, r;   // centre index (tile-relative), h2, f2, gamma_L / gamma_V
};
struct __align__(16) RecAmp64 {
    double w, se, sk;       // 0.016 r (1-r), strengths
    uint32_t edges, pad;    // window, tile-relative, clamped to the tile: klo | (khi + 1) << 16
};

// The Whiting profile is evaluated in y = (nu_k - nu0) / gamma_V = +-2x, so that
// 1 + 4x^2 = 1 + y^2 is one FMA and x^2.25 = 2^-2.25 |y|^2.25.
constexpr double kTwoM225 = 0.21022410381342863;   // 2^-2.25

__device__ const NodeBasis<kNodes> kBasis(kNodePos);
__device__ const NodeBasis<kNodes64> kBasis64(kNodePos64);

// Constants of the single-precision profile.  The kernels set them once,
// outside their loops, and an empty asm keeps them in scalar registers: VOP3
// instructions take no literal on this chip, so a constant rebuilt inside
// the loop costs a vector move per use.
struct ShapeConsts {
    float c225;   // 2.25 (the exponent of |y|)
    float cw;     // 0.1 * 2^-2.25 (0.1 x^2.25 from |y|^2.25)
    float cg;     // -2.772/4 log2(e) (the Gaussian exponent from 1 + y^2)
    float ce;     // -0.4 * 2^-2.25 log2(e) (the other exponent)
};

__device__ __forceinline__ ShapeConsts shape_consts()
{
    ShapeConsts K{2.25f, (float)(0.1 * kTwoM225), (float)(-2.772 / 4.0 * kLog2e),
                  (float)(-0.4 * kTwoM225 * kLog2e)};
    asm volatile("" : "+s"(K.c225), "+s"(K.cw), "+s"(K.cg), "+s"(K.ce));
    return K;
}

// The profile divided by s = r = gL/gV (the staged strengths carry the
// factor s back): rational part [1/(1+4x^2) - 0.016 (1-r)/(1+0.1 x^2.25)]
// over one reciprocal, whose numerator (1+0.1 x^2.25) - 0.016 (1-r)(1+4x^2)
// is one FMA; also returns 1 + y^2 and |y|^2.25 for the exponential part.
// A line with r below kRScaleMin is staged with s = kRScaleMin instead, which
// adds a Lorentzian of at most kRScaleMin of the line's own peak.  (Two
// reciprocals save instructions but measured 4 % slower: the transcendental
// pipe, not the instruction count, then sets the pace.)
__device__ __forceinline__ float shape_rational_f32(float kf, const RecPos &q, const ShapeConsts &K, float &d1,
                                                    float &p)
{
    const float y = fmaf(kf - q.k0f, q.hg, -q.fg);
    d1 = fmaf(y, y, 1.0f);
    p = __builtin_amdgcn_exp2f(K.c225 * __builtin_amdgcn_logf(fabsf(y)));
    const float d2 = fmaf(p, K.cw, 1.0f);
    const float num = fmaf(-q.qw, d1, d2);
    return num * __builtin_amdgcn_rcpf(d1 * d2);
}

// Smallest normalisation s of the staged profile (2^-40).
constexpr double kRScaleMin = 9.094947017729282e-13;

// Exponential part [(1-r) e^{-2.772 x^2} + 0.016 r(1-r) e^{-0.4 x^2.25}] / s
// added to P, with x^2 = (d1 - 1)/4 folded into the exponent's FMA; wexp_f32
// adds the second term alone.
__device__ __forceinline__ float wexp_f32(float qw, const ShapeConsts &K, float p, float P)
{
    return fmaf(qw, __builtin_amdgcn_exp2f(p * K.ce), P);
}
__device__ __forceinline__ float shape_exp_f32(float qw, float qg, const ShapeConsts &K, float d1, float p, float P)
{
    const float gs = __builtin_amdgcn_exp2f(fmaf(d1, K.cg, -K.cg));
    return fmaf(qg, gs, wexp_f32(qw, K, p, P));
}

// Block -> (tile, cell) order of the accumulation grid: groups of 8 tiles x
// all cells; within a group XCD x (workgroups go round-robin over the 8 XCDs,
// each with its own L2) takes tile 8g + x for every cell, so the cells of one
// tile share their candidate lines in one L2 while tiles stay interleaved
// across XCDs.  (Measured against tile-fastest order: 3 % faster; against a
// contiguous range of tiles per XCD: 37 % faster, the per-XCD work being
// uneven because line density varies along nu.)
__device__ __forceinline__ void block_tile_cell(uint32_t b, int32_t n_cells, int32_t n_tiles, int &tile,
                                                int &cell)
{
    const uint32_t gsz = (uint32_t)kXCDs * (uint32_t)n_cells;
    const uint32_t g = b / gsz, r = b % gsz;
    const uint32_t full = (uint32_t)n_tiles / kXCDs;
    if (g < full) {
        tile = (int)(g * kXCDs + r % kXCDs);
        cell = (int)(r / kXCDs);
    } else {   // last partial group of tiles
        tile = (int)(g * kXCDs + r / (uint32_t)n_cells);
        cell = (int)(r % (uint32_t)n_cells);
    }
}

// Square root of x > 0 from the hardware reciprocal square root (about 5e-8
// relative) and one Newton step on y^2 = x.  Measured on the chip, the fourth
// root as two such steps stays within 4.2e-15 relative of x^(1/4) over
// [1e-20, 1e4], against 38 instructions for two correctly rounded roots.
__device__ __forceinline__ double sqrt_newton(double x)
{
    const double r = __builtin_amdgcn_rsq(x);
    const double y = x * r;
    return fma(fma(-y, y, x), 0.5 * r, y);
}

// Lines per block: partials of at most kBlock terms are added plainly in single
// precision, blocks are merged in double precision.  A block is one ballot
// mask: one bit per line.
constexpr int kBlock = 64;
using BlockMask = uint64_t;

#ifndef LRT_NODE_LINES
#define LRT_NODE_LINES 128
#endif
constexpr int kNodeLines = LRT_NODE_LINES;

// Shared memory of the single-precision accumulation: the staged lines of a
// round, and per wave the node sums of its intervals (its two 64-point ones,
// then one of each larger size, shared with the other waves under it).
constexpr int kSets = kPPL + kLevels - 1;
// Wave w of a group owns slices w and w + 4 of the tile, kSliceStep points apart:
// a round's lines lie close together in the sorted list, so their windows reach
// neighbouring slices, which then belong to different waves.  With two
// neighbouring slices per wave half of the waves waited at a round's end for
// the other half: stagnation line 392 -> 342 ms, 48 cells x 32,768 points 1.39 ->
// 1.15 ms, 24 cells x 20,001 points in double precision 1.80 -> 1.39 ms; windows
// of 300 points (gamma_V 1.5) 13.1 -> 11.7 ms per band of 65,536 points and 400
// cells.
constexpr int kSliceStep = 256;
constexpr uint32_t kOwnSlices = 0x11u;
struct AccumLds {
    RecPos pos[kStage];
    RecAmp amp[kStage];
    RecMode mode[kStage];
    uint32_t any[kStage / kBlock];   // per block of lines, of any line: its slices | its intervals << 8
    double node[kAccumThreads / 64][kSets][2][kNodes];
};

// x on the lanes of the slice at point s0 that are inside a line's window (edges,
// the same in every lane), zero on the others.  The lane mask is built in
// scalar registers, whose unit has room beside the vector unit that bounds the
// accumulation: two vector instructions instead of the seven of unpacking and
// comparing both bounds (stagnation line 403 -> 392 ms).
template <typename T>
__device__ __forceinline__ T in_window(T x, uint32_t edges, int32_t s0)
{
    const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)edges);
    const int32_t a = max((int32_t)(e & 0xffffu) - s0, 0), b = min((int32_t)(e >> 16) - s0, 64);
    const uint64_t m = (~uint64_t(0) << (a & 63)) & (~uint64_t(0) >> ((64 - b) & 63));
    return __builtin_amdgcn_inverse_ballot_w64(m) ? x : T(0);
}

// The terms of one staged line (bit t of the block masks) on this wave's
// slices, the first at point s0, added to the block partials.
template <typename Mask>
__device__ __forceinline__ void line_terms(const RecPos &qr, const RecAmp &ar, int t, int32_t s0, const float (&kf)[kPPL],
                                           const ShapeConsts &K, const Mask (&m_in)[kPPL],
                                           const Mask (&m_core)[kPPL], const Mask (&m_edge)[kPPL],
                                           float (&ae)[kPPL], float (&ak)[kPPL])
{
    const RecPos q = qr;
    const RecAmp a = ar;
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        if (!((m_in[j] >> t) & 1u)) continue;      // slice outside the window, or at nodes
        float d1, pw;
        float P = shape_rational_f32(kf[j], q, K, d1, pw);
        // Within kCoreHalfWidth gamma_V of the centre the exponentials
        // contribute; beyond it they are below 2^-30 of the term.  Both
        // conditions are wave-uniform; the empty asm keeps them real
        // scalar branches instead of computing both sides and selecting.
        if ((m_core[j] >> t) & 1u) {
            asm volatile("");
            P = shape_exp_f32(q.qw, a.qg, K, d1, pw, P);
        }
        // slice crossing a window edge: mask the lanes outside
        if ((m_edge[j] >> t) & 1u) {
            asm volatile("");
            P = in_window(P, a.edges, s0 + kSliceStep * j);
        }
        ae[j] = fmaf(P, a.se, ae[j]);
        ak[j] = fmaf(P, a.sk, ak[j]);
    }
}

// The terms of a block's lines (mask m, those with the exponential mw) at the
// nodes of one interval, added to the lane's sums.  The wave takes four lines
// at a time, sixteen lanes to a line, each lane at its node x (tile-relative):
// the records of four consecutive lines are read from one base address, and a
// lane whose line has no bit adds zero.  (The lines an interval takes lie in
// two runs of the sorted list, so few of the four are idle.)
__device__ __forceinline__ void node_terms(const RecPos *pos, const RecAmp *amp, BlockMask m, BlockMask mw, float x,
                                           uint32_t grp, const ShapeConsts &K, float &ae, float &ak)
{
    uint32_t off = grp * 16u;
    const uint64_t mine = m >> grp;
    // 32 lines at a time: constant bit positions in 32-bit halves
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t mh = (uint32_t)(m >> (32 * h)), wh = (uint32_t)(mw >> (32 * h));
        if (mh == 0) continue;
        const uint32_t mi = (uint32_t)(mine >> (32 * h));
        asm volatile("" : "+v"(off));
        const char *pb = (const char *)pos + off, *ab = (const char *)amp + off;
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            if (((mh >> (4 * g)) & 15u) == 0) continue;
            const RecPos q = *(const RecPos *)(pb + (32 * h + 4 * g) * 16);
            const float2 a = *(const float2 *)(ab + (32 * h + 4 * g) * 16);
            float d1, p;
            float P = shape_rational_f32(x, q, K, d1, p);
            if ((wh >> (4 * g)) & 15u) {
                asm volatile("");
                P = wexp_f32(q.qw, K, p, P);
            }
            // all bits of P, or none
            const int32_t keep = (int32_t)(mi << (31 - 4 * g)) >> 31;
            P = __int_as_float(__float_as_int(P) & keep);
            ae = fmaf(P, a.x, ae);
            ak = fmaf(P, a.y, ak);
        }
    }
}

// The bits of any lane.
__device__ __forceinline__ uint32_t wave_or(uint32_t v)
{
    v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr 1, 2, 4, 8
    v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);   // row_bcast 15, 31
    v |= __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);
    return (uint32_t)__builtin_amdgcn_readlane(v, 63);
}

// Adds a round's sums of the four lane groups to an interval's node sums
// (acc[0]: eta, acc[1]: kappa), in a fixed order: the halves of the wave are
// added pairwise (its lower half then holds eta, its upper half kappa), then
// the two groups of each half.
__device__ __forceinline__ void node_flush(float pe, float pk, int lane, double (*acc)[kNodes])
{
    const uint64_t a = __double_as_longlong((double)pe), b = __double_as_longlong((double)pk);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    const double t = __longlong_as_double(((uint64_t)hi[0] << 32) | lo[0]) +
                     __longlong_as_double(((uint64_t)hi[1] << 32) | lo[1]);
    const uint64_t c = __double_as_longlong(t);
    const auto l2 = __builtin_amdgcn_permlane16_swap((uint32_t)c, (uint32_t)c, false, false);
    const auto h2 = __builtin_amdgcn_permlane16_swap((uint32_t)(c >> 32), (uint32_t)(c >> 32), false, false);
    const double v = __longlong_as_double(((uint64_t)h2[0] << 32) | l2[0]) +
                     __longlong_as_double(((uint64_t)h2[1] << 32) | l2[1]);
    if ((lane & 16) == 0) acc[lane >> 5][lane & 15] += v;
}

// The node sums of a tile's intervals brought down to its 64-point intervals:
// the waves' parts of each interval, then level by level from the whole tile,
// each interval's polynomial taken at the nodes of its halves.  An interval's
// sums end up with the first wave that shares it, a slice's with its wave.  Called by the whole workgroup, after
// a barrier, tid the thread of its group; ends with a barrier.
template <int N, int kThreads>
__device__ __forceinline__ void nodes_down(double (&sums)[kThreads / 64][kSets][2][N], const NodeBasis<N> &basis,
                                           int tid)
{
#pragma unroll
    for (int l = kLevels - 1; l >= 0; --l) {
        // thread -> (interval, quantity, node)
        const int node = tid % N, qy = tid / N % 2;
        for (int it = tid / (2 * N); it < (kSlices >> l); it += kThreads / (2 * N)) {
            const int w0 = l > 0 ? it << (l - 1) : it % (kThreads / 64);
            const int set = l > 0 ? kPPL - 1 + l : it / (kThreads / 64);
            double v = sums[w0][set][qy][node];
            for (int w = 1; w < (1 << l) / 2; ++w) v += sums[w0 + w][set][qy][node];
            if (l < kLevels - 1) {
                const double *up = sums[(it >> 1) << l][kPPL + l][qy];
#pragma unroll 8
                for (int q = 0; q < N; ++q) {
                    const double c = (it & 1) ? basis.half[N - 1 - q][N - 1 - node] : basis.half[q][node];
                    v = fma(c, up[q], v);
                }
            }
            sums[w0][set][qy][node] = v;
        }
        __syncthreads();
    }
}

// Adds the sums of a workgroup's other groups (accum_groups) to those of
// group 0, in their order.  buf: per group 2 kPPL kThreads doubles of LDS that no
// thread needs any more.  Called by the whole workgroup.
template <int kGroups, int kThreads, typename F>
__device__ __forceinline__ void add_groups(F buf, int group, int tid, double (&se)[kPPL], double (&sk)[kPPL])
{
    if constexpr (kGroups > 1) {
        if (group > 0) {
            double *b = buf(group);
#pragma unroll
            for (int j = 0; j < kPPL; ++j) {
                b[2 * j * kThreads + tid] = se[j];
                b[(2 * j + 1) * kThreads + tid] = sk[j];
            }
        }
        __syncthreads();
        if (group == 0) {
#pragma unroll
            for (int o = 1; o < kGroups; ++o) {
                const double *b = buf(o);
#pragma unroll
                for (int j = 0; j < kPPL; ++j) {
                    se[j] += b[2 * j * kThreads + tid];
                    sk[j] += b[(2 * j + 1) * kThreads + tid];
                }
            }
        }
    }
}

// eta and kappa of one cell on one tile (kTilePoints points starting at the
// global index kt) in single precision: every round stages kStage candidate
// lines (one FP64 setup per thread) into LDS, then each wave evaluates the
// staged lines on its kPPL slices of 64 points, point by point or at the nodes
// of the intervals it owns: the 64-point intervals of its slices, one 128-point
// interval, and of each larger one every 2^n-th block of lines, shared with
// other waves.  Lanes hold the sums in double
// precision; the function returns eta[j], kappa[j] of point kt + kw + kSliceStep j +
// lane (scaled by 2^-ese, 2^-esk).  Must be called by the whole workgroup: kGroups
// groups of kAccumThreads threads, of which each takes every kGroups-th round
// with its own shared memory (sg[group]), tid the thread of the group; group 0
// returns the results.
template <int kGroups>
__device__ __forceinline__ void accum_cell_tile_f32(AccumLds *sg, int group, int tid, const DevGrid &g,
                                                    const CellConst &kc, const CellSpecies *csc,
                                                    const double *lnd_c, int ese, int esk, int2 rg, int32_t kt,
                                                    int32_t kw, int lane, float (&eta)[kPPL],
                                                    float (&kap)[kPPL])
{
    AccumLds &sm = sg[group];
    constexpr int kWaves = kAccumThreads / 64, kBlocks = kStage / kBlock;
    static_assert(kTilePoints == 1 << kTileBits && kPPL == 2 && kSliceStep == 64 * kWaves && kWaves * kPPL == kSlices && kBlocks == 4,
                  "a wave owns two slices and one 128-point interval");
    const uint32_t wave = (uint32_t)(kw / 64);
    const ShapeConsts K = shape_consts();
    float kf[kPPL];
    float ae[kPPL], ak[kPPL];
    double se[kPPL], sk[kPPL];
    // A tile with few lines is summed point by point: below kNodeLines candidate
    // lines the interpolation at the end costs more than the nodes save (131
    // cells, 6,000 lines on 100,003 points, 30 to 60 lines a tile: 776 us per
    // solve with a bound of 64, 727 with 128, the same up to 512).
    const bool at_nodes = rg.y - rg.x >= kNodeLines;
    double (*acc)[2][kNodes] = sm.node[wave];
    float x64 = 0.0f;
    if (at_nodes) {
        for (int j = lane; j < kSets * 2 * kNodes; j += 64) (&acc[0][0][0])[j] = 0.0;
#pragma unroll
        for (int i = 0; i < kNodes; ++i)
            if ((lane & 15) == i) x64 = (float)kNodePos[i];
    }
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        kf[j] = (float)(kw + kSliceStep * j + lane);
        asm volatile("" : "+v"(kf[j]));   // keep the float index in a register
        se[j] = sk[j] = 0.0;
        ae[j] = ak[j] = 0.0f;
    }
    uint32_t used = 0u;   // intervals that have taken a line's nodes
    for (int b0 = rg.x; b0 < rg.y; b0 += kGroups * kStage) {
        const int base = b0 + group * kStage;
        // stage: one (cell, line) setup per thread, in double precision
        RecPos rp;
        RecAmp ra;
        RecMode rm;
        rp.k0f = rp.hg = rp.fg = rp.qw = ra.se = ra.sk = ra.qg = 0.0f;
        ra.edges = rm.pt = rm.node = 0u;
        const int n = rg.y - base;   // lines left
        // (opaque, so that no per-lane line pointers are kept across the rounds)
        uint32_t t = (uint32_t)tid;
        asm volatile("" : "+v"(t));
        if ((int)t < n) {
            PairF64 p;
            const DevLines &L = lines_arg();
            const CellConst &k = reread(&kc);
            if (pair_setup(L, g, k, csc, lnd_c, base, t, p)) {
                const int32_t lo = p.klo - kt, hi = p.khi - kt;
                const double frac0 = line_at(L.frac0, base, t);
                const int32_t k0 = line_at(L.k0, base, t) - kt;
                rp.k0f = (float)k0;
                rp.hg = (float)(2.0 * g.h * p.inv2g);
                rp.fg = (float)(2.0 * frac0 * p.inv2g);
                // profile divided by s = r, strengths times s
                const double sc = fmax(p.r, kRScaleMin), isc = rcp_f64(sc);
                rp.qw = (float)(0.016 * p.r * (1.0 - p.r) * isc);
                ra.qg = (float)((1.0 - p.r) * isc);
                ra.se = (float)ldexp(p.se * sc, -ese);
                ra.sk = (float)ldexp(p.sk * sc, -esk);
                ra.edges = (uint32_t)min(max(lo, 0), kTilePoints) | ((uint32_t)min(max(hi + 1, 0), kTilePoints) << 16);
                // gamma_V, the two reaches and the centre in grid steps, the reaches
                // rounded up and the centre down with a step of margin (k0 is
                // clamped on very long grids, so the centre includes frac0)
                const float gs = __builtin_amdgcn_rcpf(rp.hg);
                const float yG = __builtin_amdgcn_sqrtf(37.0f - __builtin_amdgcn_logf((float)sc));
                const float cf = floorf(fmaf(rp.fg, gs, rp.k0f));
                rm = line_modes<false>(lo, hi, (int32_t)fmaxf(-1e9f, fminf(cf, 1e9f)) - 1,
                                (int32_t)fminf(yG * gs, 1.1e9f) + 2,
                                (int32_t)fminf((float)kCoreHalfWidth * gs, 1.1e9f) + 2, at_nodes);
            }
        }
        sm.pos[tid] = rp;
        sm.amp[tid] = ra;
        sm.mode[tid] = rm;
        const uint32_t any = wave_or((rm.pt & 0xffu) | (rm.node << 16 >> 8));
        if (lane == 0) sm.any[wave] = any;
        __syncthreads();
        // Control of the lines on this wave, as bit masks over a block in
        // scalar registers: lane t reads the masks of the block's line t, one
        // ballot per (interval, flag).  The loops then visit only the blocks
        // with a line for this wave, and of those only such lines, in line order.
        uint32_t of[kBlocks];
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) of[b] = (uint32_t)uniform_i((int32_t)sm.any[b]);
        const uint32_t in_nodes = (of[0] | of[1] | of[2] | of[3]) >> 8;
        used |= in_nodes;
        auto blocks_of = [&](uint32_t bits) {
            uint32_t m = 0u;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) m |= (of[b] & bits) ? 1u << b : 0u;
            return m;
        };
#pragma unroll 1
        for (uint32_t todo4 = blocks_of(kOwnSlices << wave); todo4; todo4 &= todo4 - 1u) {
            const int l0 = __builtin_ctz(todo4) * kBlock;
            const uint32_t mi = sm.mode[l0 + lane].pt >> wave;
            const BlockMask todo = (BlockMask)__ballot((mi & kOwnSlices) != 0);
            BlockMask m_in[kPPL], m_edge[kPPL], m_core[kPPL];
#pragma unroll
            for (int j = 0; j < kPPL; ++j) {
                m_in[j] = (BlockMask)__ballot(mi & (1u << (kWaves * j)));
                m_edge[j] = (BlockMask)__ballot(mi & (1u << (8 + kWaves * j)));
                m_core[j] = (BlockMask)__ballot(mi & (1u << (16 + kWaves * j)));
            }
            // groups of 8 lines: within a group the LDS offsets are constants
            // from one base address held in a vector register, and the block
            // masks, shifted once per group, are tested at constant bits; a
            // group that no line of it reaches is skipped whole
            for (int g8 = 0; g8 < kBlock; g8 += 8) {
                const uint32_t gt = (uint32_t)(todo >> g8) & 0xffu;
                if (gt == 0) continue;
                uint32_t gi[kPPL], gc[kPPL], ge[kPPL];
#pragma unroll
                for (int j = 0; j < kPPL; ++j) {
                    gi[j] = (uint32_t)(m_in[j] >> g8);
                    gc[j] = (uint32_t)(m_core[j] >> g8);
                    ge[j] = (uint32_t)(m_edge[j] >> g8);
                }
                // one LDS base per group (a byte offset in a vector register),
                // not one per line
                uint32_t off = (uint32_t)((l0 + g8) * 16);
                asm volatile("" : "+v"(off));
                const RecPos *rp8 = (const RecPos *)((const char *)sm.pos + off);
                const RecAmp *ra8 = (const RecAmp *)((const char *)sm.amp + off);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if ((gt >> u) & 1u) line_terms(rp8[u], ra8[u], u, kw, kf, K, gi, gc, ge, ae, ak);
            }
#pragma unroll
            for (int j = 0; j < kPPL; ++j) {
                se[j] += (double)ae[j];
                sk[j] += (double)ak[j];
                ae[j] = ak[j] = 0.0f;
            }
        }
        // Nodes, one interval after the other over the whole round (at most 64
        // terms per lane, added plainly): the two 64-point intervals, then of
        // level l interval wave >> (l-1), whose blocks of lines the 2^(l-1)
        // waves wave>>(l-1) << (l-1) on share.
#pragma unroll 1
        for (int j = 0; j < (in_nodes ? kSets : 0); ++j) {
            const int l = max(0, j - (kPPL - 1));
            const uint32_t it = l > 0 ? wave >> (l - 1) : (uint32_t)(wave + kWaves * j);
            const uint32_t bit = 1u << (node_bit0(l) + it), wbit = 1u << (16 + l);
            uint32_t todo4 = blocks_of(bit << 8);
            // the blocks b with b = wave (mod 2^(l-1))
            if (l == 2) todo4 &= (wave & 1u) ? 0xau : 0x5u;
            if (l == 3) todo4 &= 1u << wave;
            if (todo4 == 0) continue;
            const float w = (float)(64 << l);
            const float x = fmaf(x64, (float)(1 << l), (float)it * w + (0.5f * w - 0.5f));
            float pe = 0.0f, pk = 0.0f;
#pragma unroll 1
            for (; todo4; todo4 &= todo4 - 1u) {
                const int l0 = __builtin_ctz(todo4) * kBlock;
                const uint32_t nb = sm.mode[l0 + lane].node;
                const BlockMask m = (BlockMask)__ballot((nb & bit) != 0);
                const BlockMask mw = m & (BlockMask)__ballot((nb & wbit) != 0);
                node_terms(sm.pos + l0, sm.amp + l0, m, mw, x, (uint32_t)lane >> 4, K, pe, pk);
            }
            node_flush(pe, pk, lane, acc[j]);
        }
        __syncthreads();
    }
    // node sums to the points, where there are any: with windows of 40 to 90 points
    // no line takes nodes (32,768 cells x 65,536 points 163 -> 144 ms).  All waves
    // have seen the same masks; several groups have seen different ones.
    if (at_nodes && (kGroups > 1 || used)) {
        nodes_down<kNodes, kAccumThreads>(sm.node, kBasis, tid);
#pragma unroll 8
        for (int q = 0; q < kNodes; ++q) {
            const double c = kBasis.pt[q][lane];
#pragma unroll
            for (int j = 0; j < kPPL; ++j) {
                se[j] = fma(c, acc[j][0][q], se[j]);
                sk[j] = fma(c, acc[j][1][q], sk[j]);
            }
        }
        __syncthreads();   // the next call clears the sums
    }
    add_groups<kGroups, kAccumThreads>([&](int o) { return (double *)&sg[o]; }, group, tid, se, sk);
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        eta[j] = (float)se[j];
        kap[j] = (float)sk[j];
    }
}

template <int kGroups>
__global__ __launch_bounds__(kAccumThreads *kGroups) __attribute__((amdgpu_waves_per_eu(LRT_ACCUM_WAVES)))
void accum_f32_kernel(
    DevLines L, DevGrid g, const CellConst *cc, const CellSpecies *cs, const int32_t *escale,
    const int2 *ranges, int32_t n_cells, int32_t n_species, int32_t k_first, int32_t n_band,
    int32_t n_tiles, uint32_t b0, DevCont ct, float *eta, float *kappa)
{
    static_assert(sizeof(AccumLds) >= 2 * kPPL * kAccumThreads * sizeof(double), "add_groups");
    __shared__ AccumLds sm[kGroups];
    int tile, c;
    block_tile_cell(b0 + blockIdx.x, n_cells, n_tiles, tile, c);
    // the wave index is uniform across the wave: keep it (and every bound
    // derived from it) in scalar registers so slice tests are scalar branches
    constexpr int kWaves = kAccumThreads / 64;
    const int lane = threadIdx.x & 63, wave_all = uniform_i(threadIdx.x >> 6);
    const int group = wave_all / kWaves, wave = wave_all % kWaves;
    const int tid = threadIdx.x & (kAccumThreads - 1);
    const int32_t kt = k_first + tile * kTilePoints;   // first (global) point of the tile
    const int32_t kw = wave * 64;               // first point of the wave, tile-relative
    const int32_t kend = k_first + n_band;             // exclusive, global
    float e[kPPL], kp[kPPL];
    accum_cell_tile_f32<kGroups>(sm, group, tid, g, cc[c], cs + (int64_t)c * n_species, cr_row(L, c),
                                 escale[2 * c + 0], escale[2 * c + 1], ranges[(int64_t)c * n_tiles + tile], kt,
                                 kw, lane, e, kp);
    if (group > 0) return;
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        const uint32_t kk = (uint32_t)kt + (uint32_t)(kw + kSliceStep * j + lane);   // (may pass 2^31)
        if (kk < (uint32_t)kend) {
            const int64_t o = (int64_t)c * n_band + (int32_t)(kk - (uint32_t)k_first);
            if (ct.n_thr >= 0) {
                // atomic continuum, added in double precision and rounded once
                double ce, ck;
                continuum_point(ct, c, g.nu_min + (double)kk * g.h, ce, ck);
                e[j] = (float)((double)e[j] + ldexp(ce, -escale[2 * c + 0]));
                kp[j] = (float)((double)kp[j] + ldexp(ck, -escale[2 * c + 1]));
            }
            eta[o] = e[j];
            kappa[o] = kp[j];
        }
    }
}

// Reach of e^{-0.4 x^2.25} in double precision, in units of gamma_V: at y = 2x =
// 16 it is 2^-59 of the rational part, for any r.  The Gaussian's reach is y_G
// (lrt_nodes.h).  A lane of a slice within a term's reach but beyond it adds what
// the term is there.
constexpr double kF64WexpReach = 16.0;

// Rational part r/(1+4x^2) - w/(1+0.1 x^2.25) over one quotient (the hardware
// reciprocal refined to the rounding of a division); also x^2 and x^2.25.
__device__ __forceinline__ double shape_rational_f64(double k, const RecPos64 &q, double w, double &u, double &p)
{
    const double x = fabs(fma(k - q.k0, q.h2, -q.f2));
    u = x * x;
    p = u * (x > 0.0 ? sqrt_newton(sqrt_newton(x)) : 0.0);
    const double d1 = fma(4.0, u, 1.0), d2 = fma(0.1, p, 1.0);
    const double num = fma(q.r, d2, -(w * d1)), den = d1 * d2;
    const double inv = rcp_f64(den), P = num * inv;
    return fma(fma(-den, P, num), inv, P);
}
// e^v of v <= 0 (zero from -745 on, however far)
__device__ __forceinline__ double exp_neg_f64(double v) { return exp_of(exp_parts(v)); }

// The terms of one staged line (bit t of the block masks) on this wave's
// slices of points kd[j], added to the sums.
template <typename Mask>
__device__ __forceinline__ void line_terms_f64(const RecPos64 &qr, const RecAmp64 &ar, int t, int32_t s0,
                                               const double (&kd)[kPPL],
                                               const Mask (&m_in)[kPPL], const Mask (&m_w)[kPPL],
                                               const Mask (&m_g)[kPPL], const Mask (&m_edge)[kPPL],
                                               double (&se)[kPPL], double (&sk)[kPPL])
{
    const RecPos64 q = qr;
    const RecAmp64 a = ar;
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        if (!((m_in[j] >> t) & 1u)) continue;
        double u, p;
        double P = shape_rational_f64(kd[j], q, a.w, u, p);
        // exponentials by slice (wave-uniform)
        if ((m_g[j] >> t) & 1u) {
            asm volatile("");
            P = fma(1.0 - q.r, exp_neg_f64(-2.772 * u), P);
        }
        if ((m_w[j] >> t) & 1u) {
            asm volatile("");
            P = fma(a.w, exp_neg_f64(-0.4 * p), P);
        }
        if ((m_edge[j] >> t) & 1u) {
            asm volatile("");
            P = in_window(P, a.edges, s0 + kSliceStep * j);
        }
        se[j] = fma(a.se, P, se[j]);
        sk[j] = fma(a.sk, P, sk[j]);
    }
}

// As node_terms, two lines at a time with 32 nodes each.
__device__ __forceinline__ void node_terms_f64(const RecPos64 *pos, const RecAmp64 *amp, BlockMask m, BlockMask mw,
                                               double x, uint32_t grp, double &ae, double &ak)
{
#pragma unroll 1
    for (int b = 0; b < 64; b += 16) {
        const uint32_t mh = (uint32_t)(m >> b) & 0xffffu, wh = (uint32_t)(mw >> b);
        if (mh == 0) continue;
        const uint32_t mi = mh >> grp;
        uint32_t off = (grp + (uint32_t)b) * 32u;
        asm volatile("" : "+v"(off));
        const char *pb = (const char *)pos + off, *ab = (const char *)amp + off;
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            if (((mh >> (2 * g)) & 3u) == 0) continue;
            const RecPos64 q = *(const RecPos64 *)(pb + 64 * g);
            const RecAmp64 a = *(const RecAmp64 *)(ab + 64 * g);
            double u, p;
            double P = shape_rational_f64(x, q, a.w, u, p);
            if ((wh >> (2 * g)) & 3u) {
                asm volatile("");
                P = fma(a.w, exp_neg_f64(-0.4 * p), P);
            }
            P = ((mi >> (2 * g)) & 1u) ? P : 0.0;
            ae = fma(P, a.se, ae);
            ak = fma(P, a.sk, ak);
        }
    }
}

// As node_flush: the halves of the wave added, eta to the lower half's nodes,
// kappa to the upper half's.
__device__ __forceinline__ void node_flush_f64(double pe, double pk, int lane, double (*acc)[kNodes64])
{
    const uint64_t a = __double_as_longlong(pe), b = __double_as_longlong(pk);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    acc[lane >> 5][lane & 31] += __longlong_as_double(((uint64_t)hi[0] << 32) | lo[0]) +
                                 __longlong_as_double(((uint64_t)hi[1] << 32) | lo[1]);
}

struct AccumLds64 {
    RecPos64 pos[kThreadsF64];
    RecAmp64 amp[kThreadsF64];
    RecMode mode[kThreadsF64];
    uint32_t any[kThreadsF64 / kBlock];
    double node[kThreadsF64 / 64][kSets][2][kNodes64];
};

// Candidate lines from which the double-precision tile uses nodes: 64, 128 and
// 256 measure the same within 1 % (1.82 ms, 1.39 since, on 24 cells x 20,001 points of a
// line-dense spectrum); below 128 no line setup fills two waves.
constexpr int32_t kNodeLines64 = 128;

// Double-precision accumulation: 512-point tiles, 4 waves, 2 points per lane,
// the wings at 32 nodes per interval.  Bound by the FP64 VALU.  32 nodes bring
// the interpolation to 1e-16 of a term; with every term at the points the same
// kernel takes 2.38 ms instead of 1.82 ms (24 cells x 20,001 points), with a
// library exponential, a division and two square roots per term besides 3.12 ms.
// Its LDS leaves room for 5 waves per SIMD.
template <int kGroups>
__global__ __launch_bounds__(kThreadsF64 *kGroups) __attribute__((amdgpu_waves_per_eu(kGroups > 2 ? 4 : 6)))
void accum_f64_kernel(
    DevLines L, DevGrid g, const CellConst *cc, const CellSpecies *cs, const int2 *ranges,
    int32_t n_cells, int32_t n_species, int32_t k_first, int32_t n_band, int32_t n_tiles,
    uint32_t b0, DevCont ct, double *eta, double *kappa)
{
    constexpr int kWaves = kThreadsF64 / 64, kBlocks = kThreadsF64 / kBlock;
    static_assert(kTileF64 == 1 << kTileBits && kSliceStep == 64 * kWaves && kWaves * kPPL == kSlices && kBlocks == 4,
                  "a wave owns two slices and one 128-point interval");
    static_assert(sizeof(AccumLds64) >= 2 * kPPL * kThreadsF64 * sizeof(double), "add_groups");
    __shared__ AccumLds64 sg[kGroups];
    int tile, c;
    block_tile_cell(b0 + blockIdx.x, n_cells, n_tiles, tile, c);
    const int lane = threadIdx.x & 63, wave_all = uniform_i(threadIdx.x >> 6);
    const int group = wave_all / kWaves, wave = wave_all % kWaves;
    const int tid = threadIdx.x & (kThreadsF64 - 1);
    AccumLds64 &sm = sg[group];
    const int32_t kt = k_first + tile * kTileF64;
    const int32_t kw = wave * 64;   // tile-relative
    const int32_t kend = k_first + n_band;
    const CellConst &kc = cc[c];
    const CellSpecies *csc = cs + (int64_t)c * n_species;
    const double *lnd_c = cr_row(L, c);
    const int2 rg = ranges[(int64_t)c * n_tiles + tile];
    const bool at_nodes = rg.y - rg.x >= kNodeLines64;

    double se[kPPL], sk[kPPL], kd[kPPL];
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        se[j] = sk[j] = 0.0;
        kd[j] = (double)(kw + kSliceStep * j + lane);
    }
    double (*acc)[2][kNodes64] = sm.node[wave];
    double x64 = 0.0;
    if (at_nodes) {
        for (int j = lane; j < kSets * 2 * kNodes64; j += 64) (&acc[0][0][0])[j] = 0.0;
#pragma unroll
        for (int i = 0; i < kNodes64; ++i)
            if ((lane & 31) == i) x64 = kNodePos64[i];
    }

    uint32_t used = 0u;
    for (int b0r = rg.x; b0r < rg.y; b0r += kGroups * kThreadsF64) {
        const int base = b0r + group * kThreadsF64;
        RecPos64 rp{0.0, 0.0, 0.0, 0.0};
        RecAmp64 ra{0.0, 0.0, 0.0, 0u, 0u};
        RecMode rm{0u, 0u};
        uint32_t t = (uint32_t)tid;
        asm volatile("" : "+v"(t));
        if ((int)t < rg.y - base) {
            PairF64 p;
            const DevLines &L = lines_arg();
            const CellConst &k = reread(&kc);
            if (pair_setup(L, g, k, csc, lnd_c, base, t, p)) {
                const int32_t lo = p.klo - kt, hi = p.khi - kt;
                rp.k0 = (double)(line_at(L.k0, base, t) - kt);
                const double frac0 = line_at(L.frac0, base, t);
                rp.h2 = g.h * p.inv2g;
                rp.f2 = frac0 * p.inv2g;
                rp.r = p.r;
                ra.w = 0.016 * p.r * (1.0 - p.r);
                ra.se = p.se;
                ra.sk = p.sk;
                ra.edges = (uint32_t)min(max(lo, 0), kTileF64) | ((uint32_t)min(max(hi + 1, 0), kTileF64) << 16);
                // the reaches and the centre in grid steps (as the single-precision form)
                const float gs = __builtin_amdgcn_rcpf((float)(2.0 * rp.h2));
                const float yG = gauss_reach_f64(p.r);
                const float cf = floorf((float)rp.k0 + (float)(frac0 * g.inv_h));
                rm = line_modes(lo, hi, (int32_t)fmaxf(-1e9f, fminf(cf, 1e9f)) - 1,
                                (int32_t)fminf(yG * gs, 1.1e9f) + 2,
                                (int32_t)fminf((float)kF64WexpReach * gs, 1.1e9f) + 2, at_nodes);
            }
        }
        sm.pos[tid] = rp;
        sm.amp[tid] = ra;
        sm.mode[tid] = rm;
        const uint32_t any = wave_or((rm.pt & 0xffu) | (rm.node << 16 >> 8));
        if (lane == 0) sm.any[wave] = any;
        __syncthreads();
        uint32_t of[kBlocks];
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) of[b] = (uint32_t)uniform_i((int32_t)sm.any[b]);
        const uint32_t in_nodes = (of[0] | of[1] | of[2] | of[3]) >> 8;
        used |= in_nodes;
        auto blocks_of = [&](uint32_t bits) {
            uint32_t m = 0u;
#pragma unroll
            for (int b = 0; b < kBlocks; ++b) m |= (of[b] & bits) ? 1u << b : 0u;
            return m;
        };
#pragma unroll 1
        for (uint32_t todo4 = blocks_of(kOwnSlices << wave); todo4; todo4 &= todo4 - 1u) {
            const int l0 = __builtin_ctz(todo4) * kBlock;
            const uint32_t mi = sm.mode[l0 + lane].pt >> wave;
            const BlockMask todo = (BlockMask)__ballot((mi & kOwnSlices) != 0);
            BlockMask m_in[kPPL], m_edge[kPPL], m_w[kPPL], m_g[kPPL];
#pragma unroll
            for (int j = 0; j < kPPL; ++j) {
                m_in[j] = (BlockMask)__ballot(mi & (1u << (kWaves * j)));
                m_edge[j] = (BlockMask)__ballot(mi & (1u << (8 + kWaves * j)));
                m_w[j] = (BlockMask)__ballot(mi & (1u << (16 + kWaves * j)));
                m_g[j] = (BlockMask)__ballot(mi & (1u << (24 + kWaves * j)));
            }
            for (int g8 = 0; g8 < kBlock; g8 += 8) {
                const uint32_t gt = (uint32_t)(todo >> g8) & 0xffu;
                if (gt == 0) continue;
                uint32_t gi[kPPL], gw[kPPL], gg[kPPL], ge[kPPL];
#pragma unroll
                for (int j = 0; j < kPPL; ++j) {
                    gi[j] = (uint32_t)(m_in[j] >> g8);
                    gw[j] = (uint32_t)(m_w[j] >> g8);
                    gg[j] = (uint32_t)(m_g[j] >> g8);
                    ge[j] = (uint32_t)(m_edge[j] >> g8);
                }
                uint32_t off = (uint32_t)((l0 + g8) * 32);
                asm volatile("" : "+v"(off));
                const RecPos64 *rp8 = (const RecPos64 *)((const char *)sm.pos + off);
                const RecAmp64 *ra8 = (const RecAmp64 *)((const char *)sm.amp + off);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if ((gt >> u) & 1u) line_terms_f64(rp8[u], ra8[u], u, kw, kd, gi, gw, gg, ge, se, sk);
            }
        }
        // nodes, as the single-precision form
#pragma unroll 1
        for (int j = 0; j < (in_nodes ? kSets : 0); ++j) {
            const int l = max(0, j - (kPPL - 1));
            const uint32_t it = l > 0 ? (uint32_t)wave >> (l - 1) : (uint32_t)(wave + kWaves * j);
            const uint32_t bit = 1u << (node_bit0(l) + it), wbit = 1u << (16 + l);
            uint32_t todo4 = blocks_of(bit << 8);
            if (l == 2) todo4 &= (wave & 1) ? 0xau : 0x5u;
            if (l == 3) todo4 &= 1u << wave;
            if (todo4 == 0) continue;
            const double w = (double)(64 << l);
            const double x = fma(x64, (double)(1 << l), (double)it * w + (0.5 * w - 0.5));
            double pe = 0.0, pk = 0.0;
#pragma unroll 1
            for (; todo4; todo4 &= todo4 - 1u) {
                const int l0 = __builtin_ctz(todo4) * kBlock;
                const uint32_t nb = sm.mode[l0 + lane].node;
                const BlockMask m = (BlockMask)__ballot((nb & bit) != 0);
                const BlockMask mw = m & (BlockMask)__ballot((nb & wbit) != 0);
                node_terms_f64(sm.pos + l0, sm.amp + l0, m, mw, x, (uint32_t)lane >> 5, pe, pk);
            }
            node_flush_f64(pe, pk, lane, acc[j]);
        }
        __syncthreads();
    }
    if (at_nodes && (kGroups > 1 || used)) {
        nodes_down<kNodes64, kThreadsF64>(sm.node, kBasis64, tid);
#pragma unroll 4
        for (int q = 0; q < kNodes64; ++q) {
            const double b = kBasis64.pt[q][lane];
#pragma unroll
            for (int j = 0; j < kPPL; ++j) {
                se[j] = fma(b, acc[j][0][q], se[j]);
                sk[j] = fma(b, acc[j][1][q], sk[j]);
            }
        }
        if (kGroups > 1) __syncthreads();   // add_groups overwrites the sums
    }
    add_groups<kGroups, kThreadsF64>([&](int o) { return (double *)&sg[o]; }, group, tid, se, sk);
    if (group > 0) return;
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        const uint32_t kq = (uint32_t)kt + (uint32_t)(kw + kSliceStep * j + lane);   // (may pass 2^31)
        if (kq < (uint32_t)kend) {
            const int64_t o = (int64_t)c * n_band + (int32_t)(kq - (uint32_t)k_first);
            if (ct.n_thr >= 0) {   // atomic continuum
                double ce, ck;
                continuum_point(ct, c, g.nu_min + (double)kq * g.h, ce, ck);
                se[j] += ce;
                sk[j] += ck;
            }
            eta[o] = se[j];
            kappa[o] = sk[j];
        }
    }
}

// ---------------------------------------------------------------------------
// in-window term count (the evaluation count of the metric)
// ---------------------------------------------------------------------------

__global__ void count_kernel(DevLines L, DevGrid g, const CellConst *cc, const CellSpecies *cs,
                             const int2 *band_ranges, int32_t n_cells, int32_t n_species,
                             int32_t k_first, int32_t n_band, unsigned long long *count)
{
    // lines i in the cell's candidate range for the band, grid-stride in x
    unsigned long long n = 0, nc = 0;
    for (int c = blockIdx.y; c < n_cells; c += gridDim.y) {
        const int2 rg = band_ranges[c];
        for (int64_t i0 = (int64_t)rg.x + (int64_t)blockIdx.x * blockDim.x; i0 < rg.y;
             i0 += (int64_t)gridDim.x * blockDim.x) {
            PairF64 p;
            if (i0 + threadIdx.x < rg.y &&
                pair_setup(L, g, cc[c], cs + (int64_t)c * n_species, cr_row(L, c), i0, threadIdx.x, p)) {
                const int32_t a = max(p.klo, k_first), b = min(p.khi, k_first + n_band - 1);
                if (b >= a) n += (unsigned long long)(b - a + 1);
                const int32_t ca = max(p.kclo, k_first), cb = min(p.kchi, k_first + n_band - 1);
                if (cb >= ca) nc += (unsigned long long)(cb - ca + 1);
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        n += __shfl_xor(n, o);
        nc += __shfl_xor(nc, o);
    }
    if ((threadIdx.x & 63) == 0) {
        if (n) atomicAdd(&count[0], n);
        if (nc) atomicAdd(&count[1], nc);
    }
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, int64_t n)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = v;
}

__global__ void check_cells_kernel(DevCells cells, int32_t *flags)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int S = cells.n_species;
    if (t >= (int64_t)cells.n_cells * (S + 1)) return;
    const int64_t c = t / (S + 1), s = t % (S + 1);
    if (s == S) {
        const double a = cells.T_tr[c], b = cells.T_v[c], e = cells.n_e[c];
        if (!(a > 0.0 && a <= DBL_MAX && b > 0.0 && b <= DBL_MAX)) atomicOr(&flags[0], 1);
        if (!(e >= 0.0 && e <= DBL_MAX)) atomicOr(&flags[1], 1);
    } else {
        const double n = cells.N[c * S + s];
        if (!(n >= 0.0 && n <= DBL_MAX)) atomicOr(&flags[1], 1);
    }
}

__global__ void fill_u64_kernel(unsigned long long *p, unsigned long long v, int64_t n)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = v;
}

// ---------------------------------------------------------------------------
// a7: serving.  One workgroup per (request, tile, chunk) item of an epoch's
// list, so workgroups retire all through an epoch and work on other streams
// (admissions, result copies) finds free slots without waiting for the epoch.
// An item accumulates eta/kappa of each cell of its chunk on its tile (in LDS /
// registers, never stored) and marches through them at once, producing the
// chunk's transmittance T and source S per point: I_out = I_in T + S.  The
// workgroup that completes the last chunk of a tile composes the tile's chunks
// far -> observer, and the one that completes the last tile sums the tiles:
// every sum runs in a fixed order, so nothing depends on what else shares the
// epoch or on the order in which items finish.
// ---------------------------------------------------------------------------

// One linear-j segment of length Ls (cm) from far node (fe, fk) to near node
// ne (scaled single-precision coefficients with their power-of-two scales),
// composed into the chunk's transmittance and source at ts[loc],
// ts[kTilePoints + loc]: I <- I e^-t + Ls (wf fe + wn ne), t = fk Ls.
__device__ __forceinline__ void linear_j_step(const float (&fe)[kPPL], const float (&fk)[kPPL], int fee, int fek,
                                              const float (&ne)[kPPL], int nee, double Ls, double *ts,
                                              int32_t kw, int lane)
{
    const double Lf = ldexp(Ls, fee), Ln = ldexp(Ls, nee);
    const float Lk = (float)fmin(ldexp(Ls, fek), 3.0e38);
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        int32_t loc = kw + kSliceStep * j + lane;
        asm volatile("" : "+v"(loc));   // recomputed here, not held across the accumulation
        const float t = fk[j] * Lk;
        const float ex = __builtin_amdgcn_exp2f(t * (float)(-kLog2e));
        float wf, wn;
        linear_j_weights_f32(t, ex, wf, wn);
        ts[loc] *= (double)ex;
        ts[kTilePoints + loc] = fma(ts[kTilePoints + loc], (double)ex, (double)(wf * fe[j]) * Lf + (double)(wn * ne[j]) * Ln);
    }
}

// Compose the chunks of the tile's points far -> observer (I <- I T + S in
// chunk order, from the far boundary's blackbody intensity when there is
// one), write I and the tile's trapezoid sum (h/2 at both window ends) in a
// fixed order: each thread's points, the wave's lanes by xor-shuffles, then
// the waves in order.  Called by the whole workgroup.
__device__ __forceinline__ void serve_compose_tile(const ServeReq &R, const DevGrid &g, int32_t tile, int32_t kw,
                                                   int lane, double *s_part)
{
    double part = 0.0;
#pragma unroll
    for (int j = 0; j < kPPL; ++j) {
        const int32_t loc = kw + kSliceStep * j + lane;
        const int32_t t = tile * kTilePoints + loc;
        if (t < R.n_window) {
            double I = R.T_far > 0.0 ? planck_f64(g.nu_min + (double)(R.k_first + t) * g.h, R.T_far) : 0.0;
            for (int32_t m = 0; m < R.n_chunks; ++m) {
                const double *ts = R.TS + ((int64_t)tile * R.n_chunks + m) * 2 * kTilePoints;
                I = fma(I, ts[loc], ts[kTilePoints + loc]);
            }
            R.I_out[t] = I;
            const double w = (t == 0 || t == R.n_window - 1) ? 0.5 * g.h : g.h;
            part = fma(w, I, part);
        }
    }
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
    if (lane == 0) s_part[kw / 64] = part;
    __syncthreads();
    if (threadIdx.x == 0) {
        double sum = 0.0;
        for (int wv = 0; wv < kAccumThreads / 64; ++wv) sum += s_part[wv];
        R.tile_part[tile] = sum;
    }
}

__global__ __launch_bounds__(kAccumThreads) __attribute__((amdgpu_waves_per_eu(LRT_SERVE_WAVES)))
void serve_kernel(DevLines L, DevGrid g, const ServeReq *reqs, const ServeItem *items, int32_t n_species)
{
    __shared__ AccumLds sm;
    __shared__ int32_t s_last;
    __shared__ double s_part[kAccumThreads / 64];
    const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6);
    const int32_t kw = wave * 64;
    {
        const ServeItem w = items[blockIdx.x];
        // the request's fields are read where used: held in registers across
        // the cell loop they would crowd out the accumulation's
        const ServeReq &R = reqs[w.req];
        const int32_t kt = R.k_first + w.tile * kTilePoints;
        const int32_t c0 = w.chunk * R.chunk_cells;
        const int32_t c1 = min(R.n_cells, c0 + R.chunk_cells);
        // the chunk's transmittance T and source S per point live in its own
        // slice of the request's buffer (each lane owns its points), not in
        // registers across the cells
        double *ts = R.TS + ((int64_t)w.tile * R.n_chunks + w.chunk) * 2 * kTilePoints;
#pragma unroll
        for (int j = 0; j < kPPL; ++j) {
            const int32_t loc = kw + kSliceStep * j + lane;
            ts[loc] = 1.0;
            ts[kTilePoints + loc] = 0.0;
        }
        // linear-j: the chunk owns the segments that end at its cells' midpoint
        // nodes (the first from the far end, the last chunk's also to the
        // observer), so it starts one cell early for its first far node
        float pe[kPPL], pk[kPPL];
        int pee = 0, pek = 0;
        double pds = 0.0;
        const bool linear = R.linear != 0;
        const int32_t cs0 = (linear && c0 > 0) ? c0 - 1 : c0;
        for (int32_t c = cs0; c < c1; ++c) {
            float e[kPPL], kp[kPPL];
            const int ese = R.escale[2 * c + 0], esk = R.escale[2 * c + 1];
            accum_cell_tile_f32<1>(&sm, 0, threadIdx.x, g, R.cc[c], R.cs + (int64_t)c * n_species,
                                R.lnd ? R.lnd + (int64_t)c * R.lnd_stride : nullptr, ese, esk,
                                R.ranges[(int64_t)c * R.n_tiles + w.tile], kt, kw, lane, e, kp);
            if (R.ct.n_thr >= 0) {
                // atomic continuum, added in double precision and rounded once
#pragma unroll
                for (int j = 0; j < kPPL; ++j) {
                    // (recomputed per cell: the per-point parts hoisted out of
                    // the cell loop would be spilled across the accumulation)
                    uint32_t kk = (uint32_t)kt + (uint32_t)(kw + kSliceStep * j + lane);
                    asm volatile("" : "+v"(kk));
                    const double nu = g.nu_min + (double)kk * g.h;
                    double ce, ck;
                    continuum_point(R.ct, c, nu, ce, ck);
                    e[j] = (float)((double)e[j] + ldexp(ce, -ese));
                    kp[j] = (float)((double)kp[j] + ldexp(ck, -esk));
                }
            }
            const double ds = R.ds[c];
            if (!linear) {
                float dsu;
                double dsl;
                segment_scales(ds, ese, esk, dsu, dsl);
#pragma unroll
                for (int j = 0; j < kPPL; ++j) {
                    int32_t loc = kw + kSliceStep * j + lane;
                    asm volatile("" : "+v"(loc));
                    double at, em;
                    segment_f32(e[j], kp[j], dsu, dsl, at, em);
                    ts[loc] *= at;
                    ts[kTilePoints + loc] = fma(ts[kTilePoints + loc], at, em);
                }
                continue;
            }
            if (c >= c0) {
                if (c == 0)   // far end -> first midpoint, both nodes the first cell's state
                    linear_j_step(e, kp, ese, esk, e, ese, 0.5 * ds, ts, kw, lane);
                else          // midpoint -> midpoint, kappa from the far node
                    linear_j_step(pe, pk, pee, pek, e, ese, 0.5 * (pds + ds), ts, kw, lane);
            }
#pragma unroll
            for (int j = 0; j < kPPL; ++j) {
                pe[j] = e[j];
                pk[j] = kp[j];
            }
            pee = ese;
            pek = esk;
            pds = ds;
        }
        if (linear && c1 == R.n_cells)   // last midpoint -> observer
            linear_j_step(pe, pk, pee, pek, pe, pee, 0.5 * pds, ts, kw, lane);
        // publish this chunk's T and S; the workgroup that brings the tile's
        // count to n_chunks composes the tile (device-scope fences around the
        // counter: the chunks may have run on other XCDs)
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) s_last = atomicAdd(R.done + w.tile, 1) == R.n_chunks - 1;
        __syncthreads();
        if (!s_last) return;
        __threadfence();
        serve_compose_tile(R, g, w.tile, kw, lane, s_part);
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) s_last = atomicAdd(R.done + R.n_tiles, 1) == R.n_tiles - 1;
        __syncthreads();
        if (!s_last) return;
        __threadfence();
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int32_t t = 0; t < R.n_tiles; ++t) sum += R.tile_part[t];
            *R.I_int = sum;
            *R.I_int_host = sum;
        }
    }
}




}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

hipError_t launch_thermo(const DevSpecies &sp, const DevCells &cells, const DevWidths &wd, double M_min,
                         uint64_t species_mask, CellConst *cc, CellSpecies *cs, hipStream_t st)
{
    const int64_t n = (int64_t)cells.n_cells * cells.n_species;
    if (n == 0) return hipSuccess;
    if (n > (int64_t)UINT32_MAX) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(thermo_kernel, dim3((unsigned)n), dim3(64), 0, st, sp, cells, wd, M_min, species_mask, cc, cs);
    return hipGetLastError();
}

hipError_t launch_ranges(const DevLines &L, const DevGrid &g, const CellConst *cc, int32_t n_cells,
                         int32_t k_first, int32_t n_band, int32_t tile_points, int2 *ranges,
                         hipStream_t st)
{
    const int32_t n_tiles = tiles_of(n_band, tile_points);
    const int64_t n = (int64_t)n_cells * n_tiles;
    hipLaunchKernelGGL(ranges_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, L, g, cc,
                       n_cells, k_first, n_band, tile_points, n_tiles, ranges);
    return hipGetLastError();
}

hipError_t launch_scale_bound(const DevBins &B, const CellConst *cc, const CellSpecies *cs,
                              const double *cont_lnb, int32_t n_cells, int32_t n_species,
                              int32_t *escale, hipStream_t st)
{
    if (n_cells == 0) return hipSuccess;
    if (n_cells < 8192)
        hipLaunchKernelGGL(scale_bound_kernel<4>, dim3((unsigned)n_cells), dim3(256), 0, st, B, cc, cs, cont_lnb,
                           n_cells, n_species, escale);
    else
        hipLaunchKernelGGL(scale_bound_kernel<1>, dim3((unsigned)n_cells), dim3(64), 0, st, B, cc, cs, cont_lnb,
                           n_cells, n_species, escale);
    return hipGetLastError();
}

hipError_t launch_cont_cells(const ContThr *thr, int32_t n_thr, const ContRec *rec, int32_t n_rec,
                             const DevCells &cells, const CellSpecies *cs, const DevCR &cr,
                             uint64_t species_mask, double nu_lo, double nu_hi, double *cum, double *ff,
                             double *lnb, hipStream_t st)
{
    if (cells.n_cells == 0) return hipSuccess;
    hipLaunchKernelGGL(cont_cells_kernel, dim3(blocks_for(cells.n_cells, 64)), dim3(64), 0, st, thr,
                       n_thr, rec, n_rec, cells, cs, cr, species_mask, nu_lo, nu_hi, cum, ff, lnb);
    return hipGetLastError();
}

hipError_t launch_accum_f32(const DevLines &L, const DevGrid &g, const CellConst *cc,
                            const CellSpecies *cs, const int32_t *escale, const int2 *ranges,
                            int32_t n_cells, int32_t n_species, int32_t k_first, int32_t n_band,
                            const DevCont &ct, float *eta, float *kappa, hipStream_t st)
{
    const int32_t n_tiles = tiles_of(n_band, kTilePoints);
    const int64_t n_blocks = (int64_t)n_tiles * n_cells;
    if (n_blocks > (int64_t)UINT32_MAX) return hipErrorInvalidConfiguration;
    const int groups = accum_groups(n_blocks, L.n, g.n_points, true);
    for (int64_t b0 = 0; b0 < n_blocks; b0 += kMaxLaunchBlocks) {
        const dim3 grid((unsigned)std::min(kMaxLaunchBlocks, n_blocks - b0));
#define LRT_ACCUM(G)                                                                                             \
    hipLaunchKernelGGL((accum_f32_kernel<G>), grid, dim3(kAccumThreads * G), 0, st, L, g, cc, cs, escale, ranges, \
                       n_cells, n_species, k_first, n_band, n_tiles, (uint32_t)b0, ct, eta, kappa)
        if (groups == 4) LRT_ACCUM(4); else if (groups == 2) LRT_ACCUM(2); else LRT_ACCUM(1);
#undef LRT_ACCUM
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_accum_f64(const DevLines &L, const DevGrid &g, const CellConst *cc,
                            const CellSpecies *cs, const int2 *ranges, int32_t n_cells,
                            int32_t n_species, int32_t k_first, int32_t n_band, const DevCont &ct,
                            double *eta, double *kappa, hipStream_t st)
{
    const int32_t n_tiles = tiles_of(n_band, kTileF64);
    const int64_t n_blocks = (int64_t)n_tiles * n_cells;
    if (n_blocks > (int64_t)UINT32_MAX) return hipErrorInvalidConfiguration;
    const int groups = accum_groups(n_blocks, L.n, g.n_points, false);
    for (int64_t b0 = 0; b0 < n_blocks; b0 += kMaxLaunchBlocks) {
        const dim3 grid((unsigned)std::min(kMaxLaunchBlocks, n_blocks - b0));
#define LRT_ACCUM(G)                                                                                   \
    hipLaunchKernelGGL((accum_f64_kernel<G>), grid, dim3(kThreadsF64 * G), 0, st, L, g, cc, cs, ranges, \
                       n_cells, n_species, k_first, n_band, n_tiles, (uint32_t)b0, ct, eta, kappa)
        if (groups == 4) LRT_ACCUM(4); else if (groups == 2) LRT_ACCUM(2); else LRT_ACCUM(1);
#undef LRT_ACCUM
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_count(const DevLines &L, const DevGrid &g, const CellConst *cc,
                        const CellSpecies *cs, const int2 *band_ranges, int32_t n_cells,
                        int32_t n_species, int32_t k_first, int32_t n_band,
                        unsigned long long *count, hipStream_t st)
{
    if (L.n == 0) return hipSuccess;
    hipLaunchKernelGGL(count_kernel, dim3(64, min(n_cells, 65535)), dim3(256), 0, st, L, g, cc, cs,
                       band_ranges, n_cells, n_species, k_first, n_band, count);
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

hipError_t launch_check_cells(const DevCells &cells, int32_t *flags, hipStream_t st)
{
    const int64_t n = (int64_t)cells.n_cells * (cells.n_species + 1);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(check_cells_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, cells, flags);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, unsigned long long v, int64_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u64_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}


hipError_t launch_serve(const DevLines &L, const DevGrid &g, const ServeReq *reqs,
                        const ServeItem *items, int32_t n_items, int32_t n_species, hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    hipLaunchKernelGGL(serve_kernel, dim3((unsigned)n_items), dim3(kAccumThreads), 0, st, L, g, reqs, items,
                       n_species);
    return hipGetLastError();
}

}  // namespace lrt

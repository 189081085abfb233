// Device functions shared by the source-iteration kernels (si_tile.hip) and the
// other step kernels (kernels.hip): a slot's opacity at a temperature, the face
// coefficients, and the wave flux with the static source Q.
#pragma once
#include <hip/hip_runtime.h>
#include "common.hpp"
#include "device_math.hpp"
#include "device_common.hpp"
#include "../../include/ugkwp.h"

namespace ugk {

// Stimulated-emission factor 1 - e^{-nu/T} (Sec. 3.3's opacity), or 1 without it.
__device__ inline double stim_factor(const Consts& K, double nu, double T)
{
    return K.stim ? one_less_exp_neg(math_tab(), nu / T) : 1.0;
}

// Frequency factor of group g at temperature T: Simpson's mean of nu^-p over
// the group, times the stimulated-emission factor when that is on.
__device__ __forceinline__ double group_factor(const Dev& D, const Consts& K, int edge_off, int g, double T)
{
    if (!K.stim) return D.simpson[edge_off + g];
    const double nl = D.nu[edge_off + g], nh = D.nu[edge_off + g + 1], nm = 0.5 * (nl + nh);
    return sixth(nu_pow(nl, K.nu_power) * stim_factor(K, nl, T) + 4.0 * nu_pow(nm, K.nu_power) * stim_factor(K, nm, T)
                 + nu_pow(nh, K.nu_power) * stim_factor(K, nh, T));
}

// Group opacity from the table (Sec. 3.4-3.5's printed opacities, tabulated by the
// caller): sigma is bilinear in (ln nu, ln T) on ln sigma, constant beyond the end
// nodes, and the group value is Simpson's rule over the group.  The nu intervals and
// weights of the Simpson points are fixed by the edges and read from tab_gi / tab_ga
// (k_tab_groups at set-up); only T is located here.
struct TablePlace {
    const double* row;     // ln sigma of the material at the T node below
    double b;              // weight of the node above
};

__device__ inline TablePlace table_place(const Dev& D, const Consts& K, int m, double T)
{
    TablePlace p;
    const int jt = table_locate_guess(D.tab_lT, K.tab_nT, log(T), K.tab_lT_inv, &p.b);
    p.row = D.tab_lsig + ((int64_t)m * K.tab_nT + jt) * K.tab_nnu;
    return p;
}

// sigma at Simpson point p (0 lower edge, 1 midpoint, 2 upper edge) of the group at edge e.
// (The rounding of ln sigma, up to some 1e-15 of sigma, outweighs exp_neg's: exp_neg_fine
// here cost 3% of Olson's 2-D sweeps.)
__device__ inline double table_point(const Dev& D, const Consts& K, TabPtr mt, const TablePlace& t, int e, int p)
{
    const double a = D.tab_ga[3 * e + p];
    const double* L = t.row + D.tab_gi[3 * e + p];
    const int n = K.tab_nnu;
    const double lo = (1.0 - a) * L[0] + a * L[1], hi = (1.0 - a) * L[n] + a * L[n + 1];
    return exp_neg(mt, -((1.0 - t.b) * lo + t.b * hi));
}

// of material m at T, the group at edge e = edge_off + g
__device__ inline double table_group_sigma(const Dev& D, const Consts& K, int m, int e, double T)
{
    const TabPtr mt = math_tab();
    const TablePlace t = table_place(D, K, m, T);
    const double v0 = table_point(D, K, mt, t, e, 0), v1 = table_point(D, K, mt, t, e, 1);
    return sixth(v0 + 4.0 * v1 + table_point(D, K, mt, t, e, 2));
}

// The same for the groups of a cell in consecutive lanes (g of Gp, edges g <= G, `on` for
// the whole cell), t the place of the cell's T: the upper edge is the next lane's lower
// one.  Called by whole wavefronts; two exponentials and eight table loads a lane instead
// of three and twelve.
__device__ inline double table_group_sigma_lanes(const Dev& D, const Consts& K, const TablePlace& t, int edge_off,
                                                 int g, int G, int Gp, bool on)
{
    const TabPtr mt = math_tab();
    const int e = edge_off + g;
    double v0 = 0.0, v1 = 0.0;
    if (on && g <= G) {
        v0 = table_point(D, K, mt, t, e, 0);
        if (g < G) v1 = table_point(D, K, mt, t, e, 1);
    }
    double v2 = next_lane(v0);
    if (on && g == G - 1 && G == Gp) v2 = table_point(D, K, mt, t, e, 2);
    return sixth(v0 + 4.0 * v1 + v2);
}

// T^-q; the paper's q = 1/2 without pow().
__device__ inline double temp_pow(double T, double q) { return q == 0.5 ? 1.0 / sqrt(T) : pow(T, -q); }

// The volumetric source acts in the steps that start before its switch-off time.
__device__ inline bool source_on(const Consts& K, uint32_t step)
{
    return K.has_src && (double)step * K.dt < K.q_toff;
}

// D of a face with face opacity sf (Appendix B, Eq. C2Formula); fc is the axis'
// factor -(c/eps)^2 dt / (3 h), h the centre distance (Inst::fcx, fcy).
__device__ inline double face_coef(const Consts& K, TabPtr t, double sf, double fc)
{
    return fc * coef_c2_over_dt(t, s_of_sigma(K, sf));
}

// What a sweep forms the opacity from: fixed tables, a power of the iterate's
// temperature with the stimulated-emission factor, or the opacity table.  OP_POWER also
// stands for Olson's heat capacity alone.  (Kept apart at compile time: pow() and the
// table's look-up together cost a sweep 64 to 140 spilled scalar registers.)
enum { OP_FIXED, OP_POWER, OP_TABLE };

__host__ inline int opacity_form(const Consts& K)
{
    return K.table ? OP_TABLE : (K.t_power != 0.0 || K.stim || K.olson) ? OP_POWER : OP_FIXED;
}

// What a slot's opacity is formed from.
struct SlotMat {
    double kap;
    int mat;
};

// sigma of the group at edge + g, at T (group_factor's frequency part included)
template <int OP>
__device__ __forceinline__ double slot_sigma(const Dev& D, const Consts& K, const SlotMat& s, int edge, int g, double T)
{
    if (OP == OP_TABLE) return table_group_sigma(D, K, s.mat, edge + g, T);
    return s.kap * temp_pow(T, K.t_power) * group_factor(D, K, edge, g, T);
}

// Opacity of a face between cells of opacity a and b.
__device__ inline double face_sigma(double a, double b) { return (a + b > 0.0) ? 2.0 * (a * b) / (a + b) : 0.0; }

// What a cell's energy equation is solved from: T^n, the iterate T^k, dt / C_v (or
// Olson's H and chi and the material energy U(T^n)).
struct CellHeat {
    double Tn, Tk, dtcv, H, chi, un;
    bool pinned;
};

// T^{k+1} of a cell from the exchange summed over its groups and (LIN) its derivative;
// *uend gets Olson's material energy.  Olson's heat capacity: the energy equation in the
// material energy U, U(T^{n+1}) = U(T^n) + exchange.  Literal: U(T^{k+1}) = U(T^n) +
// exchange(phi^k), solved for T^{k+1}; linearized: one Newton step at T^k with U and the
// emission linearized, whose material energy is U(T^k) + C_v(T^k)(T^{k+1} - T^k).
// uk, ck: U and C_v at T^k (linearized, with Olson's heat capacity).
template <bool TDEP, bool LIN>
__device__ inline double cell_temperature(const Consts& K, const CellHeat& c, double uk, double ck, double contrib,
                                          double dcon, double* uend)
{
    if (TDEP && c.H > 0.0) {
        if (c.pinned) {
            *uend = c.un;
            return c.Tn;
        }
        const double wdt = K.dt / (K.eps * K.eps);
        if (LIN) {
            const double T = c.Tk + (c.un - uk + wdt * contrib) / (ck + wdt * dcon);
            *uend = uk + ck * (T - c.Tk);
            return T;
        }
        *uend = c.un + wdt * contrib;
        return olson_temperature(c.H, c.chi, *uend, c.Tk);
    }
    if (c.pinned) return c.Tn;
    return LIN ? c.Tk + (c.Tn - c.Tk + c.dtcv * contrib) / (1.0 + c.dtcv * dcon) : c.Tn + c.dtcv * contrib;
}

// The same with U(T^k) and C_v(T^k) evaluated here.
template <bool TDEP, bool LIN>
__device__ inline double cell_temperature(const Consts& K, const CellHeat& c, double contrib, double dcon, double* uend)
{
    double uk = 0.0, ck = 0.0;
    if (TDEP && LIN && c.H > 0.0) {
        uk = olson_energy(c.H, c.chi, c.Tk);
        ck = olson_cv(c.H, c.chi, c.Tk);
    }
    return cell_temperature<TDEP, LIN>(K, c, uk, ck, contrib, dcon, uend);
}

// Residual sub-slots of a 2-D sweep k for instance inst: [RES_SLOTS][n_inst][RES_SUB],
// so that the slots of sweep 0 form one range cleared at the start of a step.
__device__ inline Resid* res_slot(const Dev& D, const Consts& K, int inst, int k)
{
    return D.res + ((int64_t)(k % RES_SLOTS) * K.n_inst + inst) * RES_SUB;
}

// The stopping test by one wavefront, r the sub-slot of each lane: max|rho^{k+1} - rho^k|
// <= si_tol max|rho^{k+1}| and max|T^{k+1} - T^k| <= si_tol max T^{k+1} (Algorithm 2).
__device__ inline bool resid_converged(const Consts& K, const Resid& r)
{
    const double drho = bitsd(wave_max_bits(bitsd(r.drho))), mrho = bitsd(wave_max_bits(bitsd(r.rho)));
    const double dT = bitsd(wave_max_bits(bitsd(r.dT))), mT = bitsd(wave_max_bits(bitsd(r.T)));
    return drho <= K.si_tol * mrho && dT <= K.si_tol * mT;
}

__device__ inline double minmod_diff(double a, double b)
{
    if (!(a * b > 0.0)) return 0.0;
    return fabs(a) < fabs(b) ? a : b;
}

// The faces of a slot's cell in the order XLO, XHI, YLO, YHI (the first two in
// 1-D): whether the neighbour across lies in the instance, its slot, the face's
// tally slot and area.  Index arithmetic only, so that a kernel can issue every
// load of the stencil before it waits for the first.
struct CellFaces {
    bool inside[4];
    int64_t nbj[4], fslot[4];
    double S[4];
};

template <int DIM>
__device__ inline CellFaces cell_faces(const Inst& I, int64_t j, int ix, int iy, int g)
{
    CellFaces F;
    const int Gp = I.Gp, nx = I.nx;
#pragma unroll
    for (int q = 0; q < 2 * DIM; ++q) {
        const bool lo = (q & 1) == 0;
        if (q < 2) {
            F.inside[q] = lo ? ix > 0 : ix < nx - 1;
            F.nbj[q] = j + (lo ? -Gp : Gp);
            F.fslot[q] = I.fx_off + (((int64_t)iy * (nx + 1) + ix + (lo ? 0 : 1)) << I.lgGp) + g;
            F.S[q] = I.dy;
        } else {
            F.inside[q] = lo ? iy > 0 : iy < I.ny - 1;
            F.nbj[q] = j + (lo ? -(int64_t)nx * Gp : (int64_t)nx * Gp);
            F.fslot[q] = I.fy_off + (((int64_t)(iy + (lo ? 0 : 1)) * nx + ix) << I.lgGp) + g;
            F.S[q] = I.dx;
        }
    }
    return F;
}

// Wave flux through the faces of slot j and its static source Q (Remark 3:
// coefficient C4 - e^{-s} where the cell sampled particles, C4 where it did
// not).  *inflow gets the energy the wave flux brings in through the domain
// boundary.
// EXT: compiled with the slope terms and the boundary-source ghosts (which the
// flags then switch); without it the base flux only, at fewer registers.
template <int DIM, bool EXT>
__device__ inline double wave_source(const Dev& D, const Consts& K, const Inst& I, int64_t j, const Slot& s,
                                     const CellFaces& F, double* inflow_out, const double* src, bool sub_rhop)
{
    const int g = s.g, nx = I.nx;
    const int ix = DIM == 1 ? s.lcell : s.lcell % nx, iy = DIM == 1 ? 0 : s.lcell / nx;
    const double cq = K.cq;
    const double* phib = D.phib + (int64_t)s.inst * 4 * MAX_G;
    constexpr int nf = 2 * DIM;
    const bool slopes = EXT && (K.flags & UGKWP_FLAG_SLOPES) != 0;
    const bool bpart = EXT && (K.flags & UGKWP_FLAG_BOUNDARY_PARTICLES) != 0;
    // every load first
    // the wave coefficient of a sampled slot: W(s), or this step's joint-cell value
    const double* wsamp = K.tau_C > 0.0 ? D.wsn : D.wc;
    const int nb_here = D.nbi[j];
    const double wc_here = wsamp[j], c4_here = D.c4[j], rho_here = D.rho[j];
    const double rhoh_here = sub_rhop ? src[j] - D.rhop[j] : src[j];
    double sl_here[2] = {0.0, 0.0}, b_here = 0.0, es_here = 0.0, wphys_here = 0.0;
    if (slopes) {
        sl_here[0] = D.sx[j];
        if (DIM == 2) sl_here[1] = D.sy[j];
        b_here = D.bcoef[j];
    }
    if (bpart) {
        es_here = D.es[j];
        wphys_here = D.wc[j];
    }
    int nb_n[4];
    double wc_n[4], c4_n[4], rhoh_n[4], pb[4], sl_n[4], b_n[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        nb_n[q] = 0;
        wc_n[q] = c4_n[q] = rhoh_n[q] = pb[q] = sl_n[q] = b_n[q] = 0.0;
        if (q >= nf) continue;
        if (F.inside[q]) {
            const int64_t n = F.nbj[q];
            nb_n[q] = D.nbi[n];
            wc_n[q] = wsamp[n];
            c4_n[q] = D.c4[n];
            rhoh_n[q] = sub_rhop ? src[n] - D.rhop[n] : src[n];
            if (slopes) {
                sl_n[q] = q < 2 ? D.sx[n] : D.sy[n];
                b_n[q] = D.bcoef[n];
            }
        } else if (I.bc[q] == BC_PLANCK) {
            pb[q] = phib[q * MAX_G + g];
        }
    }
    // gross particle crossings into / out of the cell
    const int64_t fl = I.fx_off + (((int64_t)iy * (nx + 1) + ix) << I.lgGp) + g;
    const int64_t fr = fl + I.Gp;
    const double tx0 = D.ftx[fl * 2 + 0], tx1 = D.ftx[fr * 2 + 1], tx2 = D.ftx[fl * 2 + 1], tx3 = D.ftx[fr * 2 + 0];
    double ty0 = 0.0, ty1 = 0.0, ty2 = 0.0, ty3 = 0.0;
    if (DIM == 2) {
        const int64_t fb = I.fy_off + (((int64_t)iy * nx + ix) << I.lgGp) + g;
        const int64_t ft = fb + ((int64_t)nx << I.lgGp);
        ty0 = D.fty[fb * 2 + 0]; ty1 = D.fty[ft * 2 + 1];
        ty2 = D.fty[fb * 2 + 1]; ty3 = D.fty[ft * 2 + 0];
    }
    const double Ah = nb_here > 0 ? wc_here : c4_here;
    const double here = Ah * rhoh_here;
    const double cs = K.c * K.c * K.dt / (6.0 * K.eps * K.eps);
    double fsum = 0.0, inflow = 0.0;
    // flux through a face along +axis: cq (A_low rho^h_low - A_high rho^h_high), with
    // slopes the upwind profiles at the face and cs (B_low s_low + B_high s_high)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q >= nf) continue;
        const bool lo = (q & 1) == 0;
        double Fpos;
        double there;
        if (!F.inside[q]) {
            const int bc = I.bc[q];
            if (bc == BC_REFLECT) continue;
            // a Planckian ghost that emitted boundary-source particles keeps C4 - e^{-s}
            double Ag = c4_here;
            if (bpart && bc == BC_PLANCK) {
                const double eov = es_here * pb[q];
                if (eov * I.V > 0.0 && K.n_cap >= 1 && eov / I.w_ref >= 1.0) Ag = wphys_here;
            }
            there = bc == BC_PLANCK ? Ag * pb[q] : 0.0;
        }
        if (!slopes) {
            if (F.inside[q]) {
                const double An = nb_n[q] > 0 ? wc_n[q] : c4_n[q];
                there = An * rhoh_n[q];
            }
            Fpos = lo ? cq * (there - here) : cq * (here - there);
        } else {
            const double slh = sl_here[q >> 1], h = q < 2 ? I.dx : I.dy;
            // this cell is the high cell of a LO face and the low cell of a HI face
            const double hv = Ah * (rhoh_here + (lo ? -0.5 : 0.5) * h * slh);
            const double hs = b_here * slh;
            double ts = 0.0;
            if (F.inside[q]) {
                const double An = nb_n[q] > 0 ? wc_n[q] : c4_n[q];
                there = An * (rhoh_n[q] + (lo ? 0.5 : -0.5) * h * sl_n[q]);
                ts = b_n[q] * sl_n[q];
            }
            Fpos = lo ? cq * (there - hv) + cs * (ts + hs) : cq * (hv - there) + cs * (hs + ts);
        }
        const double Fin = lo ? Fpos : -Fpos;
        fsum += F.S[q] * Fin;
        if (!F.inside[q]) inflow += K.dt * F.S[q] * Fin / K.c;
    }
    double a_in = tx0 + tx1;
    double a_out = tx2 + tx3;
    if (DIM == 2) {
        a_in += ty0 + ty1;
        a_out += ty2 + ty3;
    }
    *inflow_out = inflow;
    const double Q = rho_here + I.dt_V * fsum + (a_in - a_out) / I.V;
    // a volumetric source adds dt q in the steps it is on
    return source_on(K, *D.step) ? Q + K.dt * D.qsrc[j] : Q;
}

}  // namespace ugk

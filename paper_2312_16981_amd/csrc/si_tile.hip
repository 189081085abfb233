// The 1-D source iteration (Appendix B, Eq. macroSysAppendixIte, Algorithm 2),
// several sweeps per launch; see si_tile.hpp for the rounds.
//
// What bounds it: one sweep of a slab of a few thousand slots is a chain of
// about a microsecond (stencil, group sum, temperature, Planck integrals), but
// a launch per sweep took 5-6 us (10-15 with a temperature-dependent opacity):
// the chain, plus the launch, the loads of the slot's seven inputs and the
// residuals' atomics.  A round reads the inputs once, keeps them in registers
// and passes phi (and a T-dependent sigma) to the neighbouring cells through
// LDS, one barrier per sweep.  Source iteration of a step, a launch per sweep and now: a
// slab of 100 x 10 slots (3 sweeps) 25 and 12.6 us, 300 x 24 (31) 241 and 78, 1000 x 24
// with a T-dependent opacity (15) 221 and 90, 501 x 33 with the wave flux of every
// iterate (10) 181 and 72, 256 slabs of up to 4096 x 64 (4) 1452 and 1252.
#include "common.hpp"
#include "device_math.hpp"
#include "device_common.hpp"
#include "si_common.hpp"
#include "si_tile.hpp"
#include "kernels.hpp"

namespace ugk {

template <bool LIN, bool REG>
struct TileTab {
    RegTab r;
    __device__ inline TileTab() : r(reg_tab<LIN>()) {}
    __device__ inline const RegTab& sweep() const { return r; }
};
template <bool LIN>
struct TileTab<LIN, false> {
    __device__ inline TabPtr sweep() const { return math_tab(); }     // loaded again in every sweep
};

// The parts of a slot's wave flux that stay the same over the sweeps (WIT): its
// coefficient of rho^h and of the slope, rho^p, rho^n, the particles' net crossings and
// the source, and the Planckian ghosts' A phi(T_b).
struct WaveStatic {
    double A, B, rhop, rhon, pc, src, gl, gh;
};

__device__ inline WaveStatic wave_static(const Dev& D, const Consts& K, const Inst& I, int64_t j, int ix, int g,
                                         double pbl, double pbh)
{
    WaveStatic w;
    const bool sampled = D.nbi[j] > 0, bpart = (K.flags & UGKWP_FLAG_BOUNDARY_PARTICLES) != 0;
    const double c4 = D.c4[j];
    w.A = sampled ? (K.tau_C > 0.0 ? D.wsn : D.wc)[j] : c4;
    w.B = (K.flags & UGKWP_FLAG_SLOPES) ? D.bcoef[j] : 0.0;
    w.rhop = D.rhop[j];
    w.rhon = D.rho[j];
    w.src = source_on(K, *D.step) ? K.dt * D.qsrc[j] : 0.0;
    const int64_t fl = I.fx_off + ((int64_t)ix << I.lgGp) + g, fr = fl + I.Gp;
    const double a_in = D.ftx[fl * 2 + 0] + D.ftx[fr * 2 + 1], a_out = D.ftx[fl * 2 + 1] + D.ftx[fr * 2 + 0];
    w.pc = (a_in - a_out) / I.V;
    // a Planckian ghost that emitted boundary-source particles keeps C4 - e^{-s}
    double Al = c4, Ah = c4;
    if (bpart) {
        const double es = D.es[j], wc = D.wc[j];
        if (es * pbl * I.V > 0.0 && K.n_cap >= 1 && es * pbl / I.w_ref >= 1.0) Al = wc;
        if (es * pbh * I.V > 0.0 && K.n_cap >= 1 && es * pbh / I.w_ref >= 1.0) Ah = wc;
    }
    w.gl = Al * pbl;
    w.gh = Ah * pbh;
    return w;
}

// FIRST: round 0, which also evaluates the wave flux and Q; OP: how the opacity
// (and Olson's heat capacity) follows the iterate; LIN: the linearized sweep;
// EXT: slope terms and boundary-source ghosts in the wave flux; WIT: the wave flux of
// every sweep k >= 1 from its iterate (its cells reach two further with slopes, and the
// rounds after the first one more, K.tile_H in all); CPT cells per thread; REG: the
// Planck coefficients in registers (TileTab).
template <bool FIRST, bool SINGLE, int OP, bool LIN, bool EXT, bool WIT, int CPT, bool REG>
__global__ __launch_bounds__(SINGLE ? tile_max_threads(OP != OP_FIXED, REG) : TILE_BATCH_THREADS) void k_si_tile(Dev D, Consts K, int round)
{
    constexpr bool TDEP = OP != OP_FIXED, TABLE = OP == OP_TABLE;
    extern __shared__ double lds[];
    __shared__ unsigned long long lres[TILE_S_MAX][4][WAVE];    // residual maxima per sweep and lane
    __shared__ int dec[TILE_S_MAX + 1];
    static_assert(sizeof(lres) + sizeof(dec) == TILE_RES_LDS, "");
    const int lane = threadIdx.x & (WAVE - 1);
    warm_args<sizeof(Dev) + sizeof(Consts)>();
    const uint32_t now = *D.step;
    if (!FIRST && SINGLE) tile_gather(D, K, round - 1, dec);
    if (!(K.gate == GATE_OFF || now == K.gate)) return;
    // the block's instance and tile
    Inst I;
    int inst = 0, tile = blockIdx.x;
    if (SINGLE) {
        I = K.inst0;
    } else {
        const int2 bt = D.tile_blk[blockIdx.x];
        inst = __builtin_amdgcn_readfirstlane(bt.x);
        tile = __builtin_amdgcn_readfirstlane(bt.y);
        I = D.inst[inst];
    }
    const TilePlan plan = tile_plan(K, D.prev_ist[inst].conv_sweeps);
    if (!FIRST) {
        if (SINGLE) {
            __syncthreads();
            const int out = tile_outcome(K, round - 1, plan, dec);
            if (out != 0) {
                if (blockIdx.x == 0 && threadIdx.x == 0 && dec[TILE_S_MAX] == 0) tile_record(D, 0, out);
                return;
            }
        } else if (D.ist[inst].conv_sweeps != 0) {
            return;
        }
    }
    const TileRound rd = tile_round(K, plan, round);
    if (rd.ns == 0) return;
    if (FIRST && blockIdx.x == 0 && threadIdx.x == 0 && K.has_src) *D.src_on = source_on(K, now) ? 1 : 0;
    for (int q = threadIdx.x; q < rd.ns * 4 * WAVE; q += blockDim.x) lres[0][0][q] = 0ull;

    const int nx = I.nx, G = I.G, Gp = I.Gp;
    const int g = threadIdx.x & (Gp - 1), cpb = blockDim.x >> I.lgGp, C = cpb * CPT;
    const int W = C - 2 * K.tile_H;
    const int x0 = tile * W, x1 = min(x0 + W, nx), c0 = x0 - K.tile_H;      // interior, first cell
    const bool active = g < G;
    const bool slopes = WIT && (K.flags & UGKWP_FLAG_SLOPES) != 0;
    // Every sweep's output is right `reach` cells further in than its input from an end
    // beyond which the instance goes on: cell ci takes part up to sweep mlim.
    const int reach = slopes ? 2 : 1, behind = WIT && !FIRST ? 1 : 0;
    // rows of the tile's cells and the one beyond on either side: phi and (TDEP) sigma
    // twice, alternating; WIT: the wave flux's terms
    const int row = (C + 2) << I.lgGp;
    double* const Lphi = lds;
    double* const Lsig = lds + 2 * row;
    double* const Lup = lds + (TDEP ? 4 : 2) * row;      // A rho^h at the cell's high face
    double* const Ldn = Lup + row;                       // and at its low face
    double* const Lbs = Ldn + row;                       // B s
    const int64_t ncg = K.n_cg;
    // the round's input: phi(T^n) and rho^n, or the last sweep before it
    const double* phi_in = D.phi0;
    const double* rho_in = D.rho;
    const double* T_in = D.T;
    if (!FIRST) {
        const TileOut o = tile_out(K, plan, rd.k0 - 1);
        phi_in = o.final ? D.phi0n : D.tile_phi + o.at * ncg;
        rho_in = o.final ? D.rho_new : D.tile_rho + o.at * ncg;
        T_in = o.final ? D.T_new : D.tile_T + (int64_t)o.at * K.ncell;
    }
    double nu_lo = 0.0, nu_top = 0.0;
    if (g <= G) nu_lo = D.nu[I.edge_off + g];
    if (g == G - 1 && G == Gp) nu_top = D.nu[I.edge_off + G];
    // the ghosts' phi: Planckian, or 0 (a mirror's is taken from the cell)
    const double pbl = active && I.bc[XLO] == BC_PLANCK ? D.phib[((int64_t)inst * 4 + XLO) * MAX_G + g] : 0.0;
    const double pbh = active && I.bc[XHI] == BC_PLANCK ? D.phib[((int64_t)inst * 4 + XHI) * MAX_G + g] : 0.0;

    double phi[CPT], rho[CPT], Q[CPT], lam[CPT], rl[CPT], sig[CPT], Dl[CPT], Dh[CPT];
    double dph[CPT], infl[CPT];
    CellHeat ht[CPT];
    WaveStatic ws[CPT];
    SlotMat mat[CPT];
    int mlim[CPT];
    // every load first
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        const int ci = (threadIdx.x >> I.lgGp) + r * cpb, ix = c0 + ci;
        const bool ok = ix >= 0 && ix < nx, act = ok && active;
        const int64_t j = I.cg_off + ((int64_t)ix << I.lgGp) + g;
        const int cell = I.cell_off + ix;
        phi[r] = rho[r] = Q[r] = lam[r] = sig[r] = Dl[r] = Dh[r] = dph[r] = 0.0;
        infl[r] = 0.0;
        rl[r] = 1.0;
        ht[r] = {1.0, 1.0, 0.0, 0.0, 0.0, 0.0, false};
        mat[r].kap = 0.0;
        mat[r].mat = 0;
        ws[r] = WaveStatic{};
        mlim[r] = ok ? TILE_S_MAX : -1;
        if (ok && c0 > 0) mlim[r] = min(mlim[r], ci / reach - behind);
        if (ok && c0 + C < nx) mlim[r] = min(mlim[r], (C - 1 - ci) / reach - behind);
        double beyond = 0.0, sbeyond = 0.0;      // phi and sigma of the cell beyond the tile's end
        if (ok) {
            ht[r].Tn = D.T[cell];
            ht[r].Tk = FIRST ? ht[r].Tn : T_in[cell];
            ht[r].pinned = D.pinned[cell] != 0;
            ht[r].dtcv = D.dtcv[cell];
            if (TDEP && K.olson) {
                ht[r].H = D.olH[cell];
                ht[r].chi = D.olchi[cell];
            }
            if (TABLE) mat[r].mat = D.tab_mat[cell];
        }
        if (act) {
            phi[r] = phi_in[j];
            rho[r] = rho_in[j];
            if (!FIRST && !WIT) Q[r] = D.Q[j];
            if (WIT) ws[r] = wave_static(D, K, I, j, ix, g, ix == 0 ? pbl : 0.0, ix == nx - 1 ? pbh : 0.0);
            if (TDEP) {
                if (!TABLE) mat[r].kap = D.kappa[j];
            } else {
                lam[r] = D.sv[j];
                sig[r] = D.sig[j];
                const int64_t f = I.fx_off + ((int64_t)ix << I.lgGp) + g;
                Dl[r] = D.Dx[f];
                Dh[r] = D.Dx[f + Gp];
            }
            const bool el = ci == 0 && ix > 0, eh = ci == C - 1 && ix < nx - 1;
            if (el || eh) {
                const int64_t jb = j + (el ? -Gp : Gp);
                const int cb = cell + (el ? -1 : 1);
                beyond = phi_in[jb];
                SlotMat nb = {0.0, 0};
                if (TABLE) nb.mat = D.tab_mat[cb];
                else if (TDEP) nb.kap = D.kappa[jb];
                if (TDEP) sbeyond = FIRST ? D.sig[jb] : slot_sigma<OP>(D, K, nb, I.edge_off, g, T_in[cb]);
            }
            if (TDEP) sig[r] = FIRST ? D.sig[j] : slot_sigma<OP>(D, K, mat[r], I.edge_off, g, ht[r].Tk);
        }
        // the ghosts' values stay in both rows (no cell's update writes there)
        const int l = ((ci + 1) << I.lgGp) + g;
        const double ghost = ix == -1 ? pbl : (ix == nx ? pbh : 0.0);
        Lphi[l] = ok ? phi[r] : ghost;
        Lphi[l + row] = ok ? phi[r] : ghost;
        if (TDEP) Lsig[l] = sig[r];
        if (ci == 0) {
            Lphi[l - Gp] = ix == 0 ? pbl : beyond;
            Lphi[l - Gp + row] = ix == 0 ? pbl : 0.0;
            if (TDEP) Lsig[l - Gp] = sbeyond;
        }
        if (ci == C - 1) {                       // (a tile holds at least two cells)
            Lphi[l + Gp] = ix == nx - 1 ? pbh : beyond;
            Lphi[l + Gp + row] = ix == nx - 1 ? pbh : 0.0;
            if (TDEP) Lsig[l + Gp] = sbeyond;
        }
        if (!TDEP) rl[r] = 1.0 / (1.0 + lam[r]);
        // Q, and the linearized sweep's phi' at T^k (its upper-edge term from lane g + 1)
        if (FIRST && act) {
            const Slot s = {inst, ix, g, true, true};
            const CellFaces F = cell_faces<1>(I, j, ix, 0, g);
            Q[r] = wave_source<1, EXT>(D, K, I, j, s, F, &infl[r], D.rhoh, false);
            if (!WIT && ix >= x0 && ix < x1) {
                D.Q[j] = Q[r];
                if (infl[r] != 0.0)
                    atomicAdd(D.diag_sub + ((int64_t)inst * DIAG_SUB + (blockIdx.x & (DIAG_SUB - 1))) * 8 + 0, infl[r]);
            }
        }
        if (LIN) {
            const TabPtr mt = math_tab();
            const double we = ok && g <= G ? planck_edge_weight(mt, nu_lo / ht[r].Tk) : 0.0;
            double wh = next_lane(we);
            if (ok && g == G - 1 && G == Gp) wh = planck_edge_weight(mt, nu_top / ht[r].Tk);
            if (act) dph[r] = 4.0 * phi[r] / ht[r].Tk + K.a * K.c * (ht[r].Tk * ht[r].Tk * ht[r].Tk) * over_pi4_15(we - wh);
        }
    }
    __syncthreads();

    const TileTab<LIN, REG> tab;
    if (TDEP && K.olson)
#pragma unroll
        for (int r = 0; r < CPT; ++r) ht[r].un = olson_energy(ht[r].H, ht[r].chi, ht[r].Tn);
    int cur = 0;
    for (int m = 0; m < rd.ns; ++m) {
        const double* Pc = Lphi + cur * row;
        const double* Sc = Lsig + cur * row;
        double* Pn = Lphi + (cur ^ 1) * row;
        double* Sn = Lsig + (cur ^ 1) * row;
        // the sweep's output: in place, or its plane
        const bool final = rd.k0 + m == plan.fin;
        const int at = (round & 1) * K.tile_cap + m;
        double* const rho_out = final ? D.rho_new : D.tile_rho + at * ncg;
        double* const phi_out = final ? D.phi0n : D.tile_phi + at * ncg;
        double* const T_out = final ? D.T_new : D.tile_T + (int64_t)at * K.ncell;
        if (WIT && !(FIRST && m == 0)) {
            // the wave flux from the iterate rho^h = rho^k - rho^p (Algorithm 2): rho^h
            // to the neighbours (through the row the new phi will take), the slopes
            // (MINMOD, limited to a non-negative profile), then both to the faces
            if (slopes) {
#pragma unroll
                for (int r = 0; r < CPT; ++r) {
                    const int ci = (threadIdx.x >> I.lgGp) + r * cpb, ix = c0 + ci;
                    if (ix >= 0 && ix < nx) Pn[((ci + 1) << I.lgGp) + g] = rho[r] - ws[r].rhop;
                }
                __syncthreads();
            }
#pragma unroll
            for (int r = 0; r < CPT; ++r) {
                const int ci = (threadIdx.x >> I.lgGp) + r * cpb, ix = c0 + ci, l = ((ci + 1) << I.lgGp) + g;
                const double rh = rho[r] - ws[r].rhop;
                if (slopes) {
                    const double lf = ix > 0 ? Pn[l - Gp] : (I.bc[XLO] == BC_REFLECT ? rh : pbl);
                    const double rt = ix < nx - 1 ? Pn[l + Gp] : (I.bc[XHI] == BC_REFLECT ? rh : pbh);
                    double sx = minmod_diff(rh - lf, rt - rh) / I.dx;
                    if (!(rh > 0.0)) sx = 0.0;
                    else if (fabs(sx) * I.dx > 2.0 * rh) sx = sx * (2.0 * rh / (fabs(sx) * I.dx));
                    Lup[l] = ws[r].A * (rh + 0.5 * I.dx * sx);
                    Ldn[l] = ws[r].A * (rh + -0.5 * I.dx * sx);
                    Lbs[l] = ws[r].B * sx;
                } else {
                    Lup[l] = ws[r].A * rh;
                }
            }
            __syncthreads();
            const double cs = K.c * K.c * K.dt / (6.0 * K.eps * K.eps);
#pragma unroll
            for (int r = 0; r < CPT; ++r) {
                const int ci = (threadIdx.x >> I.lgGp) + r * cpb, ix = c0 + ci, l = ((ci + 1) << I.lgGp) + g;
                if (ix < 0 || ix >= nx || !active) continue;
                const double* const dn = slopes ? Ldn : Lup;
                const double hs = slopes ? Lbs[l] : 0.0;
                double fsum = 0.0, inflow = 0.0;
                if (ix > 0 || I.bc[XLO] != BC_REFLECT) {
                    const double there = ix > 0 ? Lup[l - Gp] : ws[r].gl;
                    double F = K.cq * (there - dn[l]);
                    if (slopes) F += cs * ((ix > 0 ? Lbs[l - Gp] : 0.0) + hs);
                    fsum += I.dy * F;
                    if (ix == 0) inflow += K.dt * I.dy * F / K.c;
                }
                if (ix < nx - 1 || I.bc[XHI] != BC_REFLECT) {
                    const double there = ix < nx - 1 ? dn[l + Gp] : ws[r].gh;
                    double F = K.cq * (Lup[l] - there);
                    if (slopes) F += cs * (hs + (ix < nx - 1 ? Lbs[l + Gp] : 0.0));
                    fsum += I.dy * -F;
                    if (ix == nx - 1) inflow += K.dt * I.dy * -F / K.c;
                }
                Q[r] = ws[r].rhon + I.dt_V * fsum + ws[r].pc + ws[r].src;
                infl[r] = inflow;
            }
        }
        const auto& mt = tab.sweep();
        const TabPtr ct = math_tab();
        double dr = 0.0, mr = 0.0, dT = 0.0, mT = 0.0;
#pragma unroll
        for (int r = 0; r < CPT; ++r) {
            const int ci = (threadIdx.x >> I.lgGp) + r * cpb, ix = c0 + ci;
            const bool work = m <= mlim[r];
            if (__ballot(work) == 0ull) continue;
            const bool act = work && active;
            const bool inner = work && ix >= x0 && ix < x1;
            const int l = ((ci + 1) << I.lgGp) + g;
            double contrib = 0.0, dcon = 0.0, rr = 0.0, b = 0.0;
            if (act) {
                if (TDEP) {
                    // the coefficient step of Algorithm 2 at T^k
                    lam[r] = s_of_sigma(K, sig[r]);
                    rl[r] = 1.0 / (1.0 + lam[r]);
                    Dl[r] = face_coef(K, ct, ix > 0 ? face_sigma(sig[r], Sc[l - Gp]) : sig[r], I.fcx);
                    Dh[r] = face_coef(K, ct, ix < nx - 1 ? face_sigma(sig[r], Sc[l + Gp]) : sig[r], I.fcx);
                }
                double pl = Pc[l - Gp], ph = Pc[l + Gp];
                if (ix == 0 && I.bc[XLO] == BC_REFLECT) pl = phi[r];
                if (ix == nx - 1 && I.bc[XHI] == BC_REFLECT) ph = phi[r];
                double lap = I.dy * Dl[r] * (pl - phi[r]);
                lap += I.dy * Dh[r] * (ph - phi[r]);
                b = Q[r] + I.dt_V * lap;
                const double em = quotient(b - phi[r], 1.0 + lam[r], rl[r]);
                contrib = sig[r] * em;
                if (LIN) dcon = quotient(sig[r] * dph[r], 1.0 + lam[r], rl[r]);
                else rr = quotient(b + lam[r] * phi[r], 1.0 + lam[r], rl[r]);
            }
            contrib = group_sum(contrib, Gp);
            if (LIN) dcon = group_sum(dcon, Gp);
            double Tnew = 1.0, uend = 0.0;
            bool bad = false;
            if (work) {
                Tnew = cell_temperature<TDEP, LIN>(K, ht[r], contrib, dcon, &uend);
                if (LIN && active) {
                    const double pe = ht[r].pinned ? phi[r] : phi[r] + dph[r] * (Tnew - ht[r].Tk);
                    rr = quotient(b + lam[r] * pe, 1.0 + lam[r], rl[r]);
                }
                if (!(Tnew > 0.0) || !isfinite(Tnew)) {
                    bad = true;
                    Tnew = 1.0;
                }
            }
            // phi^{k+1}: lane g evaluates its lower edge, the upper one comes from lane g + 1
            const bool edge_lane = work && g <= G;
            const double xe = edge_lane ? nu_lo / Tnew : 0.0;
            double ve = 0.0, we = 0.0;
            if (edge_lane) {
                if (LIN) planck_edge_both(mt, xe, &ve, &we);
                else ve = planck_edge_value(mt, xe);
            }
            double xh = next_lane(xe), vh = next_lane(ve), wh = LIN ? next_lane(we) : 0.0;
            if (work && g == G - 1 && G == Gp) {
                xh = nu_top / Tnew;
                if (LIN) planck_edge_both(mt, xh, &vh, &wh);
                else vh = planck_edge_value(mt, xh);
            }
            if (act) {
                const double pn = phi_from_band(K.a, K.c, Tnew, planck_band_from_edges(xe, ve, xh, vh));
                if (inner) {
                    const int64_t j = I.cg_off + ((int64_t)ix << I.lgGp) + g;
                    rho_out[j] = rr;
                    phi_out[j] = pn;
                    dr = nan_max(dr, fabs(rr - rho[r]));
                    mr = nan_max(mr, fabs(rr));
                    if (WIT) {
                        // the flux and its boundary inflow, for the commit
                        (final ? D.Q : D.tile_Q + at * ncg)[j] = Q[r];
                        if (ix == 0 || ix == nx - 1)
                            tile_inflow(D, K, inst, final ? 2 * K.tile_cap : at)[(ix == 0 ? 0 : MAX_G) + g] = infl[r];
                    }
                }
                rho[r] = rr;
                phi[r] = pn;
                Pn[l] = pn;
                if (LIN) dph[r] = 4.0 * pn / Tnew + K.a * K.c * (Tnew * Tnew * Tnew) * over_pi4_15(we - wh);
            }
            if (TDEP && m + 1 < rd.ns) {
                if (TABLE) {
                    TablePlace t = {nullptr, 0.0};
                    if (work) t = table_place(D, K, mat[r].mat, Tnew);
                    sig[r] = table_group_sigma_lanes(D, K, t, I.edge_off, g, G, Gp, work);
                } else if (act) sig[r] = slot_sigma<OP>(D, K, mat[r], I.edge_off, g, Tnew);
                if (act) Sn[l] = sig[r];
            }
            if (inner && g == 0) {
                const int cell = I.cell_off + ix;
                T_out[cell] = Tnew;
                if (TDEP && ht[r].H > 0.0) (final ? D.uend : D.tile_u + (int64_t)at * K.ncell)[cell] = uend;
                dT = nan_max(dT, fabs(Tnew - ht[r].Tk));
                mT = nan_max(mT, bad ? __builtin_nan("") : Tnew);
            }
            if (work) ht[r].Tk = Tnew;
        }
        // the sweep's residual maxima per lane (non-negative or NaN, ordered by their
        // bits) over the block's wavefronts; a reduction over the lanes in every
        // wavefront and sweep would cost more than the rest of the update's arithmetic
        // outside the Planck integrals, so it is left to the end of the round
        atomicMax(&lres[m][0][lane], dbits(dr));
        atomicMax(&lres[m][1][lane], dbits(mr));
        if (g == 0) {
            atomicMax(&lres[m][2][lane], dbits(dT));
            atomicMax(&lres[m][3][lane], dbits(mT));
        }
        cur ^= 1;
        __syncthreads();
    }
    for (int q = threadIdx.x / WAVE; q < rd.ns * 4; q += blockDim.x / WAVE) {
        const unsigned long long v = wave_max_bits(bitsd(lres[0][q][lane]));
        if (lane == 0) ((unsigned long long*)(tile_res(D, K, round, q >> 2) + blockIdx.x))[q & 3] = v;
    }
}

// The outcome of a round for every instance of a batch still running, one
// wavefront per instance.
__global__ void k_tile_decide(Dev D, Consts K, int round)
{
    if (!gate_open(D, K, 0)) return;
    const int inst = blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
    const int lane = threadIdx.x & (WAVE - 1);
    if (inst >= K.n_inst || D.ist[inst].conv_sweeps != 0) return;
    const TileRound q = tile_round(K, tile_plan(K, D.prev_ist[inst].conv_sweeps), round);
    const int b0 = D.tile_start[inst], b1 = D.tile_start[inst + 1];
    for (int m = 0; m < q.ns; ++m) {
        const int v = tile_test(D, K, round, m, b0, b1, lane);
        if (v == 0) continue;
        if (lane == 0) tile_record(D, inst, v > 0 ? q.k0 + m + 1 : -1);
        return;
    }
}

// The same for a single instance of many tiles, by one block.  (Every block of the next
// launch reading every entry is quadratic in the mesh.)
constexpr int DECIDE_THREADS = 1024;
__global__ __launch_bounds__(DECIDE_THREADS) void k_tile_decide_one(Dev D, Consts K, int round)
{
    if (!gate_open(D, K, 0) || D.ist[0].conv_sweeps != 0) return;
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x / WAVE;
    const TileRound q = tile_round(K, tile_plan(K, D.prev_ist[0].conv_sweeps), round);
    __shared__ Resid part[DECIDE_THREADS / WAVE];
    for (int m = 0; m < q.ns; ++m) {
        const Resid x = tile_wave_most(tile_most(D, K, round, m, threadIdx.x, K.tile_blocks, DECIDE_THREADS));
        if (lane == 0) part[wid] = x;
        __syncthreads();
        Resid y = {0ull, 0ull, 0ull, 0ull};
        if (lane < DECIDE_THREADS / WAVE) y = part[lane];
        const int v = tile_verdict(K, tile_wave_most(y));      // every wavefront the same
        if (v != 0) {
            // (all wavefronts have read `conv_sweeps` before the first barrier)
            if (threadIdx.x == 0) tile_record(D, 0, v > 0 ? q.k0 + m + 1 : -1);
            return;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// launchers

template <bool FIRST, bool SINGLE, int OP, bool LIN, bool EXT, bool WIT>
static void tile_launch(const Dev& D, const Consts& K, int round, hipStream_t st)
{
    const int gmax = SINGLE ? K.inst0.Gp : MAX_G;
    const size_t lds = tile_rows_lds(K.tile_threads, K.tile_cpt, gmax, WIT, OP != OP_FIXED);
    if constexpr (SINGLE) {
        if constexpr (!WIT && OP == OP_FIXED) {
            if (K.tile_reg) {
                k_si_tile<FIRST, true, OP, LIN, EXT, false, 1, true><<<K.tile_blocks, K.tile_threads, lds, st>>>(D, K, round);
                return;
            }
        }
        k_si_tile<FIRST, true, OP, LIN, EXT, WIT, 1, false><<<K.tile_blocks, K.tile_threads, lds, st>>>(D, K, round);
    } else {
        k_si_tile<FIRST, false, OP, LIN, EXT, WIT, TILE_BATCH_CPT, false><<<K.tile_blocks, K.tile_threads, lds, st>>>(D, K, round);
    }
}

template <bool SINGLE, int OP, bool LIN>
static void tile_mode(const Dev& D, const Consts& K, int round, hipStream_t st)
{
    const bool ext = (K.flags & (UGKWP_FLAG_SLOPES | UGKWP_FLAG_BOUNDARY_PARTICLES)) != 0;
    if (K.flags & UGKWP_FLAG_WAVE_ITER) {
        if (round == 0) tile_launch<true, SINGLE, OP, LIN, true, true>(D, K, round, st);
        else tile_launch<false, SINGLE, OP, LIN, true, true>(D, K, round, st);
    } else if (round > 0) {
        tile_launch<false, SINGLE, OP, LIN, false, false>(D, K, round, st);
    } else if (ext) {
        tile_launch<true, SINGLE, OP, LIN, true, false>(D, K, round, st);
    } else {
        tile_launch<true, SINGLE, OP, LIN, false, false>(D, K, round, st);
    }
}

void launch_si_rounds(const Dev& D, const Consts& K, int r0, int r1, hipStream_t st)
{
    const bool lin = (K.flags & UGKWP_FLAG_SI_LINEARIZED) != 0;
    const int op = opacity_form(K);
    for (int r = r0; r < r1; ++r) {
        if (K.n_inst == 1) {
            if (op == OP_TABLE) lin ? tile_mode<true, OP_TABLE, true>(D, K, r, st) : tile_mode<true, OP_TABLE, false>(D, K, r, st);
            else if (op == OP_POWER) lin ? tile_mode<true, OP_POWER, true>(D, K, r, st) : tile_mode<true, OP_POWER, false>(D, K, r, st);
            else lin ? tile_mode<true, OP_FIXED, true>(D, K, r, st) : tile_mode<true, OP_FIXED, false>(D, K, r, st);
            if (!K.tile_fold) k_tile_decide_one<<<1, DECIDE_THREADS, 0, st>>>(D, K, r);
        } else {
            if (op == OP_TABLE) lin ? tile_mode<false, OP_TABLE, true>(D, K, r, st) : tile_mode<false, OP_TABLE, false>(D, K, r, st);
            else if (op == OP_POWER) lin ? tile_mode<false, OP_POWER, true>(D, K, r, st) : tile_mode<false, OP_POWER, false>(D, K, r, st);
            else lin ? tile_mode<false, OP_FIXED, true>(D, K, r, st) : tile_mode<false, OP_FIXED, false>(D, K, r, st);
            k_tile_decide<<<(unsigned)((K.n_inst * WAVE + 255) / 256), 256, 0, st>>>(D, K, r);
        }
    }
}

}  // namespace ugk

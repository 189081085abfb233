// The source iteration's sweeps of a 2-D mesh whose opacity follows the iterate
// (single-instance contexts; Appendix B, Eq. macroSysAppendixIte, Algorithm 2).
//
// What bounds it: double-precision arithmetic.  A thread per slot that forms its four
// face coefficients from its neighbours' opacities does every face twice; of 1157
// vector instructions a wavefront, 320 went there, 210 to Olson's heat capacity, 305
// to the next iterate's tabulated opacity, and 107 us to a sweep of 285 x 285 cells of
// 24 groups (168 to the first, with the wave flux).  A block therefore takes a patch of
// cells (4 x 4 with 32 lanes a cell): the opacity, phi and A rho^h of the patch and of the
// cells around it go to LDS, every face of the patch is computed once (2.5 a cell instead
// of 4) and passed on, and what depends on a cell's temperature alone is evaluated by one
// thread per cell: some 700 instructions, 74 us a sweep (116 the first).  (Means over every
// launch of Olson's problem in its first 80 steps, those past convergence included; over
// its 225 steps 84 and 140 us, where a sweep that works takes 95 and one past convergence 22.)
#include "common.hpp"
#include "device_math.hpp"
#include "device_common.hpp"
#include "si_common.hpp"
#include "kernels.hpp"

namespace ugk {

constexpr int GRID_LG = 9, GRID_THREADS = 1 << GRID_LG;
// log2 of a patch's sides, from log2 of the lanes per cell
__host__ __device__ inline int grid_lx(int lg) { return (GRID_LG - lg + 1) >> 1; }
__host__ __device__ inline int grid_ly(int lg) { return (GRID_LG - lg) >> 1; }

// Three blocks of 8 wavefronts per CU where the registers nearly allow it by themselves: 81 of
// them left two (the first sweep of the mesh above 116 -> 137 us).
template <int OP, bool EXT>
constexpr int grid_min_waves() { return OP == OP_TABLE && !EXT ? 6 : 1; }

template <bool FIRST, int OP, bool LIN, bool EXT>
__global__ __launch_bounds__(GRID_THREADS) __attribute__((amdgpu_waves_per_eu(grid_min_waves<OP, EXT>()))) void k_si_grid(Dev D, Consts K, int k, const double* phi_in,
                                                          double* phi_out, int decide_prev, const double* rho_in,
                                                          double* rho_out)
{
    constexpr bool TDEP = OP != OP_FIXED;
    extern __shared__ double lds[];
    __shared__ unsigned long long lres[4][WAVE];     // residual maxima per lane
    __shared__ int stop;
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x / WAVE;
    const uint32_t now = *D.step;
    const int cs_prev = FIRST ? 0 : D.ist[0].conv_sweeps;
    Resid res_prev = {0ull, 0ull, 0ull, 0ull};
    if (decide_prev && wid == 0) res_prev = res_slot(D, K, 0, k - 1)[lane];
    if (!(K.gate == GATE_OFF || now == K.gate)) return;
    if (FIRST && blockIdx.x == 0 && threadIdx.x == 0 && K.has_src) *D.src_on = source_on(K, now) ? 1 : 0;   // for the commit's ledger
    const Inst& I = K.inst0;
    const int nx = I.nx, ny = I.ny, G = I.G, Gp = I.Gp, lg = I.lgGp;
    // the patch, of 2^lx x 2^ly cells
    const int lx = grid_lx(lg), ly = grid_ly(lg), TX = 1 << lx, TY = 1 << ly;
    const uint32_t patches_x = (uint32_t)(nx + TX - 1) >> lx;
    const uint32_t patch = xcd_band(blockIdx.x, gridDim.x);
    const int py = (int)(patch / patches_x), px = (int)(patch - (uint32_t)py * patches_x);
    const int g = threadIdx.x & (Gp - 1), c = threadIdx.x >> lg;
    const int cx = c & (TX - 1), cy = c >> lx;
    const int ix = (px << lx) + cx, iy = (py << ly) + cy;
    const bool ok = ix < nx && iy < ny, act = ok && g < G;
    const int lcell = iy * nx + ix, cell = I.cell_off + lcell;
    const int64_t j = I.cg_off + ((int64_t)lcell << lg) + g;
    const int row = (TX + 2) << lg;                 // of the maps
    double* const Lphi = lds;
    double* const Lwav = Lphi + (TY + 2) * row;     // FIRST: the map of A rho^h
    double* const Lsig = Lwav + (FIRST ? (TY + 2) * row : 0);
    double* const Lfx = Lsig + (TY + 2) * row;      // [TY][TX + 1] faces along x
    double* const Lfy = Lfx + ((TY * (TX + 1)) << lg);      // [TY + 1][TX] along y
    double* const cell_a = Lfy + (((TY + 1) * TX) << lg);   // two values per cell, see below
    double* const cell_b = cell_a + (GRID_THREADS >> lg);
    // What is needed once a cell and takes long (Olson's energy and heat capacity, the
    // place of T in the table) is evaluated by the block's last threads, one a cell,
    // beside the other wavefronts' work, and passed on through LDS (every lane of a cell
    // evaluating them: 260 of a wavefront's 990 instructions, 77 us a sweep).
    const int cw = (int)threadIdx.x - (GRID_THREADS - (GRID_THREADS >> lg));
    const int wx = (px << lx) + (cw & (TX - 1)), wy = (py << ly) + (cw >> lx);
    const bool cell_lane = cw >= 0 && wx < nx && wy < ny;
    const int wcell = I.cell_off + wy * nx + wx;
    const double* phib = D.phib;
    // sigma of the sweeps' input iterate: the step's tables at T^n, the table's values
    // written by the sweep before, or formed here from T^k (both of buffers that no block
    // of this launch writes)
    auto sigma_in = [&](int64_t slot, int cl) __attribute__((always_inline)) -> double {
        if (FIRST || OP == OP_FIXED) return D.sig[slot];
        if (OP == OP_TABLE) return D.tab_sig[(int64_t)(k & 1) * K.n_cg + slot];
        return slot_sigma<OP>(D, K, {D.kappa[slot], 0}, I.edge_off, g, D.T_it[(int64_t)(k & 1) * K.ncell + cl]);
    };

    // every load first: the slot, the cell, and of the cells around the patch the
    // thread's share (their phi, or a ghost's; sigma < 0 beyond the boundary)
    double phi = 0.0, Qj = 0.0, rho_prev = 0.0, sig = 0.0;
    CellHeat ht = {1.0, 1.0, 0.0, 0.0, 0.0, 0.0, false};
    int mat = 0;
    double nu_lo = 0.0, nu_top = 0.0;
    if (g <= G) nu_lo = D.nu[I.edge_off + g];
    if (g == G - 1 && G == Gp) nu_top = D.nu[I.edge_off + G];
    if (ok) {
        ht.Tn = D.T[cell];
        ht.Tk = FIRST ? ht.Tn : D.T_new[cell];
        ht.pinned = D.pinned[cell] != 0;
        ht.dtcv = D.dtcv[cell];
        if (TDEP && K.olson) {
            ht.H = D.olH[cell];
            ht.chi = D.olchi[cell];
            if (!FIRST) ht.un = D.ol_un[cell];
        }
    }
    double wT = 1.0, wH = 0.0, wchi = 0.0;
    if (TDEP && cell_lane) {
        if (OP == OP_TABLE) mat = D.tab_mat[wcell];
        if (K.olson) {
            wT = FIRST ? D.T[wcell] : D.T_new[wcell];
            wH = D.olH[wcell];
            wchi = D.olchi[wcell];
        }
    }
    // A rho^h of a slot (the wave flux's upwind quantity, Remark 3), and the round's static
    // part of Q; with slopes or boundary sources wave_source forms it from the arrays
    constexpr bool FLUX = FIRST && !EXT;
    const double* wsamp = K.tau_C > 0.0 ? D.wsn : D.wc;
    auto wave_up = [&](int64_t slot) __attribute__((always_inline)) -> double {
        const double w = wsamp[slot], c4 = D.c4[slot];
        return (D.nbi[slot] > 0 ? w : c4) * D.rhoh[slot];
    };
    double here = 0.0, c4 = 0.0, lam = 0.0, Df[4] = {0.0, 0.0, 0.0, 0.0};
    if (act) {
        phi = phi_in[j];
        if (!FIRST) Qj = D.Q[j];
        if (FLUX) {
            here = wave_up(j);
            c4 = D.c4[j];
        }
        rho_prev = rho_in[j];
        sig = sigma_in(j, cell);
        if (!TDEP) {
            lam = D.sv[j];
            const int64_t fl = I.fx_off + (((int64_t)iy * (nx + 1) + ix) << lg) + g;
            const int64_t fb = I.fy_off + ((int64_t)lcell << lg) + g;
            Df[0] = D.Dx[fl];
            Df[1] = D.Dx[fl + Gp];
            Df[2] = D.Dy[fb];
            Df[3] = D.Dy[fb + ((int64_t)nx << lg)];
        }
    }
    // a cell around the patch, h = 0 .. 2 (TX + TY) - 1 (below, above, left, right): its
    // place in the maps, sigma (< 0 beyond the boundary), phi (or the ghost's) and A rho^h
    struct Around {
        int l;
        double s, p, w;
    };
    auto around = [&](int h) __attribute__((always_inline)) -> Around {
        const bool vert = h < 2 * TX;
        const int hq = vert ? h >> lx : (h - 2 * TX) >> ly, hp = vert ? h & (TX - 1) : (h - 2 * TX) & (TY - 1);
        const int hx = vert ? hp : (hq ? TX : -1), hy = vert ? (hq ? TY : -1) : hp;
        const int gx = (px << lx) + hx, gy = (py << ly) + hy;
        Around a = {(hy + 1) * row + ((hx + 1) << lg) + g, -1.0, 0.0, 0.0};
        if (gx >= 0 && gx < nx && gy >= 0 && gy < ny) {
            const int hc = gy * nx + gx;
            const int64_t hj = I.cg_off + ((int64_t)hc << lg) + g;
            a.s = 0.0;
            if (g < G) {
                a.p = phi_in[hj];
                if (TDEP) a.s = sigma_in(hj, I.cell_off + hc);
                if (FLUX) a.w = wave_up(hj);
            }
        } else {
            const int q = vert ? (hq ? YHI : YLO) : (hq ? XHI : XLO);
            if (I.bc[q] == BC_PLANCK && g < G) a.p = phib[q * MAX_G + g];
        }
        return a;
    };
    const int n_around = 2 * (TX + TY);
    Around ar = {0, 0.0, 0.0, 0.0};
    if (c < n_around) ar = around(c);
    double inflow = 0.0, crossings = 0.0, rhon = 0.0, src = 0.0;
    if (FIRST && EXT && act) {
        const Slot s = {0, lcell, g, true, true};
        const CellFaces F = cell_faces<2>(I, j, ix, iy, g);
        Qj = wave_source<2, true>(D, K, I, j, s, F, &inflow, D.rhoh, false);
    }
    if (FLUX && act) {
        // the particles' gross crossings into and out of the cell
        const int64_t fl = I.fx_off + (((int64_t)iy * (nx + 1) + ix) << lg) + g, fr = fl + Gp;
        const int64_t fb = I.fy_off + ((int64_t)lcell << lg) + g, ft = fb + ((int64_t)nx << lg);
        double a_in = D.ftx[fl * 2 + 0] + D.ftx[fr * 2 + 1], a_out = D.ftx[fl * 2 + 1] + D.ftx[fr * 2 + 0];
        a_in += D.fty[fb * 2 + 0] + D.fty[ft * 2 + 1];
        a_out += D.fty[fb * 2 + 1] + D.fty[ft * 2 + 0];
        crossings = (a_in - a_out) / I.V;
        rhon = D.rho[j];
        if (source_on(K, now)) src = K.dt * D.qsrc[j];
    }
    if (decide_prev) {
        // the stopping test of the sweep before, by every block from the same residuals,
        // while the loads are under way; block 0 records it
        if (wid == 0) {
            const bool conv = cs_prev == 0 && resid_converged(K, res_prev);
            if (lane == 0) {
                stop = (conv || cs_prev != 0) ? 1 : 0;
                if (conv && blockIdx.x == 0) {
                    D.ist[0].conv_sweeps = k;
                    atomicAdd((unsigned long long*)(D.counters + CNT_CONV), 1ull);
                }
            }
        }
        __syncthreads();
        if (stop) return;
    } else if (cs_prev != 0) {
        return;
    }
    if (threadIdx.x < 4 * WAVE) lres[wid][lane] = 0ull;
    const int l = (cy + 1) * row + ((cx + 1) << lg) + g;
    // (a slot of the patch beyond the boundary is a ghost where it touches the mesh)
    if (TDEP) Lsig[l] = ok ? sig : -1.0;
    Lphi[l] = phi;
    if (FLUX) Lwav[l] = here;
    if (!ok && ix == nx && iy < ny && I.bc[XHI] == BC_PLANCK) Lphi[l] = phib[XHI * MAX_G + g];
    if (!ok && iy == ny && ix < nx && I.bc[YHI] == BC_PLANCK) Lphi[l] = phib[YHI * MAX_G + g];
    for (int h = c; h < n_around; h += GRID_THREADS >> lg) {
        if (h > c) ar = around(h);
        if (TDEP) Lsig[ar.l] = ar.s;
        Lphi[ar.l] = ar.p;
        if (FLUX) Lwav[ar.l] = ar.w;
    }
    __syncthreads();
    const TabPtr mt = math_tab();
    // the faces: each thread its cell's low ones, and the patch's far ones shared out
    auto face = [&](int a, int b, double fc) __attribute__((always_inline)) -> double {
        const double sa = Lsig[a], sb = Lsig[b];
        return face_coef(K, mt, sa < 0.0 ? fmax(sb, 0.0) : (sb < 0.0 ? sa : face_sigma(sa, sb)), fc);
    };
    const int lfx = ((cy * (TX + 1) + cx) << lg) + g, lfy = ((cy * TX + cx) << lg) + g;
    if (TDEP) {
        Lfx[lfx] = Df[0] = face(l - Gp, l, I.fcx);
        Lfy[lfy] = Df[2] = face(l - row, l, I.fcy);
    }
    if (TDEP && c < TX + TY) {
        if (c < TX) Lfy[((TY * TX + c) << lg) + g] = face(TY * row + ((c + 1) << lg) + g, (TY + 1) * row + ((c + 1) << lg) + g, I.fcy);
        else {
            const int r = c - TX;
            Lfx[((r * (TX + 1) + TX) << lg) + g] = face((r + 1) * row + (TX << lg) + g, (r + 1) * row + ((TX + 1) << lg) + g, I.fcx);
        }
    }
    if (TDEP && K.olson && (LIN || FIRST) && cell_lane) {
        cell_a[cw] = olson_energy(wH, wchi, wT);
        if (LIN) cell_b[cw] = olson_cv(wH, wchi, wT);
    }
    // linearized iteration: d phi_g / dT at T^k, its upper-edge term from lane g+1
    double dph = 0.0;
    if (LIN) {
        const double we = ok && g <= G ? planck_edge_weight(mt, nu_lo / ht.Tk) : 0.0;
        double wh = next_lane(we);
        if (ok && g == G - 1 && G == Gp) wh = planck_edge_weight(mt, nu_top / ht.Tk);
        if (act) dph = 4.0 * phi / ht.Tk + K.a * K.c * (ht.Tk * ht.Tk * ht.Tk) * over_pi4_15(we - wh);
    }
    if (TDEP) __syncthreads();
    double contrib = 0.0, dcon = 0.0, r = 0.0, b = 0.0, rl = 1.0;    // rl = 1 / (1 + lambda)
    double dr = 0.0, mr = 0.0, dT = 0.0, mT = 0.0;
    if (FLUX && act) {
        // the flux through each face along +axis is cq (A_low rho^h_low - A_high rho^h_high)
        double fsum = 0.0;
        const double S[4] = {I.dy, I.dy, I.dx, I.dx};
        const bool edge[4] = {ix == 0, ix == nx - 1, iy == 0, iy == ny - 1};
        const int at[4] = {l - Gp, l + Gp, l - row, l + row};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (edge[q] && I.bc[q] == BC_REFLECT) continue;
            const double Fin = K.cq * ((edge[q] ? c4 * Lphi[at[q]] : Lwav[at[q]]) - here);
            fsum += S[q] * Fin;
            if (edge[q]) inflow += K.dt * S[q] * Fin / K.c;
        }
        Qj = rhon + I.dt_V * fsum + crossings;
        if (source_on(K, now)) Qj = Qj + src;
    }
    if (act) {
        if (TDEP) {
            lam = s_of_sigma(K, sig);
            Df[1] = Lfx[lfx + Gp];
            Df[3] = Lfy[lfy + (TX << lg)];
        }
        double pl = Lphi[l - Gp], ph = Lphi[l + Gp], pb = Lphi[l - row], pt = Lphi[l + row];
        if (ix == 0 && I.bc[XLO] == BC_REFLECT) pl = phi;
        if (ix == nx - 1 && I.bc[XHI] == BC_REFLECT) ph = phi;
        if (iy == 0 && I.bc[YLO] == BC_REFLECT) pb = phi;
        if (iy == ny - 1 && I.bc[YHI] == BC_REFLECT) pt = phi;
        double lap = I.dy * Df[0] * (pl - phi);
        lap += I.dy * Df[1] * (ph - phi);
        lap += I.dx * Df[2] * (pb - phi);
        lap += I.dx * Df[3] * (pt - phi);
        b = Qj + I.dt_V * lap;
        rl = 1.0 / (1.0 + lam);
        const double em = quotient(b - phi, 1.0 + lam, rl);
        contrib = sig * em;
        if (LIN) dcon = quotient(sig * dph, 1.0 + lam, rl);
        else r = quotient(b + lam * phi, 1.0 + lam, rl);
    }
    // group sum over the Gp lanes of the cell (every lane gets the same bits)
    contrib = group_sum(contrib, Gp);
    if (LIN) dcon = group_sum(dcon, Gp);
    double Tnew = 1.0, uend = 0.0;
    bool bad = false;
    if (ok) {
        double uk = 0.0, ck = 0.0;
        if (TDEP && K.olson && (LIN || FIRST)) {
            uk = cell_a[c];
            if (LIN) ck = cell_b[c];
        }
        if (FIRST) ht.un = uk;
        Tnew = cell_temperature<TDEP, LIN>(K, ht, uk, ck, contrib, dcon, &uend);
        if (act) {
            if (LIN) {
                // rho^{k+1} with the linearized emission of T^{k+1}
                const double pe = ht.pinned ? phi : phi + dph * (Tnew - ht.Tk);
                r = quotient(b + lam * pe, 1.0 + lam, rl);
            }
            dr = fabs(r - rho_prev);
            mr = fabs(r);
        }
        if (!(Tnew > 0.0) || !isfinite(Tnew)) {
            bad = true;
            Tnew = 1.0;
        }
        if (g == 0) {
            dT = fabs(Tnew - ht.Tk);
            mT = Tnew;
        }
    }
    if (OP == OP_TABLE) {
        // the place of T^{k+1} in the table, beside the Planck integrals
        __syncthreads();
        if (g == 0) cell_a[c] = Tnew;
        __syncthreads();
        if (cell_lane) {
            const TablePlace t = table_place(D, K, mat, cell_a[cw]);
            cell_a[cw] = __longlong_as_double((long long)(t.row - D.tab_lsig));
            cell_b[cw] = t.b;
        }
    }
    // phi^{k+1}: lane g evaluates the Planck edge value at its lower edge nu_g / T,
    // takes the upper one from lane g+1 (lane G-1 evaluates it itself when G = Gp)
    const bool edge_lane = ok && g <= G;
    const double xe = edge_lane ? nu_lo / Tnew : 0.0, ve = edge_lane ? planck_edge_value(mt, xe) : 0.0;
    double xh = next_lane(xe), vh = next_lane(ve);
    if (ok && g == G - 1 && G == Gp) {
        xh = nu_top / Tnew;
        vh = planck_edge_value(mt, xh);
    }
    double sig_next = 0.0;
    if (OP == OP_TABLE) {
        __syncthreads();
        sig_next = table_group_sigma_lanes(D, K, {D.tab_lsig + (int64_t)__double_as_longlong(cell_a[c]), cell_b[c]}, I.edge_off, g, G, Gp, ok);
    }
    if (blockIdx.x == 0 && threadIdx.x < RES_SUB) {
        const Resid z = {0ull, 0ull, 0ull, 0ull};
        res_slot(D, K, 0, k + 1)[threadIdx.x] = z;
    }
    if (act) {
        if (FIRST) D.Q[j] = Qj;
        rho_out[j] = r;
        phi_out[j] = phi_from_band(K.a, K.c, Tnew, planck_band_from_edges(xe, ve, xh, vh));
        // the next sweep's group sigma, at this sweep's T^{k+1}
        if (OP == OP_TABLE) D.tab_sig[(int64_t)((k + 1) & 1) * K.n_cg + j] = sig_next;
        // the boundary wave inflow: summed here, or with the wave flux of every
        // sweep from its iterate kept per slot for the commit (that of the last sweep)
        if (FIRST && (K.flags & UGKWP_FLAG_WAVE_ITER)) D.winflow[j] = inflow;
        else if (inflow != 0.0) atomicAdd(D.diag_sub + (blockIdx.x & (DIAG_SUB - 1)) * 8 + 0, inflow);
    }
    if (ok && g == 0) {
        if (bad) {
            atomicOr((unsigned long long*)(D.counters + CNT_ERR), ERR_TEMP);
        }
        D.T_new[cell] = Tnew;
        if (OP == OP_POWER) D.T_it[(int64_t)((k + 1) & 1) * K.ncell + cell] = Tnew;
        if (TDEP && ht.H > 0.0) D.uend[cell] = uend;
        if (TDEP && FIRST && K.olson) D.ol_un[cell] = ht.un;
    }
    // residual maxima (non-negative or NaN: as bit patterns): per lane over the block's
    // wavefronts in LDS, then over the lanes by one wavefront each (a reduction over the
    // lanes takes some 27 instructions)
    atomicMax(&lres[0][lane], dbits(dr));
    atomicMax(&lres[1][lane], dbits(mr));
    if (g == 0) {
        atomicMax(&lres[2][lane], dbits(dT));
        atomicMax(&lres[3][lane], dbits(mT));
    }
    __syncthreads();
    if (wid < 4) {
        const unsigned long long v = wave_max_bits(bitsd(lres[wid][lane]));
        if (lane == 0)
            atomicMax(&((unsigned long long*)(res_slot(D, K, 0, k) + (blockIdx.x & (RES_SUB - 1))))[wid], v);
    }
}

template <int OP, bool LIN>
static auto grid_kernel(const Consts& K, int k)
{
    if (k > 0) return k_si_grid<false, OP, LIN, false>;
    // the first sweep evaluates the wave flux: with slope terms or boundary-source
    // ghosts, its extended instantiation
    return (K.flags & (UGKWP_FLAG_SLOPES | UGKWP_FLAG_BOUNDARY_PARTICLES)) ? k_si_grid<true, OP, LIN, true>
                                                                           : k_si_grid<true, OP, LIN, false>;
}

void launch_si_grid(const Dev& D, const Consts& K, int k, const double* phi_in, double* phi_out, int decide_prev,
                    const double* rho_in, double* rho_out, hipStream_t st)
{
    const bool lin = (K.flags & UGKWP_FLAG_SI_LINEARIZED) != 0;
    const int op = opacity_form(K);
    auto kern = op == OP_TABLE   ? (lin ? grid_kernel<OP_TABLE, true>(K, k) : grid_kernel<OP_TABLE, false>(K, k))
                : op == OP_POWER ? (lin ? grid_kernel<OP_POWER, true>(K, k) : grid_kernel<OP_POWER, false>(K, k))
                                 : (lin ? grid_kernel<OP_FIXED, true>(K, k) : grid_kernel<OP_FIXED, false>(K, k));
    const Inst& I = K.inst0;
    const int lx = grid_lx(I.lgGp), ly = grid_ly(I.lgGp), TX = 1 << lx, TY = 1 << ly;
    const unsigned nb = (unsigned)(((I.nx + TX - 1) >> lx) * ((I.ny + TY - 1) >> ly));
    // maps, faces and the values per cell: 29 to 40 KB (the most with 64 lanes a cell: 48)
    const size_t map = (size_t)(TX + 2) * (TY + 2) * I.Gp, faces = (size_t)((TX + 1) * TY + TX * (TY + 1)) * I.Gp;
    const size_t lds = ((k == 0 ? 2 : 1) * map + (op == OP_FIXED ? 0 : map + faces + 2 * TX * TY)) * sizeof(double);
    kern<<<nb, GRID_THREADS, lds, st>>>(D, K, k, phi_in, phi_out, decide_prev, rho_in, rho_out);
}

}  // namespace ugk

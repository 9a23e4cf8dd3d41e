// The BZP barostat (App. E): NpT, or NpH with both thermostats off;
// isotropic (one v_W) or anisotropic (one v_W per dimension, each driven by
// the diagonal element of the centroid-virial stress tensor in its
// dimension and scaling the centroids and the box in that dimension).
// An OBABO step at a synchronized state is
//   O(dt/2) on the beads and on v_W; B(dt/2) on v_W and the beads together;
//   A(dt): the centroid mode under the barostat, the other modes by the free
//   ring-polymer flow, L <- exp(dt v_W) L; forces in the new box;
//   B(dt/2); O(dt/2) on v_W and on the beads.
// A BAOAB step is B(dt/2); A(dt/2); O(dt) on the beads and on v_W; A(dt/2)
// with the new v_W; forces; B(dt/2).
// The barostat's force is (3/W)[P V (P_CV - P_ext) + P kB T], the value for
// which the enthalpy H + K_W + U_W + J_W (App. A) is conserved in NpH.  Its
// kick is the exact flow of the kick: the centroid kinetic term, linear in
// time along the kick, integrates to h sum m|v~0|^2 + h^2 sum f~0.v~0 +
// (h^3/3) sum |f~0|^2/m from the momenta at the kick's start.  Its O step
// over a time t uses c1 = exp(-t/tau_0) and noise sqrt(P kB T / W) z, z the
// first Gaussian of counter (2^64 - 1, 0, s, q).
//
// The kicks need sums over all atoms taken between per-element updates, so a
// step is two passes, each followed by a one-block finalize (scalar barostat
// work), then the force pass in the new box.
#include "pimd_internal.h"
#include "pimd_device.h"

namespace pimd {

int npt_grid(int N, int P)
{
    const int A = kBlock / P;
    return (N + A - 1) / A;
}

// sinh(u)/u, by its Taylor series near 0
__device__ __forceinline__ double sinhc(double u)
{
    if (fabs(u) < 1e-3) {
        const double u2 = u * u;
        return 1.0 + u2 / 6.0 * (1.0 + u2 / 20.0 * (1.0 + u2 / 42.0));
    }
    return sinh(u) / u;
}

// v_W after a kick of length h.  k0x2 = sum m |v~0|^2, fv = sum f~0 . v~0,
// f2 = sum |f~0|^2 / m at the kick's start; k0x2 - vir + w = 3 P V P_CV.
__device__ double baro_kick(const NptArgs &a, double vw, double h, double k0x2, double vir,
                            double w, double V, double fv, double f2)
{
    const double W = a.wmass;
    return vw + h / W * (k0x2 - vir + w - 3.0 * (double)a.f.P * V * a.p_ext + 3.0 * a.kTP) +
           h * h / W * fv + h * h * h / (3.0 * W) * f2;
}

// One dimension's v_W after a kick of length h (anisotropic): the sums are
// that dimension's; k0x2 - vir + w = P V P_CV^aa.
__device__ double baro_kick_dim(const NptArgs &a, double vw, double h, double k0x2, double vir,
                                double w, double V, double fv, double f2)
{
    const double W = a.wmass;
    return vw + h / W * (k0x2 - vir + w - (double)a.f.P * V * a.p_ext + a.kTP) + h * h / W * fv +
           h * h * h / (3.0 * W) * f2;
}

// The noise of v_W's O step q of step s: the three Gaussians of the barostat's
// counter (isotropic: the first; anisotropic: one per dimension)
__device__ __forceinline__ void baro_noise(const NptArgs &a, unsigned long long s, unsigned long long q,
                                           double z[3])
{
    gauss3(a.f.seed, kBaroNoiseIndex, 0u, s, z, (unsigned)q);
}

__device__ __forceinline__ double baro_o(const NptArgs &a, double vw, double z)
{
    return a.bc1 * vw + a.bc2 * a.bsig * z;
}

// v_W of dimension d: the isotropic one, or that dimension's
__device__ __forceinline__ double vw_of(const NptArgs &a, const Ctl *c, int d)
{
    return a.aniso ? c->vwa[d] : c->vw;
}

// Matrix elements staged in LDS (P <= 64); beyond, the rows are read as they
// are needed, lanes side by side.
constexpr int kNptStage = 64 * 64;

__device__ __forceinline__ void stage_matrix(const double *m, int n, double *sM)
{
    if (n > kNptStage) return;
    constexpr int NM = 4;
    for (int e0 = threadIdx.x; e0 < n; e0 += NM * kBlock) {
        double r[NM];
#pragma unroll
        for (int u = 0; u < NM; ++u) r[u] = e0 + u * kBlock < n ? m[e0 + u * kBlock] : 0.0;
#pragma unroll
        for (int u = 0; u < NM; ++u)
            if (e0 + u * kBlock < n) sM[e0 + u * kBlock] = r[u];
    }
}

// out[d] = sum_j m[j][k] row[d][j], m row-major [P][P]: lanes k side by side
__device__ __forceinline__ void mode_sums(const double *m, const double *sM, int P, int k, const double *row,
                                          double out[3])
{
    out[0] = out[1] = out[2] = 0.0;
    auto run = [&](const double *mm) {
#pragma unroll 8
        for (int j = 0; j < P; ++j) {
            const double w = mm[j * P + k];
            out[0] += w * row[j];
            out[1] += w * row[P + j];
            out[2] += w * row[2 * P + j];
        }
    };
    if (P * P <= kNptStage)
        run(sM);
    else
        run(m);
}

// The two passes are bound by the latency of one tile (384 atoms at P = 32 are
// 48 blocks): reads, transform, O steps, reduction.  So every read is issued at
// the start, the noise is formed while they are in flight, the matrix comes
// through LDS (read in place, a row per lane, it cost each transform a chain of
// uncoalesced loads), and the positions' modes are carried from step to step as
// in the other step passes, so that no pass transforms x.  At that size pass A
// took 8.8 us and takes 6.9, pass B 10.9 and 6.8, their finalizes 6.3 and 3.9,
// now 4.8 and 3.0.

// Pass A.  Thread = (atom, mode); a block holds kBlock/P whole atoms.
// Pending closing kick (with the barostat's sums before it) and O(dt/2) of the
// last step; the estimators' sums; with NPT_STEP the opening O(dt/2) and the
// barostat's sums after it.  Writes v~ and f~.  AN: the anisotropic barostat.
template <bool AN>
__global__ __launch_bounds__(kBlock) void k_npt_a(NptArgs na, int mode)
{
    constexpr int NQ = AN ? NP_COUNT_ANISO : NP_COUNT, W = npt_row(AN);
    const FusedArgs &a = na.f;
    const int P = a.P, N = a.N, A = kBlock / P;
    __shared__ double sM[kNptStage];
    __shared__ double sF[3 * kBlock];
    __shared__ double red[NQ * (kBlock / 64)];
    const int t = threadIdx.x, la = t / P, k = t - la * P;
    const int i = blockIdx.x * A + la;
    const bool act = la < A && i < N;
    const unsigned oi = act ? (unsigned)a.orig[i] : 0u;
    const unsigned long long step = a.ctl->step;
    const bool closing = mode != NPT_EST && !a.ctl->synced;
    const bool opening = mode == NPT_STEP;
    const size_t vb = (size_t)i * 3 * P + k;
    double fr[3] = {0.0, 0.0, 0.0}, yt[3] = {0.0, 0.0, 0.0}, vt[3] = {0.0, 0.0, 0.0}, mk[8];
    double hm = 0.0, im = 0.0, sg = 0.0;
    if (act) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            fr[d] = a.f[vb + d * P];
            yt[d] = a.yt[vb + d * P];
            vt[d] = a.v[vb + d * P];
        }
        hm = a.atoms[i * 4 + AT_HALF_M];
        im = a.atoms[i * 4 + AT_INV_M];
        sg = a.atoms[i * 4 + AT_SIGMA];
#pragma unroll
        for (int q = 0; q < 8; ++q) mk[q] = a.modes[k * 8 + q];
    }
    stage_matrix(a.MT, P * P, sM);
    double zc[3] = {0.0, 0.0, 0.0}, zo[3] = {0.0, 0.0, 0.0};
    if (act && a.obabo && a.nvt) {
        if (closing) gauss3(a.seed, oi, (unsigned)k, step - 1, zc, 1u);
        if (opening) gauss3(a.seed, oi, (unsigned)k, step, zo, 0u);
    }
    if (act) {
#pragma unroll
        for (int d = 0; d < 3; ++d) sF[(la * 3 + d) * P + k] = fr[d];
    }
    __syncthreads();
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    if (act) {
        double ft[3];
        mode_sums(a.MT, sM, P, k, sF + la * 3 * P, ft);
#pragma unroll
        for (int d = 0; d < 3; ++d) na.ft[vb + d * P] = ft[d];
        auto o_step = [&](const double *z) {
#pragma unroll
            for (int d = 0; d < 3; ++d) vt[d] = mk[MD_C1] * vt[d] + mk[MD_C2] * sg * z[d];
        };
        if (closing) {
            if (k == 0) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    acc[NP_K0A] += hm * vt[d] * vt[d];
                    acc[NP_FVA] += ft[d] * vt[d];
                    if constexpr (AN) {
                        acc[NP_K0A3 + d] += hm * vt[d] * vt[d];
                        acc[NP_FVA3 + d] += ft[d] * vt[d];
                    }
                }
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) vt[d] += a.hdt * im * ft[d];
            if (a.obabo && a.nvt) o_step(zc);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            acc[NP_EKIN] += hm * vt[d] * vt[d];
            acc[NP_ESPRING] += hm * mk[MD_SPRING] * yt[d] * yt[d];
            acc[NP_VIR] += mk[MD_NONCENTROID] * yt[d] * ft[d];
            if constexpr (AN) acc[NP_VIR3 + d] += mk[MD_NONCENTROID] * yt[d] * ft[d];
            if (k == 0) {
                acc[NP_K0] += hm * vt[d] * vt[d];
                acc[NP_F2] += ft[d] * ft[d] * im;
                if constexpr (AN) acc[NP_F23 + d] += ft[d] * ft[d] * im;
            }
        }
        if (opening) {
            if (a.obabo && a.nvt) o_step(zo);
            if (k == 0) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    acc[NP_K0B] += hm * vt[d] * vt[d];
                    acc[NP_FVB] += ft[d] * vt[d];
                    if constexpr (AN) {
                        acc[NP_K0B3 + d] += hm * vt[d] * vt[d];
                        acc[NP_FVB3 + d] += ft[d] * vt[d];
                    }
                }
            }
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            a.v[vb + d * P] = vt[d];
            if (!isfinite(vt[d])) acc[NP_BAD] = 1.0;
        }
    }
    const double r = block_fold<NQ>(acc, red);
    if (t < NQ) na.part[(size_t)blockIdx.x * W + t] = r;
}

// Pass A's finalize (one block): the closing barostat kick and O step, the
// estimators of the synchronized state, then the opening O step and kick.
// What needs no sum (the noise, log V) is formed while the partials are read.
template <bool AN>
__global__ __launch_bounds__(kBlock) void k_npt_fin_a(NptArgs na, int mode, int nblocks)
{
    const FusedArgs &a = na.f;
    Ctl *c = a.ctl;
    // pass A's sums, then the force pass's energy and cell virial, then
    // (anisotropic) the diagonal of the cell virial
    constexpr int W = npt_row(AN), NR = kBlock / W, NB = 8, NW = kBlock / 64;
    constexpr int NQ = AN ? NP_COUNT_ANISO : NP_COUNT, NE = AN ? 5 : 2;
    constexpr int TE = NQ, TW = NQ + 1, TD = NQ + 2, NT = NQ + NE;
    static_assert(NQ <= W && NT <= 64, "one lane per sum");
    __shared__ double red[NT * NW];
    const int t = threadIdx.x, l = t & 63, w = t >> 6, pq = t & (W - 1);
    const unsigned long long step = c->step;
    const bool closing = mode != NPT_EST && !c->synced;
    const bool est_now = closing || mode == NPT_EST;
    const bool opening = mode == NPT_STEP;
    double vw = c->vw;
    double vwa[3] = {c->vwa[0], c->vwa[1], c->vwa[2]};
    const double V = c->box[0] * c->box[1] * c->box[2];
    double run_sum = 0.0, run_sq = 0.0;
    if (t < kNumEst) {
        run_sum = c->sum[t];
        run_sq = c->sumsq[t];
    }
    const unsigned long long count = c->count;
    double part = 0.0;
    for (int b0 = t / W; b0 < nblocks; b0 += NB * NR) {
        double pv[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int b = b0 + u * NR;
            pv[u] = (pq < NQ && b < nblocks) ? na.part[(size_t)b * W + pq] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) part += pv[u];
    }
    double fe[NE];
#pragma unroll
    for (int q = 0; q < NE; ++q) fe[q] = 0.0;
    const double2 *fp = reinterpret_cast<const double2 *>(a.fpartials);
    for (int b0 = t; b0 < a.n_fpartials; b0 += 4 * kBlock) {
        double2 e[4];
        double g[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = b0 + u * kBlock;
            const bool in = b < a.n_fpartials;
            e[u] = in ? fp[b] : make_double2(0.0, 0.0);
            if constexpr (AN) {
#pragma unroll
                for (int d = 0; d < 3; ++d) g[u][d] = in ? na.fdiag[(size_t)b * 3 + d] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            fe[0] += e[u].x;
            fe[1] += e[u].y;
            if constexpr (AN) {
#pragma unroll
                for (int d = 0; d < 3; ++d) fe[2 + d] += g[u][d];
            }
        }
    }
    double zc[3] = {0.0, 0.0, 0.0}, zo[3] = {0.0, 0.0, 0.0};
    const double logV = log(V);
    if (a.obabo && a.nvt) {
        if (closing) baro_noise(na, step - 1, 1, zc);
        if (opening) baro_noise(na, step, 0, zo);
    }
    // the waves' sums to LDS, then lane q of wave 0 has sum q
    if (W == 16) {
        double o = part;
        swap_lanes16(part, o);
        part += o;
    }
    {
        double o = part;
        swap_lanes32(part, o);
        part += o;
        double r[(NE + 3) / 4];
        wave_fold<NE, false>(fe, r);
        if (l < NQ) red[l * NW + w] = part;
        const int q0 = fold_value(l);
        if ((l & 15) == 0) {
#pragma unroll
            for (int s = 0; s < (NE + 3) / 4; ++s)
                if (4 * s + q0 < NE) red[(NQ + 4 * s + q0) * NW + w] = r[s];
        }
    }
    __syncthreads();
    if (t >= 64) return;
    double x = 0.0;
    if (t < NT) {
        x = red[t * NW];
#pragma unroll
        for (int u = 1; u < NW; ++u) x += red[t * NW + u];
    }
    auto tot = [&](int q) { return read_lane(x, q); };
    const double h = a.hdt, P = (double)a.P;
    const double vir = tot(NP_VIR), wc = tot(TW), f2 = tot(NP_F2);
    // the kicks: one v_W, or each dimension's with that dimension's sums
    auto kick = [&](int k0, int fv, int k03, int fv3) {
        if constexpr (AN) {
#pragma unroll
            for (int d = 0; d < 3; ++d)
                vwa[d] = baro_kick_dim(na, vwa[d], h, 2.0 * tot(k03 + d), tot(NP_VIR3 + d), tot(TD + d), V,
                                       tot(fv3 + d), tot(NP_F23 + d));
        } else {
            vw = baro_kick(na, vw, h, 2.0 * tot(k0), vir, wc, V, tot(fv), f2);
        }
    };
    auto o_step = [&](const double *z) {
        if constexpr (AN) {
#pragma unroll
            for (int d = 0; d < 3; ++d) vwa[d] = baro_o(na, vwa[d], z[d]);
        } else {
            vw = baro_o(na, vw, z[0]);
        }
    };
    if (closing) {
        kick(NP_K0A, NP_FVA, NP_K0A3, NP_FVA3);
        if (a.obabo && a.nvt) o_step(zc);
    }
    if (est_now) {
        const double ekin = tot(NP_EKIN), esp = tot(NP_ESPRING), epot = tot(TE);
        const double i3v = 1.0 / (3.0 * V), iP = 1.0 / P;
        double v[kNumEst];
        v[0] = ekin;
        v[1] = esp;
        v[2] = epot;
        v[3] = ekin + esp + epot;
        v[4] = a.kT15PN - esp * iP;
        v[5] = a.kT15N - vir / (2.0 * P);
        v[6] = ekin * a.temp_norm;
        v[7] = (2.0 * tot(NP_K0) - vir + wc) * iP * i3v;
        v[8] = (2.0 * a.kT15PN - (2.0 * esp - wc) * iP) * i3v;
        v[9] = (2.0 * ekin + wc) * i3v;
        // K_W + U_W + J_W (App. A), with J_W = -P kB T ln V; anisotropic:
        // the three barostat velocities' kinetic energies
        const double kw = AN ? 0.5 * na.wmass * (vwa[0] * vwa[0] + vwa[1] * vwa[1] + vwa[2] * vwa[2])
                             : 0.5 * na.wmass * vw * vw;
        const double eb = kw + P * na.p_ext * V - na.kTP * logV;
        double mine = v[0];   // lane q records estimator q
#pragma unroll
        for (int q = 1; q < kNumEst; ++q) mine = t == q ? v[q] : mine;
        if (t < kNumEst) {
            c->value[t] = mine;
            if (mode != NPT_EST) {
                c->sum[t] = run_sum + mine;
                c->sumsq[t] = run_sq + mine * mine;
            }
        }
        if (t == 0) {
            c->volume = V;
            c->ebaro = eb;
            c->enthalpy = v[3] + eb;
            c->est_step = step;
            if (mode != NPT_EST) c->count = count + 1;
        }
    }
    if (opening) {
        if (a.obabo && a.nvt) o_step(zo);
        kick(NP_K0B, NP_FVB, NP_K0B3, NP_FVB3);
    }
    const double bad = tot(NP_BAD);
    if (t == 0) {
        if (closing) c->synced = 1;
        c->vw = vw;
#pragma unroll
        for (int d = 0; d < 3; ++d) c->vwa[d] = vwa[d];
        if (bad != 0.0) c->nonfinite = 1;
        c->ran = 1;
    }
}

// The centroid's A over a time t at barostat velocity v: position by e and s,
// velocity by ei.
struct CentroidFlow {
    double e, ei, s;
};
__device__ __forceinline__ CentroidFlow centroid_flow(double t, double v)
{
    const double u = t * v;
    return {exp(u), exp(-u), t * sinhc(u)};
}

// Pass B.  Thread = (atom, mode) for the kick and the A step, then
// (atom, bead) for the inverse transform.  Writes v~, y~, x and the centroids.
__global__ __launch_bounds__(kBlock) void k_npt_b(NptArgs na)
{
    const FusedArgs &a = na.f;
    const int P = a.P, N = a.N, A = kBlock / P;
    __shared__ double sM[kNptStage];
    __shared__ double sX[3 * kBlock];
    __shared__ double red[64];
    const int t = threadIdx.x, la = t / P, k = t - la * P;
    const int i = blockIdx.x * A + la;
    const bool act = la < A && i < N;
    const unsigned oi = act ? (unsigned)a.orig[i] : 0u;
    const unsigned long long step = a.ctl->step;
    const size_t vb = (size_t)i * 3 * P + k;
    const double sqrtP = sqrt((double)P);
    double yt[3] = {0.0, 0.0, 0.0}, x0[3] = {0.0, 0.0, 0.0}, vt[3] = {0.0, 0.0, 0.0};
    double ft[3] = {0.0, 0.0, 0.0}, cref[3] = {0.0, 0.0, 0.0}, mk[8];
    double im = 0.0, sg = 0.0, active = 0.0;
    if (act) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            yt[d] = a.yt[vb + d * P];
            vt[d] = a.v[vb + d * P];
            ft[d] = na.ft[vb + d * P];
            x0[d] = a.x[vb - k + d * P];
            if (k == 0) cref[d] = a.cref[i * 3 + d];
        }
        im = a.atoms[i * 4 + AT_INV_M];
        sg = a.atoms[i * 4 + AT_SIGMA];
        active = a.atoms[i * 4 + AT_ACTIVE];
#pragma unroll
        for (int q = 0; q < 8; ++q) mk[q] = a.modes[k * 8 + q];
    }
    stage_matrix(a.M, P * P, sM);
    // v_W per dimension (the isotropic one three times); BAOAB: v_W for the
    // second A(dt/2), after its O(dt) (noise alone, so every thread forms it;
    // the finalize forms the same value)
    double vw[3], vw2[3], z[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int d = 0; d < 3; ++d) vw[d] = vw2[d] = vw_of(na, a.ctl, d);
    if (!a.obabo && a.nvt) {
        double zw[3];
        baro_noise(na, step, 0, zw);
#pragma unroll
        for (int d = 0; d < 3; ++d) vw2[d] = baro_o(na, vw[d], na.aniso ? zw[d] : zw[0]);
        // the beads' one draw
        if (act) gauss3(a.seed, oi, (unsigned)k, step, z, 0u);
    }
    // The barostat's factors of each A, likewise while the reads are in flight
    // (the isotropic one's once), and the box's scaling over the step and since
    // the last list build.
    CentroidFlow fl[2][3];
    double bn[3], gb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const bool own = d == 0 || na.aniso;
        fl[0][d] = own ? centroid_flow(a.obabo ? na.dt : a.hdt, vw[d]) : fl[0][0];
        fl[1][d] = a.obabo ? fl[0][d] : (own ? centroid_flow(a.hdt, vw2[d]) : fl[1][0]);
        const double sd = a.obabo ? fl[0][d].e : fl[0][d].e * fl[1][d].e;
        bn[d] = a.ctl->box[d] * sd;
        gb[d] = bn[d] / a.ctl->box_build[d];
    }
    if (act) {
#pragma unroll
        for (int d = 0; d < 3; ++d) vt[d] += a.hdt * im * ft[d];
        // A: the centroid under the barostat, in absolute coordinates x~0 =
        // y~0 + sqrt(P) x_0; the other modes by the free ring-polymer flow,
        // A(dt/2) n_ times
        auto a_flow = [&](const CentroidFlow *f, int n_) {
            if (k == 0) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const double X = f[d].e * (yt[d] + sqrtP * x0[d]) + f[d].s * vt[d];
                    vt[d] *= f[d].ei;
                    yt[d] = X - sqrtP * x0[d];
                }
            } else {
                for (int rep = 0; rep < n_; ++rep) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        const double q = yt[d], p = vt[d];
                        yt[d] = mk[MD_A00] * q + mk[MD_A01] * p;
                        vt[d] = mk[MD_A10] * q + mk[MD_A11] * p;
                    }
                }
            }
        };
        if (a.obabo) {
            a_flow(fl[0], 2);
        } else {
            // A(dt/2), O(dt) on the beads, A(dt/2)
            a_flow(fl[0], 1);
            if (a.nvt) {
#pragma unroll
                for (int d = 0; d < 3; ++d) vt[d] = mk[MD_C1] * vt[d] + mk[MD_C2] * sg * z[d];
            }
            a_flow(fl[1], 1);
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            a.v[vb + d * P] = vt[d];
            sX[(la * 3 + d) * P + k] = yt[d];
            // (the centroid mode is re-referenced to the new bead 0 below)
            if (k != 0) a.yt[vb + d * P] = yt[d];
        }
    }
    __syncthreads();
    double m3[3] = {0.0, 0.0, 0.0};   // dmax^2, emax^2, non-finite
    if (act) {
        // bead j = k: x_j = x_0 + sum_m M[m][j] y~_m
        const double *yr = sX + la * 3 * P;
        double xj[3];
        mode_sums(a.M, sM, P, k, yr, xj);
        if (k == 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) a.yt[vb + d * P] = yr[d * P] - sqrtP * xj[d];
        }
        double c[3], e2 = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            xj[d] += x0[d];
            a.x[vb + d * P] = xj[d];
            c[d] = x0[d] + yr[d * P] / sqrtP;
            const double dd = xj[d] - c[d];
            e2 += dd * dd;
            if (!isfinite(xj[d])) m3[2] = 1.0;
        }
        if (active != 0.0) m3[1] = e2;
        if (k == 0) {
            // displacement from the last build's centroid carried along by the
            // box scaling (per dimension) since that build
            double d2 = 0.0;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                a.cent[i * 3 + d] = c[d];
                const double dd = c[d] - gb[d] * cref[d];
                d2 += dd * dd;
            }
            if (active != 0.0) m3[0] = d2;
            if (a.ncell > 0 && i < a.n_active) {
                // the centroid's cell in the box after this step's scaling
                double icw[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) icw[d] = (double)a.nc[d] / bn[d];
                (void)cell_of_in(a, i, c, bn, icw);
            }
        }
    }
    const double r = block_fold<3, true>(m3, red);
    if (t < 3) na.part[(size_t)blockIdx.x * kNptMax + t] = r;
}

// Pass B's finalize (one block): the box follows v_W, the step counter
// advances, and the neighbor lists are rebuilt when a bead pair inside rc
// may be missing: with g the box's scaling since the build, a pair's
// centroid distance then was at most (rc + 2 E + 2 dmax) / g, which must not
// exceed the lists' cutoff.
__global__ __launch_bounds__(kBlock) void k_npt_fin_b(NptArgs na, int nblocks)
{
    const FusedArgs &a = na.f;
    Ctl *c = a.ctl;
    __shared__ double red[64];
    __shared__ __align__(16) int sbuf[4 * kMaxCells];
    __shared__ int sflag[1];
    __shared__ double s_dec[5];   // rebuild flag, r_list, new box
    const int t = threadIdx.x;
    double m3[3] = {0.0, 0.0, 0.0};
    for (int b = t; b < nblocks; b += kBlock) {
#pragma unroll
        for (int q = 0; q < 3; ++q) m3[q] = fmax(m3[q], na.part[(size_t)b * kNptMax + q]);
    }
    // the new box and v_W, while the partials are read
    const unsigned long long step = c->step, n_rebuilds = c->n_rebuilds;
    const double rlist0 = c->rlist;
    double bx[3], bb[3], vwn[3], vw0[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        bx[d] = c->box[d];
        bb[d] = c->box_build[d];
        vwn[d] = vw0[d] = vw_of(na, c, d);
    }
    if (!a.obabo && a.nvt) {
        double z[3];
        baro_noise(na, step, 0, z);
#pragma unroll
        for (int d = 0; d < 3; ++d) vwn[d] = baro_o(na, vw0[d], na.aniso ? z[d] : z[0]);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        // (BAOAB: the two A(dt/2), around v_W's O(dt))
        if (a.obabo)
            bx[d] *= exp(na.dt * vw0[d]);
        else
            bx[d] = bx[d] * exp(a.hdt * vw0[d]) * exp(a.hdt * vwn[d]);
    }
    const double x = block_fold<3, true>(m3, red);
    if (t < 64) {
        const double dmax = sqrt(read_lane(x, 0)), emax = sqrt(read_lane(x, 1)), bad = read_lane(x, 2);
        // the smallest scaling of any dimension since the build bounds a
        // pair's distance then by its distance now over g
        double g = bx[0] / bb[0];
        if (na.aniso) {
#pragma unroll
            for (int d = 1; d < 3; ++d) g = fmin(g, bx[d] / bb[d]);
        }
        const bool rebuild = a.rc + 2.0 * (emax + dmax) > g * rlist0;
        const double rl = a.rc + a.skin + 2.0 * emax;
        if (t == 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) c->box[d] = bx[d];
            if (!a.obabo) {
                if (na.aniso) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) c->vwa[d] = vwn[d];
                } else {
                    c->vw = vwn[0];
                }
            }
            c->step = step + 1;
            c->synced = 0;
            if (c->budget > 0) c->budget = c->budget - 1;
            if (rebuild) {
                c->rebuild = 1;
                c->ebuild = emax;
                c->rlist = rl;
                c->n_rebuilds = n_rebuilds + 1;
#pragma unroll
                for (int d = 0; d < 3; ++d) c->box_build[d] = bx[d];
            } else {
                c->rebuild = 0;
            }
            if (bad != 0.0) c->nonfinite = 1;
            c->ran = 1;
            s_dec[0] = rebuild ? 1.0 : 0.0;
            s_dec[1] = rl;
#pragma unroll
            for (int d = 0; d < 3; ++d) s_dec[2 + d] = bx[d];
        }
    }
    // the centroid cell lists of a rebuild, binned in the new box by pass B
    if (a.ncell > 0) {
        __syncthreads();
        if (s_dec[0] != 0.0) {
            double icw[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) icw[d] = (double)a.nc[d] / s_dec[2 + d];
            cells_finalize(a, icw, s_dec[1], sbuf, sflag);
        }
    }
}

__global__ void k_npt_init(Ctl *c, double b0, double b1, double b2, double vw, double vx,
                           double vy, double vz)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        c->box[0] = c->box_build[0] = b0;
        c->box[1] = c->box_build[1] = b1;
        c->box[2] = c->box_build[2] = b2;
        c->vw = vw;
        c->vwa[0] = vx;
        c->vwa[1] = vy;
        c->vwa[2] = vz;
        c->volume = b0 * b1 * b2;
        c->ebaro = 0.0;
        c->enthalpy = 0.0;
    }
}

void launch_npt_init(Ctl *ctl, const double box[3], const double vw[3], hipStream_t s)
{
    hipLaunchKernelGGL(k_npt_init, dim3(1), dim3(64), 0, s, ctl, box[0], box[1], box[2], vw[0], vw[0],
                       vw[1], vw[2]);
}

void launch_npt_a(const NptArgs &a, int mode, hipStream_t s)
{
    const int grid = npt_grid(a.f.N, a.f.P);
    hipLaunchKernelGGL(a.aniso ? k_npt_a<true> : k_npt_a<false>, dim3(grid), dim3(kBlock), 0, s, a, mode);
    hipLaunchKernelGGL(a.aniso ? k_npt_fin_a<true> : k_npt_fin_a<false>, dim3(1), dim3(kBlock), 0, s, a, mode,
                       grid);
}

void launch_npt_b(const NptArgs &a, hipStream_t s)
{
    const int grid = npt_grid(a.f.N, a.f.P);
    hipLaunchKernelGGL(k_npt_b, dim3(grid), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_npt_fin_b, dim3(1), dim3(kBlock), 0, s, a, grid);
}

}  // namespace pimd

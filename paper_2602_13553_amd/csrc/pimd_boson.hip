// Bosonic exchange springs (the bosonic fix of Sec. III.C; the recursion of
// Hirshberg et al. 2019, evaluated in O(N^2) like Feldman and Hirshberg's
// algorithm, both cited by the paper).
//
// N identical particles of P beads.  The springs inside each particle's ring
// (bead j to j+1, j < P-1) are those of distinguishable particles; the link
// from bead P-1 of particle l to bead 0 of particle l' is summed over exchange
// cycles by the recursion over the cycle that holds the last particle,
//   exp(-beta_n V[n]) = (1/n) sum_{k=1..n} exp(-beta_n (E[n,k] + V[n-k])),
// E[n,k] the single ring through particles n-k..n-1 (0-based), V[0] = 0.
//
// Every term of V[n] holds the inner-ring energies of all of particles
// 0..n-1 once, so V[n] = sum_{l<n} eint[l] + V'[n], with V' the same
// recursion over the links alone (E'[n,k]: chain links n-k..n-2 plus the
// closing link n-1 -> n-k).  The kernels run V' and add the inner energies
// at the end, so no ring weight sees them.  The chain sums are differences of
// double-double prefix sums and V' is carried in double-double, so each
// weight's exponent E' + V'[n-k] - V'[n] is formed to the rounding of its
// own size, not of V_B's.
//
// The recursion is a lower triangular linear system in Z[n] = exp(-beta_n V'[n]),
//   Z[n] = (1/n) sum_j exp(-beta_n E'[n, n-j]) Z[j],   Z[0] = 1,
// whose matrix is known up front.  With c[m] the chain links' prefix sums and
// Y[n] = exp(beta_n c[n]) Z[n] its entries need one link each,
//   Y[n] = (1/n) exp(beta_n L[n-1,n]) sum_j exp(-beta_n L[n-1,j]) Y[j],
// so the whole chip forms them first and one block then solves the system by
// blocks of 64: multiply-adds along the serial chain, no exponential, no
// logarithm and no reduction across lanes.  Y spans thousands of binary
// orders, so entries and Y are (mantissa, exponent) pairs.
//
//   k_boson_prep  : inner-ring spring forces (sets f) and energies; the
//                   system's matrix in tiles; the chain links' prefix sums
//   k_boson_solve : one block: Y and V'[N]
//   k_boson_weights: a block per tile: the ring weights w[n,k] and the rows'
//                   weighted ring energies
//   k_boson_adjoint: one block: adj[n] = dV'[N]/dV'[n] by blocks of 64 from
//                   the end; V_B and EV_B
//   k_boson_rows  : a wave per n: q[n,k] = adj[n] w[n,k] (the probability of
//                   ring (n,k)'s closing link), its running sums over the
//                   columns, and the closing links' forces on the last bead
//   k_boson_cols  : 16 lanes per particle group: the chain links'
//                   probabilities (column sums of those running sums) and
//                   the remaining link forces
// Links beyond kWideLink (in units of 1/beta_n), where the exponents would
// leave 32 bits, and non-finite ones send the call through the recursion in
// log space (seq_recursion: one block of k_boson_weights, sequential in n); so
// do up to kBosonFew particles, without the solve's and the adjoint's launches.
#include "../../include/pimd.h"
#include "pimd_internal.h"
#include "pimd_device.h"

#include <cmath>
#include <mutex>

namespace pimd {

// The allocation-free entry point's scratch (pimd_boson_spring_noalloc): one
// copy per device, 2.4 MB, held until the process ends.  Host code reaches it
// only through the per-device address from hipGetSymbolAddress (in host code
// the array's name is a host-side stand-in, not a device address).
constexpr int kBosonNoAllocMaxN = 512;
static __device__ __align__(256) double scratch[boson_scr_doubles(kBosonNoAllocMaxN)];

namespace {

constexpr int kSeq = 256;   // threads of the recursion in log space
constexpr int kSeqU = (kBosonMaxN + kSeq - 1) / kSeq;   // k per thread and stage
constexpr int kSolve = 1024;   // threads of the blocked solves
constexpr int kSolveWaves = kSolve / 64;
constexpr int kT = kBosonTile;
constexpr int kTT = kT * kT;

// beta_n times a link's energy, at most, in the blocked solve: exponents up to
// 2^18 per factor stay below 2^29 through 1024 particles' products
constexpr double kWideLink = 131072.0;
constexpr int kNoExp = -(1 << 30);   // exponent of an exact zero

// Scratch (see pimd_internal.h)
struct BosonScr {
    // Tiles are laid out for 16 bytes per lane and load: a CU takes a wave's
    // load every 17 cycles whether its lanes load 4, 8 or 16 bytes.
    double *w;      // [tiles][32 row pairs][64 columns j][2 rows n] ring weights;
                    // first [tiles][32 column pairs][64 rows][2] mantissas of
                    // the matrix
    double *s;      // like w: running probabilities over j
    int *ge;        // [tiles][16][64 rows][4 columns] exponents (in s's place)
    double *ym;     // [N+1] Y: mantissa in [0.5, 1), exponent
    int *ye;
    double *xm;     // [N+1] exp(beta_n L[n-1,n]) (1 for n = N), likewise
    int *xe;
    double *chi, *clo;   // [N+1] prefix sums of the chain links (double-double)
    double *adj;    // [N+1]
    double *e0, *el;     // [N][3] the particles' first and last beads
    double *eb;     // [tiles][64] the tiles' shares of sum_k w[n,k] E'[n,k]
    double *ein;    // [kBosonInnerMax] inner spring energies per block
    double *vp;     // [2] V'[N] (double-double)
    int *wide;      // [tiles] 1: a link of the tile is beyond kWideLink
    int *slow;      // [1] 1: this call went through seq_recursion

    __device__ explicit BosonScr(const BosonArgs &a)
    {
        const int N = a.N;
        const size_t tri = boson_scr_tri(N), n1 = (size_t)N + 1;
        w = a.scr;
        s = w + tri;
        ge = reinterpret_cast<int *>(s);
        ym = s + tri;
        ye = reinterpret_cast<int *>(ym + n1);
        xm = ym + 2 * n1;
        xe = reinterpret_cast<int *>(ym + 3 * n1);
        chi = ym + 4 * n1;
        clo = ym + 5 * n1;
        adj = ym + 6 * n1;
        e0 = ym + 7 * n1;
        el = ym + 10 * n1;
        eb = ym + 13 * n1;
        ein = eb + (size_t)boson_tiles(N) * kT;
        vp = ein + kBosonInnerMax;
        wide = reinterpret_cast<int *>(vp + 2);
        slow = reinterpret_cast<int *>(vp + 2 + boson_tiles(N));
    }
};

// place of w[n, n-j] in the tiles
__device__ __forceinline__ size_t w_at(int n, int j)
{
    const int b = (n - 1) / kT, r = (n - 1) - b * kT, cb = j / kT;
    return (size_t)boson_tile(b, cb) * kTT + ((r >> 1) * kT + (j - cb * kT)) * 2 + (r & 1);
}

__device__ __forceinline__ size_t bidx(const BosonArgs &a, int j, int l, int d)
{
    return a.layout ? ((size_t)l * 3 + d) * a.P + j : ((size_t)j * a.N + l) * 3 + d;
}

// a - b under the minimum image in each periodic dimension
__device__ __forceinline__ double mic(double a, double b, double L)
{
    const double u = a - b;
    return L > 0.0 ? u - L * rint(u / L) : u;
}

// --- double-double arithmetic (error-free sums; no products involved) ---
struct DD {
    double hi, lo;
};

__device__ __forceinline__ DD two_sum(double a, double b)
{
    const double s = a + b;
    const double bb = s - a;
    return {s, (a - (s - bb)) + (b - bb)};
}

__device__ __forceinline__ DD dd_add(DD a, DD b)
{
    const DD s = two_sum(a.hi, b.hi);
    const double lo = s.lo + (a.lo + b.lo);
    const double hi = s.hi + lo;
    return {hi, lo - (hi - s.hi)};
}

__device__ __forceinline__ DD dd_add1(DD a, double b)
{
    const DD s = two_sum(a.hi, b);
    const double lo = s.lo + a.lo;
    const double hi = s.hi + lo;
    return {hi, lo - (hi - s.hi)};
}

// a - b, rounded once (to the rounding of the difference's own size)
__device__ __forceinline__ double dd_diff(DD a, DD b)
{
    const DD s = two_sum(a.hi, -b.hi);
    return s.hi + (s.lo + (a.lo - b.lo));
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}

// Block reductions of the recursion in log space (kSeq threads); every thread
// gets the result.  The waves' values are combined in wave order.  One barrier
// each: the minimum and the sums take turns and have slots of their own in red,
// so a slot is written again only after the other reduction's barrier, which
// every thread reaches past its reads.  (With two barriers each: links beyond the
// blocked solve at N = 512 1197 us a call, now 1149.)
constexpr int kSeqWaves = kSeq / 64;
__device__ __forceinline__ double seq_min(double v, double *red)
{
    v = wave_min(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = red[0];
#pragma unroll
    for (int u = 1; u < kSeqWaves; ++u) r = fmin(r, red[u]);
    return r;
}

__device__ __forceinline__ void seq_sum2(double &a, double &b, double *red)
{
    double *ra = red + kSeqWaves, *rb = ra + kSeqWaves;
    a = wave_sum(a);
    b = wave_sum(b);
    if ((threadIdx.x & 63) == 0) {
        ra[threadIdx.x >> 6] = a;
        rb[threadIdx.x >> 6] = b;
    }
    __syncthreads();
    a = ra[0];
    b = rb[0];
#pragma unroll
    for (int u = 1; u < kSeqWaves; ++u) {
        a += ra[u];
        b += rb[u];
    }
}

struct SeqLds {
    double e0[kBosonMaxN * 3];      // bead 0 of each particle
    double el[kBosonMaxN * 3];      // bead P-1
    double chi[kBosonMaxN + 1];     // prefix sums of the chain links l -> l+1 (double-double)
    double clo[kBosonMaxN + 1];
    double vhi[kBosonMaxN + 1];     // V' (double-double)
    double vlo[kBosonMaxN + 1];
    double ev[kBosonMaxN + 1];      // EV'
    double adj[kBosonMaxN + 1];     // dV'[N]/dV'[n]
    double red[16];
};

// Blocks of the inner springs (four bead coordinates per thread).
__host__ __device__ inline int inner_blocks(int N, int P)
{
    const int nb = (int)(((long long)N * 3 * P + 4 * kBlock - 1) / (4 * kBlock));
    return nb < kBosonInnerMax ? nb : kBosonInnerMax;
}

// this thread's share of the inner spring energies' sum
__device__ __forceinline__ double inner_sum(const BosonArgs &a, const BosonScr &scr, int t)
{
    return t < inner_blocks(a.N, a.P) ? scr.ein[t] : 0.0;
}

__device__ __forceinline__ double link_e(const SeqLds &s, const BosonArgs &a, int l, int l2)
{
    double e = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double u = mic(s.e0[l2 * 3 + d], s.el[l * 3 + d], a.box[d]);
        e += u * u;
    }
    return a.ks * e;
}

// The recursion in log space, sequential in n, parallel in k: V', the ring
// weights, EV' and the adjoints, for the calls that the blocked solve does not
// take.  One block.
__device__ __forceinline__ void seq_recursion(const BosonArgs &a, SeqLds &s)
{
    const int t = threadIdx.x, N = a.N;
    const BosonScr scr(a);
    double *w = scr.w;                               // ring weights w[n,k]
    for (int e = t; e < N * 3; e += kSeq) {
        s.e0[e] = scr.e0[e];
        s.el[e] = scr.el[e];
    }
    for (int m = t; m < N; m += kSeq) {
        s.chi[m] = scr.chi[m];
        s.clo[m] = scr.clo[m];
    }
    // the inner energies' sum, thread-strided, then in wave order
    double esum = inner_sum(a, scr, t);
    {
        double dummy = 0.0;
        seq_sum2(esum, dummy, s.red);   // (its barrier also publishes e0, el)
    }
    if (t == 0) {
        s.vhi[0] = 0.0;
        s.vlo[0] = 0.0;
        s.ev[0] = 0.0;
    }
    __syncthreads();

    // Forward: V'[n] = V'[n-1] + delta_n, delta_n a soft minimum of
    // b_k = E'[n,k] + V'[n-k] - V'[n-1] (all small), stabilized by the
    // minimum; w[n,k] = exp(-beta_n (b_k - delta_n)) / n.  Thread t takes
    // k = 1 + t + u kSeq.  V'[n-1] is in every thread's registers; V'[m] for
    // m < n-1 was written by thread 0 before at least one barrier.
    DD vprev = {0.0, 0.0};
    const double bn = a.bn;
    for (int n = 1; n <= N; ++n) {
        const DD chn = {s.chi[n - 1], s.clo[n - 1]};
        double b[kSeqU], E[kSeqU];
        double mloc = INFINITY;
#pragma unroll
        for (int u = 0; u < kSeqU; ++u) {
            const int k = 1 + t + u * kSeq;
            b[u] = INFINITY;
            E[u] = 0.0;
            if (k <= n) {
                const int j = n - k;
                const double c = dd_diff(chn, {s.chi[j], s.clo[j]});
                E[u] = c + link_e(s, a, n - 1, j);
                const double dv = (k == 1) ? 0.0 : dd_diff({s.vhi[j], s.vlo[j]}, vprev);
                b[u] = E[u] + dv;
                mloc = fmin(mloc, b[u]);
            }
        }
        const double m = seq_min(mloc, s.red);
        double sw = 0.0, st = 0.0;
        double ex[kSeqU];
#pragma unroll
        for (int u = 0; u < kSeqU; ++u) {
            const int k = 1 + t + u * kSeq;
            ex[u] = 0.0;
            if (k <= n) {
                ex[u] = exp(-bn * (b[u] - m));
                sw += ex[u];
                st += ex[u] * (E[u] + s.ev[n - k]);
            }
        }
        seq_sum2(sw, st, s.red);
        const double delta = m - log(sw / (double)n) / bn;
        vprev = dd_add1(vprev, delta);
        const double isw = 1.0 / sw;
#pragma unroll
        for (int u = 0; u < kSeqU; ++u) {
            const int k = 1 + t + u * kSeq;
            if (k <= n) w[w_at(n, n - k)] = ex[u] * isw;
        }
        if (t == 0) {
            s.vhi[n] = vprev.hi;
            s.vlo[n] = vprev.lo;
            s.ev[n] = st * isw;
        }
    }
    // Adjoints: adj[N] = 1, adj[n-k] += adj[n] w[n,k] for n = N..1 (the
    // targets of one n are distinct); a barrier per n makes adj[n] final.
    for (int e = t; e <= N; e += kSeq) s.adj[e] = (e == N) ? 1.0 : 0.0;
    for (int n = N; n >= 1; --n) {
        double wr[kSeqU];
#pragma unroll
        for (int u = 0; u < kSeqU; ++u) {
            const int k = 1 + t + u * kSeq;
            wr[u] = (k <= n) ? w[w_at(n, n - k)] : 0.0;
        }
        __syncthreads();
        const double an = s.adj[n];
#pragma unroll
        for (int u = 0; u < kSeqU; ++u) {
            const int k = 1 + t + u * kSeq;
            if (k <= n) s.adj[n - k] += an * wr[u];
        }
    }
    __syncthreads();
    for (int e = t; e <= N; e += kSeq) scr.adj[e] = s.adj[e];
    if (t == 0) {
        const DD vb = dd_add1({s.vhi[N], s.vlo[N]}, esum);
        a.res[0] = vb.hi + vb.lo;
        a.res[1] = esum + s.ev[N];
    }
}

// --- the blocked solve -------------------------------------------------------
// (mantissa, exponent) += (tm, te); mantissas are >= 0, and exact zeros carry
// kNoExp.  The sum keeps the larger exponent, unnormalized: within a block of
// 64 additions and products mantissas stay within 2^(+-500).
__device__ __forceinline__ void ext_add(double &am, int &ae, double tm, int te)
{
    const int e = max(ae, te);
    am = ldexp(am, ae - e) + ldexp(tm, te - e);
    ae = e;
}

// exp(p + plo) = m 2^k, m in about [0.7, 1.42), for |p| <= kWideLink: p - k ln 2
// exactly through ln 2's high part (k ln 2_hi has at most 59 bits, the
// difference at most 53), then the Taylor series to r^13 (|r| <= 0.347, next
// term below 2^-57).
__device__ __forceinline__ void exp_ext(double p, double plo, double &m, int &k)
{
    const double LN2_HI = 0x1.62e42fefa2p-1, LN2_LO = 0x1.9ef35793c7673p-41;
    const double kd = rint(p * 1.4426950408889634074);
    double r = fma(-kd, LN2_HI, p);
    r += fma(-kd, LN2_LO, plo);
    double q = 1.0 / 6227020800.0;
    q = fma(q, r, 1.0 / 479001600.0);
    q = fma(q, r, 1.0 / 39916800.0);
    q = fma(q, r, 1.0 / 3628800.0);
    q = fma(q, r, 1.0 / 362880.0);
    q = fma(q, r, 1.0 / 40320.0);
    q = fma(q, r, 1.0 / 5040.0);
    q = fma(q, r, 1.0 / 720.0);
    q = fma(q, r, 1.0 / 120.0);
    q = fma(q, r, 1.0 / 24.0);
    q = fma(q, r, 1.0 / 6.0);
    q = fma(q, r, 0.5);
    m = fma(r * r, q, r) + 1.0;
    k = (int)kd;
}

__device__ __forceinline__ double link3(const BosonArgs &a, const double *el, const double *e0)
{
    double e = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double u = mic(e0[d], el[d], a.box[d]);
        e += u * u;
    }
    return a.ks * e;
}

// Blocks 0..tiles-1: the matrix exp(beta_n (L[n-1,n] - L[n-1,j])) / n, one
// 64 x 64 tile each (columns in order, a row per lane: as the solve reads it).  Then the inner springs (forces on every bead, overwriting
// f, elementwise so that either layout is read in order; one partial energy per
// block).  The last block: the particles' end beads, packed, and the chain
// links' prefix sums.  13 us at N = 1024, P = 32 (the inner springs alone took
// 38 us with a thread per particle, whose reads are a bead row apart), bound
// by the tiles' exponentials and the launch.
__global__ __launch_bounds__(kBlock) void k_boson_prep(BosonArgs a)
{
    __shared__ double sh[2 * kBlock];
    const int t = threadIdx.x, N = a.N, P = a.P;
    const BosonScr scr(a);
    const int tiles = boson_tiles(N), inner = inner_blocks(N, P);
    if ((int)blockIdx.x < tiles) {
        if (N <= kBosonFew) return;
        const int tile = blockIdx.x;
        int b = (int)((sqrtf(8.0f * (float)tile + 1.0f) - 1.0f) * 0.5f);
        while (boson_tile(b + 1, 0) <= tile) ++b;
        while (boson_tile(b, 0) > tile) --b;
        const int cb = tile - boson_tile(b, 0);
        const int r = t & 63, n = b * kT + 1 + r;
        if (t < 3 * kT) {
            const int j = cb * kT + t / 3;
            sh[t] = j < N ? a.x[bidx(a, 0, j, t % 3)] : 0.0;
        }
        // the row's particle n-1: its last bead, and the chain link to n
        double el[3] = {0.0, 0.0, 0.0}, xm = 1.0;
        int xe = 0;
        bool bad = false;
        if (n <= N) {
            double e0n[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                el[d] = a.x[bidx(a, P - 1, n - 1, d)];
                if (n < N) e0n[d] = a.x[bidx(a, 0, n, d)];
            }
            if (n < N) {
                const double L = link3(a, el, e0n), p = a.bn * L;
                bad = !(p <= kWideLink);
                if (!bad) exp_ext(p, fma(a.bn, L, -p), xm, xe);
            }
            if (cb == b && t < kT) {
                scr.xm[n] = xm;
                scr.xe[n] = xe;
            }
        }
        const double hm = xm / (double)n;
        __syncthreads();
        double2 *gm = reinterpret_cast<double2 *>(scr.w + (size_t)tile * kTT);
        int4 *ge = reinterpret_cast<int4 *>(scr.ge + (size_t)tile * kTT);
        for (int q = t >> 6; q < kT / 4; q += kBlock / 64) {
            double m[4];
            int e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = 4 * q + u, j = cb * kT + c;
                m[u] = 0.0;
                e[u] = kNoExp;
                if (n <= N && j < n) {
                    const double L = link3(a, el, sh + 3 * c), p = a.bn * L;
                    if (p <= kWideLink) {
                        int k;
                        exp_ext(-p, -fma(a.bn, L, -p), m[u], k);
                        m[u] *= hm;
                        e[u] = k + xe + __builtin_amdgcn_frexp_exp(m[u]);
                        m[u] = __builtin_amdgcn_frexp_mant(m[u]);
                    } else {
                        bad = true;
                    }
                }
            }
            gm[(2 * q) * kT + r] = make_double2(m[0], m[1]);
            gm[(2 * q + 1) * kT + r] = make_double2(m[2], m[3]);
            ge[q * kT + r] = make_int4(e[0], e[1], e[2], e[3]);
        }
        const int any = __syncthreads_or(bad ? 1 : 0);
        if (t == 0) scr.wide[tile] = any;
        return;
    }
    if ((int)blockIdx.x < tiles + inner) {
        const int ib = blockIdx.x - tiles;
        const size_t n3p = (size_t)N * 3 * P, stride = a.layout ? 1 : (size_t)N * 3;
        const double k2 = 2.0 * a.ks;
        double e2 = 0.0;
        for (size_t e = (size_t)ib * kBlock + t; e < n3p; e += (size_t)inner * kBlock) {
            const int j = a.layout ? (int)(e % P) : (int)(e / stride);
            const double cur = a.x[e];
            const double next = j + 1 < P ? a.x[e + stride] : 0.0;
            const double prev = j > 0 ? a.x[e - stride] : 0.0;
            double g = 0.0;
            if (j + 1 < P) {
                const double u = next - cur;
                g += k2 * u;
                e2 += u * u;
            }
            if (j > 0) g -= k2 * (cur - prev);
            a.f[e] = g;
        }
        double s1[1] = {e2};
        const double r = block_fold<1>(s1, sh);
        if (t == 0) scr.ein[ib] = a.ks * r;
        return;
    }
    // end beads, and the prefix sums ch[m] = sum_{l<m} link(l, l+1), m = 0..N-1,
    // in double-double: each thread sums a contiguous chunk, the chunk totals
    // are scanned in the waves and across them, then each chunk is written out
    for (int e = t; e < N * 3; e += kBlock) {
        const int l = e / 3, d = e - l * 3;
        scr.e0[e] = a.x[bidx(a, 0, l, d)];
        scr.el[e] = a.x[bidx(a, P - 1, l, d)];
    }
    constexpr int CU = (kBosonMaxN + kBlock - 1) / kBlock;
    const int nl = N - 1;                            // chain links
    const int C = (nl + kBlock - 1) / kBlock;
    const int l0 = t * C;
    double L[CU];
    DD tot = {0.0, 0.0};
#pragma unroll
    for (int u = 0; u < CU; ++u) {
        const int l = l0 + u;
        L[u] = 0.0;
        if (u < C && l < nl) {
            double el[3], e0[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                el[d] = a.x[bidx(a, P - 1, l, d)];
                e0[d] = a.x[bidx(a, 0, l + 1, d)];
            }
            L[u] = link3(a, el, e0);
            tot = dd_add1(tot, L[u]);
        }
    }
    const int lane = t & 63, w = t >> 6;
    DD inc = tot;                                    // scan of the wave's chunk totals
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const DD v = {__shfl_up(inc.hi, off), __shfl_up(inc.lo, off)};
        if (lane >= off) inc = dd_add(v, inc);
    }
    if (lane == 63) {
        sh[2 * w] = inc.hi;
        sh[2 * w + 1] = inc.lo;
    }
    __syncthreads();
    DD run = {0.0, 0.0};                             // everything before this thread's chunk
    for (int u = 0; u < w; ++u) run = dd_add(run, {sh[2 * u], sh[2 * u + 1]});
    const DD ex = {__shfl_up(inc.hi, 1), __shfl_up(inc.lo, 1)};
    if (lane > 0) run = dd_add(run, ex);
    if (t == 0) {
        scr.chi[0] = 0.0;
        scr.clo[0] = 0.0;
    }
#pragma unroll
    for (int u = 0; u < CU; ++u) {
        const int l = l0 + u;
        if (u < C && l < nl) {
            run = dd_add1(run, L[u]);
            scr.chi[l + 1] = run.hi;
            scr.clo[l + 1] = run.lo;
        }
    }
}

__device__ __forceinline__ double lane_of(double v, int lane)
{
    union { double d; int i[2]; } u;
    u.d = v;
    u.i[0] = __builtin_amdgcn_readlane(u.i[0], lane);
    u.i[1] = __builtin_amdgcn_readlane(u.i[1], lane);
    return u.d;
}

struct SolveLds {
    double2 gm[2][kTT / 2];         // the current and the next diagonal tile
    int4 ge[2][kTT / 4];
    double ym[kBosonMaxN + 1];      // Y
    int ye[kBosonMaxN + 1];
    double pm[kSolveWaves][kT];     // the waves' sums over the columns before the block
    int pe[kSolveWaves][kT];
};

// four columns of a tile for one row (lane): mantissas and exponents
struct Quad {
    double2 a, b;
    int4 e;
};
__device__ __forceinline__ Quad quad_at(const double2 *gm, const int4 *ge, int q, int lane)
{
    return {gm[2 * q * kT + lane], gm[(2 * q + 1) * kT + lane], ge[q * kT + lane]};
}
// += those columns times Y
__device__ __forceinline__ void quad_add(double &am, int &ae, const Quad &g, const double *ym,
                                         const int *ye)
{
    ext_add(am, ae, g.a.x * ym[0], g.e.x + ye[0]);
    ext_add(am, ae, g.a.y * ym[1], g.e.y + ye[1]);
    ext_add(am, ae, g.b.x * ym[2], g.e.z + ye[2]);
    ext_add(am, ae, g.b.y * ym[3], g.e.w + ye[3]);
}

// The triangular system, one block, by blocks of 64 rows.  Wave 0 solves the
// diagonal tile: lane r holds row r's sum, and step c broadcasts the Y that
// lane c-1 has just finished, so a step is one broadcast and one multiply-add
// of (mantissa, exponent) deep (87 cycles, 2.3 us per block).  Meanwhile waves
// 1..15 sum the next block's rows over the columns known so far, and once the
// tile is solved every wave adds four of its 64 columns, fetched ahead.  Bound
// by the diagonal tiles' chain and, at large N, by one CU's reads of the matrix
// (12 B per entry; one CU reads 107 GB/s from beyond its L2, half of that with
// 8-byte lanes).  88 us at N = 1024, 35 us at N = 512; with 8- and 4-byte lanes
// 127 and 45 us, and the recursion in log space, adjoint included, 2683 and
// 1125 us.
__global__ __launch_bounds__(kSolve) void k_boson_solve(BosonArgs a)
{
    __shared__ SolveLds s;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, N = a.N;
    const BosonScr scr(a);
    const int nb = boson_blocks(N), tiles = boson_tiles(N);
    const double2 *gmat = reinterpret_cast<const double2 *>(scr.w);
    const int4 *gexp = reinterpret_cast<const int4 *>(scr.ge);
    const double2 dm0 = gmat[t], dm1 = gmat[t + kSolve];
    const int4 de0 = gexp[t];
    const int slow = __syncthreads_or(t < tiles ? scr.wide[t] : 0);
    static_assert(boson_tiles(kBosonMaxN) <= kSolve, "one flag per thread");
    if (t == 0) scr.slow[0] = slow ? 1 : 0;
    if (slow) return;                            // k_boson_weights runs seq_recursion
    constexpr int W = kSolveWaves - 1;           // waves that sum ahead
    static_assert(kT / 4 == kSolveWaves, "every wave takes four of a tile's columns");
    double am = 0.0;
    int ae = kNoExp;
    s.gm[0][t] = dm0;
    s.gm[0][t + kSolve] = dm1;
    s.ge[0][t] = de0;
    if (t == 0) {
        s.ym[0] = 0.5;
        s.ye[0] = 1;
        scr.ym[0] = 0.5;
        scr.ye[0] = 1;
    }
    __syncthreads();
    for (int b = 0; b < nb; ++b) {
        Quad last = {};                          // four of the columns [64 b, 64 b + 64) of block b+1
        const double2 *rm = gmat + (size_t)boson_tile(b + 1, 0) * (kTT / 2);
        const int4 *re = gexp + (size_t)boson_tile(b + 1, 0) * (kTT / 4);
        if (b + 1 < nb) last = quad_at(rm, re, b * (kT / 4) + w, lane);
        if (w == 0) {
            __builtin_amdgcn_s_setprio(3);
            const double2 *gm = s.gm[b & 1];
            const int4 *ge = s.ge[b & 1];
            double ym = s.ym[b * kT];
            int ye = s.ye[b * kT];
            Quad g = quad_at(gm, ge, 0, lane);
#pragma unroll 2
            for (int q = 0; q < kT / 4; ++q) {
                const Quad gn = quad_at(gm, ge, min(q + 1, kT / 4 - 1), lane);
                ext_add(am, ae, g.a.x * ym, g.e.x + ye);
                ext_add(am, ae, g.a.y * lane_of(am, 4 * q),
                        g.e.y + __builtin_amdgcn_readlane(ae, 4 * q));
                ext_add(am, ae, g.b.x * lane_of(am, 4 * q + 1),
                        g.e.z + __builtin_amdgcn_readlane(ae, 4 * q + 1));
                ext_add(am, ae, g.b.y * lane_of(am, 4 * q + 2),
                        g.e.w + __builtin_amdgcn_readlane(ae, 4 * q + 2));
                ym = lane_of(am, 4 * q + 3);
                ye = __builtin_amdgcn_readlane(ae, 4 * q + 3);
                g = gn;
            }
            __builtin_amdgcn_s_setprio(0);
            const int n = b * kT + 1 + lane;
            if (n <= N) {
                const double m = __builtin_amdgcn_frexp_mant(am);
                const int e = ae + __builtin_amdgcn_frexp_exp(am);
                s.ym[n] = m;
                s.ye[n] = e;
                scr.ym[n] = m;
                scr.ye[n] = e;
            }
            am = 0.0;
            ae = kNoExp;
        } else if (b + 1 < nb) {
            // the next diagonal tile in flight while the columns known so far
            // are summed (the next group's reads ahead of this group's sums)
            const double2 *dg = rm + (b + 1) * (kTT / 2);
            const int4 *dh = re + (b + 1) * (kTT / 4);
            constexpr int ND = (kTT / 2 + 64 * W - 1) / (64 * W), NE = (kTT / 4 + 64 * W - 1) / (64 * W);
            double2 dm[ND];
            int4 de[NE];
#pragma unroll
            for (int u = 0; u < ND; ++u) dm[u] = dg[min(t - 64 + u * 64 * W, kTT / 2 - 1)];
#pragma unroll
            for (int u = 0; u < NE; ++u) de[u] = dh[min(t - 64 + u * 64 * W, kTT / 4 - 1)];
            am = 0.0;
            ae = kNoExp;
            constexpr int U = 1;
            const int J = b * (kT / 4);           // groups of four columns before them
            Quad g[2][U];
            auto fetch = [&](int h, int j0) {
#pragma unroll
                for (int u = 0; u < U; ++u) g[h][u] = quad_at(rm, re, min(j0 + u * W, J - 1), lane);
            };
            auto add = [&](int h, int j0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = j0 + u * W;
                    if (j < J) quad_add(am, ae, g[h][u], s.ym + 4 * j, s.ye + 4 * j);
                }
            };
            if (w - 1 < J) fetch(0, w - 1);
#pragma unroll
            for (int u = 0; u < ND; ++u) {
                const int q = t - 64 + u * 64 * W;
                if (q < kTT / 2) s.gm[(b + 1) & 1][q] = dm[u];
            }
#pragma unroll
            for (int u = 0; u < NE; ++u) {
                const int q = t - 64 + u * 64 * W;
                if (q < kTT / 4) s.ge[(b + 1) & 1][q] = de[u];
            }
            for (int j0 = w - 1; j0 < J; j0 += 2 * W * U) {
                if (j0 + W * U < J) fetch(1, j0 + W * U);
                add(0, j0);
                if (j0 + 2 * W * U < J) fetch(0, j0 + 2 * W * U);
                if (j0 + W * U < J) add(1, j0 + W * U);
            }
        }
        __syncthreads();
        if (b + 1 == nb) break;
        quad_add(am, ae, last, s.ym + b * kT + 4 * w, s.ye + b * kT + 4 * w);
        s.pm[w][lane] = am;
        s.pe[w][lane] = ae;
        __syncthreads();
        if (w == 0) {
            int e = kNoExp;
#pragma unroll
            for (int u = 0; u < kSolveWaves; ++u) e = max(e, s.pe[u][lane]);
            am = 0.0;
#pragma unroll
            for (int u = 0; u < kSolveWaves; ++u) am += ldexp(s.pm[u][lane], s.pe[u][lane] - e);
            ae = e;
        }
    }
    // V'[N] = -(1/beta_n) sum_n ln(Z[n]/Z[n-1]), Z[n]/Z[n-1] = Y[n] /
    // (exp(beta_n L[n-1,n]) Y[n-1]): each term of V'[n] - V'[n-1]'s own size,
    // summed in double-double
    DD v = {0.0, 0.0};
    if (t < N) {
        const int n = t + 1;
        const double LN2_HI = 0x1.62e42fefa2p-1, LN2_LO = 0x1.9ef35793c7673p-41;
        const double m = s.ym[n] / (scr.xm[n] * s.ym[n - 1]);
        const double e = (double)(s.ye[n] - scr.xe[n] - s.ye[n - 1]);
        v.hi = -fma(e, LN2_HI, fma(e, LN2_LO, log(m))) / a.bn;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = dd_add(v, {__shfl_xor(v.hi, o), __shfl_xor(v.lo, o)});
    if (lane == 0) {
        s.pm[w][0] = v.hi;
        s.pm[w][1] = v.lo;
    }
    __syncthreads();
    if (t == 0) {
        for (int u = 1; u < kSolveWaves; ++u) v = dd_add(v, {s.pm[u][0], s.pm[u][1]});
        scr.vp[0] = v.hi;
        scr.vp[1] = v.lo;
    }
}

struct WeightLds {
    double w[kT * (kT + 1)];
    double e0[3 * kT];              // the columns' first beads, Y and chain sums
    double ym[kT];
    double ch[2 * kT];
    int ye[kT];
};

// Ring weights of one tile, w[n,k] = G[n,j] Y[j] / Y[n] (j = n - k), written
// by row pairs (the order in which the adjoint and the links read them), and the
// tile's share of each row's sum_k w[n,k] E'[n,k].  A division, not a product
// with 1 / Y[n]: Y[n] is the rounded sum of the very products divided here, so
// where one term carries the row its weight is exactly 1, and the adjoint, a
// product over up to N rows, stays exact.  (With the reciprocal each row was off
// by a rounding or two: LJ bosons N = 500, P = 32, whose rings hardly exchange,
// had link probabilities off by 8e-15, now by 7e-91; the trap N = 500, P = 32 by
// 4.7e-15, now 1.3e-15; 1.9e-15 and 1.5e-15 where exchange is strong, N = 512.
// Largest error, root mean square over 24 states, against 113-bit sums.)
// A call that the solve left runs the recursion in log space here instead
// (block 0).
__global__ __launch_bounds__(kBlock) void k_boson_weights(BosonArgs a)
{
    __shared__ union { WeightLds v; SeqLds q; } lds;
    double *sW = lds.v.w, *sE = lds.v.e0, *sYm = lds.v.ym, *sC = lds.v.ch;
    int *sYe = lds.v.ye;
    const int t = threadIdx.x, N = a.N, tile = blockIdx.x;
    const BosonScr scr(a);
    int b = (int)((sqrtf(8.0f * (float)tile + 1.0f) - 1.0f) * 0.5f);
    while (boson_tile(b + 1, 0) <= tile) ++b;
    while (boson_tile(b, 0) > tile) --b;
    const int cb = tile - boson_tile(b, 0);
    const int r = t & 63, n = b * kT + 1 + r;
    double2 *wt = reinterpret_cast<double2 *>(scr.w + (size_t)tile * kTT);
    const int4 *ge = reinterpret_cast<const int4 *>(scr.ge + (size_t)tile * kTT);
    constexpr int NQ = kT / 4 / (kBlock / 64);
    Quad g[NQ];
#pragma unroll
    for (int u = 0; u < NQ; ++u) g[u] = quad_at(wt, ge, (t >> 6) + u * (kBlock / 64), r);
    if (N <= kBosonFew || scr.slow[0]) {
        if (tile == 0) seq_recursion(a, lds.q);
        return;
    }
    if (t < 3 * kT) sE[t] = cb * kT + t / 3 < N ? scr.e0[cb * kT * 3 + t] : 0.0;
    if (t < kT && cb * kT + t < N) {
        sYm[t] = scr.ym[cb * kT + t];
        sYe[t] = scr.ye[cb * kT + t];
        sC[t] = scr.chi[cb * kT + t];
        sC[kT + t] = scr.clo[cb * kT + t];
    }
    double el[3] = {0.0, 0.0, 0.0}, ym = 1.0, iy = 1.0;
    DD cn = {0.0, 0.0};
    int yn = 0;
    if (n <= N) {
#pragma unroll
        for (int d = 0; d < 3; ++d) el[d] = scr.el[(n - 1) * 3 + d];
        ym = scr.ym[n];
        iy = 1.0 / ym;
        yn = scr.ye[n];
        cn = {scr.chi[n - 1], scr.clo[n - 1]};
    }
    __syncthreads();
    double eb = 0.0;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int c0 = 4 * ((t >> 6) + u * (kBlock / 64));
        const double gm[4] = {g[u].a.x, g[u].a.y, g[u].b.x, g[u].b.y};
        const int gx[4] = {g[u].e.x, g[u].e.y, g[u].e.z, g[u].e.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = c0 + v;
            double w = 0.0;
            if (n <= N && cb * kT + c < n) {
                w = ldexp(div_by(gm[v] * sYm[c], ym, iy), gx[v] + sYe[c] - yn);
                eb += w * (dd_diff(cn, {sC[c], sC[kT + c]}) + link3(a, el, sE + 3 * c));
            }
            sW[r * (kT + 1) + c] = w;
        }
    }
    __syncthreads();
    for (int q = t; q < kTT / 2; q += kBlock) {
        const double *w2 = sW + 2 * (q >> 6) * (kT + 1) + (q & 63);
        wt[q] = make_double2(w2[0], w2[kT + 1]);
    }
    __syncthreads();
    sW[t] = eb;
    __syncthreads();
    if (t < kT) {
        double x = sW[t];
#pragma unroll
        for (int u = 1; u < kBlock / 64; ++u) x += sW[u * 64 + t];
        scr.eb[(size_t)tile * kT + t] = x;
    }
}

struct AdjLds {
    double2 wd[2][kTT / 2];                 // the current and the next diagonal tile
    double adj[kBosonMaxN + 1 + kT];
    double pm[kSolveWaves][kT];
};

// Adjoints adj[j] = sum_{n>j} w[n,n-j] adj[n], adj[N] = 1, by blocks of 64
// columns from the end, as k_boson_solve (lane c: column c; a step broadcasts
// the adj of the row before, 47 cycles); then V_B and EV_B = the inner energies
// + sum_n adj[n] sum_k w[n,k] E'[n,k].  72 us at N = 1024, 25 us at N = 512, bound
// as the solve.
__global__ __launch_bounds__(kSolve) void k_boson_adjoint(BosonArgs a)
{
    __shared__ AdjLds s;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, N = a.N;
    const BosonScr scr(a);
    const int nb = boson_blocks(N);
    constexpr int W = kSolveWaves - 1;
    constexpr int NL = kT / 2 / kSolveWaves;       // row pairs of the last block per wave
    const double2 *wm = reinterpret_cast<const double2 *>(scr.w);
    {
        const double2 *dg = wm + (size_t)boson_tile(nb - 1, nb - 1) * (kTT / 2);
        const double2 d0 = dg[t], d1 = dg[t + kSolve];
        if (scr.slow[0]) return;
        s.wd[(nb - 1) & 1][t] = d0;
        s.wd[(nb - 1) & 1][t + kSolve] = d1;
    }
    // adj beyond N counts nothing (its rows are zero); column N itself, when
    // it starts a block of its own, is adj[N] = 1
    for (int e = t; e < kBosonMaxN + 1 + kT; e += kSolve) s.adj[e] = (e == N) ? 1.0 : 0.0;
    double acc = ((nb - 1) * kT + lane == N) ? 1.0 : 0.0;
    __syncthreads();
    for (int cb = nb - 1; cb >= 0; --cb) {
        // row pairs of the tile (cb, cb-1): rows 64 cb + 1 .. 64 cb + 64
        double2 last[NL] = {};
        if (cb > 0) {
            const double2 *lt = wm + (size_t)boson_tile(cb, cb - 1) * (kTT / 2);
#pragma unroll
            for (int u = 0; u < NL; ++u) last[u] = (lt + (w * NL + u) * kT)[lane];
        }
        if (w == 0) {
            __builtin_amdgcn_s_setprio(3);
            const double2 *wd = s.wd[cb & 1];
            double x = s.adj[(cb + 1) * kT];
            constexpr int G = 4;                 // row pairs read ahead
            double2 g[G];
#pragma unroll
            for (int u = 0; u < G; ++u) g[u] = wd[(kT / 2 - 1 - u) * kT + lane];
            for (int q = kT / 2 - 1; q >= 0; q -= G) {
                double2 gn[G];
#pragma unroll
                for (int u = 0; u < G; ++u) gn[u] = wd[max(q - G - u, 0) * kT + lane];
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    acc = fma(g[u].y, x, acc);
                    acc = fma(g[u].x, lane_of(acc, 2 * (q - u) + 1), acc);
                    x = lane_of(acc, 2 * (q - u));
                }
#pragma unroll
                for (int u = 0; u < G; ++u) g[u] = gn[u];
            }
            __builtin_amdgcn_s_setprio(0);
            s.adj[cb * kT + lane] = acc;
            acc = 0.0;
        } else if (cb > 0) {
            const double2 *dg = wm + (size_t)boson_tile(cb - 1, cb - 1) * (kTT / 2);
            constexpr int ND = (kTT / 2 + 64 * W - 1) / (64 * W);
            double2 dm[ND];
#pragma unroll
            for (int u = 0; u < ND; ++u) dm[u] = dg[min(t - 64 + u * 64 * W, kTT / 2 - 1)];
            acc = 0.0;
            constexpr int U = 4;
            const int rows = (nb - 1 - cb) * (kT / 2);   // row pairs of the blocks after cb
            double2 g[2][U];
            auto fetch = [&](int h, int q0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int q = min(q0 + u * W, rows - 1), b = cb + 1 + (q >> 5);
                    g[h][u] = (wm + (size_t)boson_tile(b, cb - 1) * (kTT / 2) + (q & 31) * kT)[lane];
                }
            };
            auto add = [&](int h, int q0) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int q = q0 + u * W;
                    const double *x = s.adj + (cb + 1) * kT + 1 + 2 * q;
                    if (q < rows) acc += g[h][u].x * x[0] + g[h][u].y * x[1];
                }
            };
            if (w - 1 < rows) fetch(0, w - 1);
#pragma unroll
            for (int u = 0; u < ND; ++u) {
                const int q = t - 64 + u * 64 * W;
                if (q < kTT / 2) s.wd[(cb - 1) & 1][q] = dm[u];
            }
            for (int q0 = w - 1; q0 < rows; q0 += 2 * W * U) {
                if (q0 + W * U < rows) fetch(1, q0 + W * U);
                add(0, q0);
                if (q0 + 2 * W * U < rows) fetch(0, q0 + 2 * W * U);
                if (q0 + W * U < rows) add(1, q0 + W * U);
            }
        }
        __syncthreads();
        if (cb == 0) break;
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const double *x = s.adj + cb * kT + 1 + 2 * (w * NL + u);
            acc += last[u].x * x[0] + last[u].y * x[1];
        }
        s.pm[w][lane] = acc;
        __syncthreads();
        if (w == 0) {
            acc = 0.0;
#pragma unroll
            for (int u = 0; u < kSolveWaves; ++u) acc += s.pm[u][lane];
        }
    }
    for (int e = t; e <= N; e += kSolve) scr.adj[e] = s.adj[e];
    double ev = 0.0, esum = inner_sum(a, scr, t);
    if (t < N) {
        const int b = t / kT;
        double eb = 0.0;
        for (int cb = 0; cb <= b; ++cb) eb += scr.eb[(size_t)boson_tile(b, cb) * kT + (t & 63)];
        ev = s.adj[t + 1] * eb;
    }
    ev = wave_sum(ev);
    esum = wave_sum(esum);
    if (lane == 0) {
        s.pm[0][w] = ev;
        s.pm[1][w] = esum;
    }
    __syncthreads();
    if (t == 0) {
        for (int u = 1; u < kSolveWaves; ++u) {
            ev += s.pm[0][u];
            esum += s.pm[1][u];
        }
        const DD vb = dd_add1({scr.vp[0], scr.vp[1]}, esum);
        a.res[0] = vb.hi + vb.lo;
        a.res[1] = esum + ev;
    }
}

// Row n, one wave: q[n,j] = adj[n] w[n,n-j], the probability of the closing
// link n-1 -> j; S[n,j] = sum_{j' <= j} q[n,j'], the probability that particle
// n-1's ring starts at j or before; the closing links' force on particle
// n-1's last bead.  With prob, row n-1 of it gets the closing links and zeros
// (its chain entry n is written by k_boson_cols).  Bound by the scans' chain
// (two rows per wave, with 16-byte reads of their pairs, took 18.7 us at
// N = 1024 against 10.9: half the waves, twice the chain).
__global__ __launch_bounds__(kBlock) void k_boson_rows(BosonArgs a)
{
    const int lane = threadIdx.x & 63, N = a.N;
    const int n = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6) + 1;
    if (n > N) return;
    const BosonScr scr(a);
    const double an = scr.adj[n];
    const size_t base = w_at(n, 0) + 2 * lane;
    const double k2 = 2.0 * a.ks;
    double el[3], g[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int d = 0; d < 3; ++d) el[d] = scr.el[(n - 1) * 3 + d];
    double carry = 0.0;
    constexpr int U = 4;                             // tiles at a time, the next ones' reads ahead
    double qn[U], xn[U][3];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = (c0 + u) * kT + lane;
            const bool ok = j < n;
            qn[u] = ok ? scr.w[base + (size_t)(c0 + u) * kTT] : 0.0;
#pragma unroll
            for (int d = 0; d < 3; ++d) xn[u][d] = scr.e0[(ok ? j : 0) * 3 + d];
        }
    };
    fetch(0);
    int c0 = 0;
    for (; c0 * kT < n; c0 += U) {
        double q[U], sc[U], x0[U][3];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            sc[u] = q[u] = an * qn[u];
#pragma unroll
            for (int d = 0; d < 3; ++d) x0[u][d] = xn[u][d];
        }
        if ((c0 + U) * kT < n) fetch(c0 + U);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d) g[d] += k2 * q[u] * mic(x0[u][d], el[d], a.box[d]);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double v = __shfl_up(sc[u], o);
                if (lane >= o) sc[u] += v;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = (c0 + u) * kT + lane;
            if (j < n) scr.s[base + (size_t)(c0 + u) * kTT] = carry + sc[u];
            if (a.prob && j < N) a.prob[(size_t)(n - 1) * N + j] = q[u];
            carry += __shfl(sc[u], 63);
        }
    }
    if (a.prob)
        for (int j = c0 * kT + lane; j < N; j += kT) a.prob[(size_t)(n - 1) * N + j] = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) g[d] = wave_sum(g[d]);
    if (lane == 0) {
#pragma unroll
        for (int d = 0; d < 3; ++d) a.f[bidx(a, a.P - 1, n - 1, d)] += g[d];
    }
}

// Column l: the chain link's probability chain[l] = sum_{n>=l+2} S[n,l] (the
// rings in which l -> l+1 is a link) and the closing links' force on particle
// l's first bead; then the chain links' forces.  A block takes 15 particles and
// the one before them, 16 lanes wide so that a row is read in 128-byte pieces;
// thread (row pair of every second row
// block, column).  17 us at N = 1024, 10 us at N = 512 (one wave per particle,
// whose lanes read a row apart: 30 and 15 us).
constexpr int kColBlock = 1024;
constexpr int kColLanes = 16;
__global__ __launch_bounds__(kColBlock) void k_boson_cols(BosonArgs a)
{
    constexpr int NW = kColBlock / 64;
    __shared__ double red[NW][4][kColLanes];
    const int t = threadIdx.x, c = t & (kColLanes - 1), N = a.N;
    // row pair of a row block; the two halves take alternate row blocks
    const int rp = (t / kColLanes) & (kT / 2 - 1), half = t / (kColBlock / 2);
    static_assert(kColBlock / kColLanes == kT, "two halves of 32 row pairs");
    const int l = (int)blockIdx.x * (kColLanes - 1) - 1 + c;
    const bool in = l >= 0 && l < N;
    const BosonScr scr(a);
    const int nb = boson_blocks(N), cb = in ? l / kT : nb;   // (a lane outside reads nothing)
    const double k2 = 2.0 * a.ks;
    double e0[3] = {0.0, 0.0, 0.0}, v[4] = {0.0, 0.0, 0.0, 0.0};
    if (in)
#pragma unroll
        for (int d = 0; d < 3; ++d) e0[d] = scr.e0[l * 3 + d];
    const double2 *wm = reinterpret_cast<const double2 *>(scr.w);
    const double2 *sm = reinterpret_cast<const double2 *>(scr.s);
    constexpr int U = 2;                             // row blocks read together
    for (int b0 = cb + half; b0 < nb; b0 += 2 * U) {
        double2 q[U], sv[U];
        double el[U][2][3];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = b0 + 2 * u, n = b * kT + 1 + 2 * rp;
            const bool ok = b < nb && n <= N && l <= n;   // (row n+1 may hold l = n)
            const size_t at = ok ? (size_t)boson_tile(b, cb) * (kTT / 2) + rp * kT + (l - cb * kT) : 0;
            q[u] = wm[at];
            sv[u] = sm[at];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const int nv = n + v;
                const bool row = ok && nv <= N && l < nv;
                const double an = row ? scr.adj[nv] : 0.0;
                (v ? q[u].y : q[u].x) = row ? an * (v ? q[u].y : q[u].x) : 0.0;
                if (!row || nv < l + 2) (v ? sv[u].y : sv[u].x) = 0.0;
#pragma unroll
                for (int d = 0; d < 3; ++d) el[u][v][d] = scr.el[((row ? nv : N) - 1) * 3 + d];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                v[d] -= k2 * q[u].x * mic(e0[d], el[u][0][d], a.box[d]);
                v[d] -= k2 * q[u].y * mic(e0[d], el[u][1][d], a.box[d]);
            }
            v[3] += sv[u].x + sv[u].y;
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[q] += __shfl_xor(v[q], 16);
        v[q] += __shfl_xor(v[q], 32);
        if ((t & 63) < kColLanes) red[t >> 6][q][c] = v[q];
    }
    __syncthreads();
    if (t >= 4 * kColLanes) return;
    // one sum per thread, in wave order
    const int q = t / kColLanes;
    double x = red[0][q][c];
    for (int u = 1; u < NW; ++u) x += red[u][q][c];
    __builtin_amdgcn_wave_barrier();
    red[0][q][c] = x;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if (t < 1 || t >= kColLanes || !in) return;
    const double cl = red[0][3][c], cm = red[0][3][c - 1];
    double g[3] = {0.0, 0.0, 0.0}, h[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        h[d] = red[0][d][c];
        if (l + 1 < N) g[d] = k2 * cl * mic(scr.e0[(l + 1) * 3 + d], scr.el[l * 3 + d], a.box[d]);
        if (l >= 1) h[d] -= k2 * cm * mic(e0[d], scr.el[(l - 1) * 3 + d], a.box[d]);
    }
    if (a.prob && l + 1 < N) a.prob[(size_t)l * N + l + 1] = cl;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        a.f[bidx(a, a.P - 1, l, d)] += g[d];
        a.f[bidx(a, 0, l, d)] += h[d];
    }
}

// ---------------------------------------------------------------------------
// The bosonic fix's step in a context (Sec. III.C: Cartesian coordinates,
// since the normal modes change under exchange; the thermostat of Eq. D3 on
// every bead with one damping time).  Thread = (atom, bead), A = kBlock/P
// atoms per block, tiles strided over the grid.  The forces are the array f
// (the potential's: force pass, trap kernel or caller) plus fs (the springs
// inside the rings and the exchange links).  Modes as the distinguishable
// pass: STEP (the pending closing kick, and OBABO's last O, then the
// estimators' sums at that synchronized state, then the opening of the new
// step: BAOAB B A O A, OBABO O B A A), CLOSE, EST, PREP (centroids only).
// The partials are those of the distinguishable pass: PF_EKIN (Cartesian
// kinetic energy), PF_VIR (sum of r . F over the potential's forces, for
// K_VR), the excursion and displacement maxima for the neighbor lists, and
// the non-finite flag.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_bpass(FusedArgs a)
{
    __shared__ double sX[3 * kBlock];    // [A][3][P] positions of the tile
    __shared__ double sC[3 * kBlock];    // [A][3] centroids
    __shared__ double red[64];
    const int P = a.P, N = a.N;
    const int A = kBlock / P;
    const int t = threadIdx.x, la = t / P, k = t - la * P;
    const bool lane_ok = la < A;
    const int mode = a.mode;
    const long long budget = a.ctl->budget;
    const unsigned long long step = a.ctl->step;
    const int synced = a.ctl->synced;
    const bool spent = (mode == FUSED_STEP && budget == 0);
    const bool closing = (mode == FUSED_STEP || mode == FUSED_CLOSE) && !synced;
    const bool est_now = closing || mode == FUSED_EST;
    const bool moves = (mode == FUSED_STEP || mode == FUSED_PREP);
    const double c1 = a.modes[MD_C1], c2 = a.modes[MD_C2];
    const double h = a.hdt;
    double acc_ekin = 0.0, acc_vir = 0.0, acc_emax = 0.0, acc_dmax = 0.0, acc_bad = 0.0;
    const int ntiles = (N + A - 1) / A;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int i = tile * A + la;
        const bool act = lane_ok && i < N;
        double x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0}, fp[3] = {0.0, 0.0, 0.0};
        double ft[3] = {0.0, 0.0, 0.0};
        double hm = 0.0, im = 0.0, sg = 0.0, active = 0.0, cref[3] = {0.0, 0.0, 0.0};
        unsigned oi = 0;
        const size_t b = (size_t)i * 3 * P + k;
        if (act) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                x[d] = a.x[b + d * P];
                v[d] = a.v[b + d * P];
                if (mode != FUSED_PREP) {
                    fp[d] = a.f[b + d * P];
                    ft[d] = fp[d] + a.fs[b + d * P];
                }
            }
            hm = a.atoms[i * 4 + AT_HALF_M];
            im = a.atoms[i * 4 + AT_INV_M];
            sg = a.atoms[i * 4 + AT_SIGMA];
            active = a.atoms[i * 4 + AT_ACTIVE];
            oi = (unsigned)a.orig[i];
            if (k == 0 && moves) {
                cref[0] = a.cref[i * 3]; cref[1] = a.cref[i * 3 + 1]; cref[2] = a.cref[i * 3 + 2];
            }
        }
        if (spent) return;
        if (act) {
            // PILE on this bead's velocity over one O step, noise of step s_
            // and O step q_ of that step, counter (atom, bead, s_, q_)
            auto o_step = [&](unsigned long long s_, unsigned long long q_) {
                double z[3];
                gauss3(a.seed, oi, (unsigned)k, s_, z, (unsigned)q_);
#pragma unroll
                for (int d = 0; d < 3; ++d) v[d] = c1 * v[d] + c2 * sg * z[d];
            };
            if (closing) {
#pragma unroll
                for (int d = 0; d < 3; ++d) v[d] += h * ft[d] * im;
                if (a.obabo && a.nvt) o_step(step - 1, 1);
            }
            if (est_now) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    acc_ekin += hm * v[d] * v[d];
                    acc_vir += x[d] * fp[d];
                }
            }
            if (mode == FUSED_STEP) {
                if (a.obabo) {
                    if (a.nvt) o_step(step, 0);
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        v[d] += h * ft[d] * im;
                        x[d] += h * v[d];
                        x[d] += h * v[d];
                    }
                } else {
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        v[d] += h * ft[d] * im;
                        x[d] += h * v[d];
                    }
                    if (a.nvt) o_step(step, 0);
#pragma unroll
                    for (int d = 0; d < 3; ++d) x[d] += h * v[d];
                }
#pragma unroll
                for (int d = 0; d < 3; ++d) a.x[b + d * P] = x[d];
            }
            if (mode == FUSED_STEP || mode == FUSED_CLOSE) {
#pragma unroll
                for (int d = 0; d < 3; ++d) a.v[b + d * P] = v[d];
            }
#pragma unroll
            for (int d = 0; d < 3; ++d)
                if (!isfinite(x[d]) || !isfinite(v[d])) acc_bad = 1.0;
        }
        if (moves) {
            // centroids, the beads' excursions and the centroids' displacement
            // since the last list build (the rebuild criterion), cells
            __syncthreads();   // the previous tile's reads of sX and sC are done
            if (act) {
#pragma unroll
                for (int d = 0; d < 3; ++d) sX[(la * 3 + d) * P + k] = x[d];
            }
            __syncthreads();
            if (act && k == 0) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    double c = 0.0;
                    for (int j = 0; j < P; ++j) c += sX[(la * 3 + d) * P + j];
                    sC[la * 3 + d] = c / (double)P;
                }
            }
            __syncthreads();
            if (act) {
                double e2 = 0.0, c[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    c[d] = sC[la * 3 + d];
                    const double u = x[d] - c[d];
                    e2 += u * u;
                }
                if (active != 0.0) acc_emax = fmax(acc_emax, e2);
                if (k == 0) {
                    double d2 = 0.0;
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        a.cent[i * 3 + d] = c[d];
                        const double u = c[d] - cref[d];
                        d2 += u * u;
                    }
                    if (active != 0.0) acc_dmax = fmax(acc_dmax, d2);
                    if (a.ncell > 0 && i < a.n_active) (void)cell_of(a, i, c);
                }
            }
        }
    }
    if (spent) return;
    const double s5[5] = {acc_ekin, 0.0, acc_vir, 0.0, 0.0};   // PF_EKIN .. PF_K0
    const double m3[3] = {acc_emax, acc_dmax, acc_bad};
    const double r = block_fold<5, 3>(s5, m3, red);
    if (t < 8) a.partials[(size_t)blockIdx.x * kPartRow + (t < 5 ? t : PF_EMAX + t - 5)] = r;
}

// Harmonic trap on Cartesian beads: f = -m mvv2e omega^2 x for every bead,
// and per block the energy sum 1/2 m mvv2e omega^2 |x|^2 (fpartials, with a
// zero virial).  Thread = (atom, bead) as in the step pass.
__global__ __launch_bounds__(kBlock) void k_btrap(FusedArgs a, double *f, double *fpartials)
{
    __shared__ double red[64];
    const int P = a.P, A = kBlock / P;
    const int t = threadIdx.x, la = t / P, k = t - la * P;
    const int i = blockIdx.x * A + la;
    double e = 0.0;
    if (!a.ctl->ran) return;   // the system took no step (uniform per block)
    if (la < A && i < a.N) {
        const double kk = 2.0 * a.atoms[i * 4 + AT_HALF_M] * a.omega2;
        const size_t b = (size_t)i * 3 * P + k;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double xv = a.x[b + d * P];
            f[b + d * P] = -kk * xv;
            e += 0.5 * kk * xv * xv;
        }
    }
    double e1[1] = {e};
    const double r = block_fold<1>(e1, red);
    if (t == 0) reinterpret_cast<double2 *>(fpartials)[blockIdx.x] = make_double2(r, 0.0);
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};

// The current device's address of scratch, looked up at its first use.
hipError_t device_scratch(double **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

int boson_args(const double *x, int32_t N, int32_t P, double kspring, double beta_n,
               const double *box, double *f, double *prob, double *out, int max_n, BosonArgs &a)
{
    if (!x || !f || !out) return report_error(PIMD_ERR_ARG, "x, f and out must be non-NULL");
    if (N < 1 || P < 1) return report_error(PIMD_ERR_ARG, "N and P must be >= 1");
    if (!(kspring >= 0.0) || !std::isfinite(kspring) || !(beta_n > 0.0) || !std::isfinite(beta_n))
        return report_error(PIMD_ERR_ARG, "kspring >= 0 and beta_n > 0 must be finite");
    if (box)
        for (int d = 0; d < 3; ++d)
            if (!(box[d] >= 0.0) || !std::isfinite(box[d]))
                return report_error(PIMD_ERR_ARG, "box lengths must be finite and >= 0");
    if (N > max_n)
        return report_error(PIMD_ERR_UNSUPPORTED, max_n == kBosonNoAllocMaxN
                                                      ? "N > 512 (the allocation-free scratch's limit)"
                                                      : "N > 1024");
    if (P > kMaxBeads) return report_error(PIMD_ERR_UNSUPPORTED, "P > 128");
    a = BosonArgs{};
    a.x = x;
    a.N = N;
    a.P = P;
    a.layout = 0;
    a.ks = kspring;
    a.bn = beta_n;
    for (int d = 0; d < 3; ++d) a.box[d] = box ? box[d] : 0.0;
    a.f = f;
    a.prob = prob;
    a.res = out;
    return PIMD_OK;
}

}  // namespace

int boson_pass_grid(int N, int P)
{
    const int A = kBlock / P;
    const int ntiles = (N + A - 1) / A;
    return ntiles < 2048 ? ntiles : 2048;
}

void launch_boson_pass(const FusedArgs &a, int grid, hipStream_t st)
{
    hipLaunchKernelGGL(k_bpass, dim3(grid), dim3(kBlock), 0, st, a);
}

int boson_trap_grid(int N, int P)
{
    const int A = kBlock / P;
    return (N + A - 1) / A;
}

void launch_boson_trap(const FusedArgs &a, double *f, double *fpartials, hipStream_t st)
{
    hipLaunchKernelGGL(k_btrap, dim3(boson_trap_grid(a.N, a.P)), dim3(kBlock), 0, st, a, f,
                       fpartials);
}

void launch_boson_springs(const BosonArgs &a, hipStream_t st)
{
    const int tiles = boson_tiles(a.N), inner = inner_blocks(a.N, a.P);
    hipLaunchKernelGGL(k_boson_prep, dim3(tiles + inner + 1), dim3(kBlock), 0, st, a);
    const bool few = a.N <= kBosonFew;   // k_boson_weights runs the whole recursion
    if (!few) hipLaunchKernelGGL(k_boson_solve, dim3(1), dim3(kSolve), 0, st, a);
    hipLaunchKernelGGL(k_boson_weights, dim3(tiles), dim3(kBlock), 0, st, a);
    if (!few) hipLaunchKernelGGL(k_boson_adjoint, dim3(1), dim3(kSolve), 0, st, a);
    hipLaunchKernelGGL(k_boson_rows, dim3((a.N + kBlock / 64 - 1) / (kBlock / 64)), dim3(kBlock), 0,
                       st, a);
    hipLaunchKernelGGL(k_boson_cols, dim3((a.N + kColLanes - 2) / (kColLanes - 1)), dim3(kColBlock), 0,
                       st, a);
}

}  // namespace pimd

using namespace pimd;

extern "C" {

int pimd_boson_spring(const double *x, int32_t N, int32_t P, double kspring, double beta_n,
                      const double *box, double *f, double *prob, double *out, void *stream)
{
    BosonArgs a;
    int rc = boson_args(x, N, P, kspring, beta_n, box, f, prob, out, kBosonMaxN, a);
    if (rc != PIMD_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = hipMalloc((void **)&a.scr, boson_scr_doubles(N) * sizeof(double));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return report_error(PIMD_ERR_OOM, "scratch allocation failed");
    }
    launch_boson_springs(a, st);
    e = hipGetLastError();
    // the scratch is freed once the kernels that read it are done
    const hipError_t es = hipStreamSynchronize(st);
    (void)hipFree(a.scr);
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) return report_error(PIMD_ERR_DEVICE, hipGetErrorString(e));
    return PIMD_OK;
}

int pimd_boson_spring_noalloc(const double *x, int32_t N, int32_t P, double kspring,
                              double beta_n, const double *box, double *f, double *prob,
                              double *out, void *stream)
{
    BosonArgs a;
    int rc = boson_args(x, N, P, kspring, beta_n, box, f, prob, out, kBosonNoAllocMaxN, a);
    if (rc != PIMD_OK) return rc;
    hipError_t e = device_scratch(&a.scr);
    if (e != hipSuccess) return report_error(PIMD_ERR_DEVICE, hipGetErrorString(e));
    // every scratch value the kernels read is written earlier in the same
    // call, so nothing needs clearing
    launch_boson_springs(a, (hipStream_t)stream);
    e = hipGetLastError();
    if (e != hipSuccess) return report_error(PIMD_ERR_DEVICE, hipGetErrorString(e));
    return PIMD_OK;
}

}  // extern "C"

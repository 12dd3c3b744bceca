// HIP kernels for gfx950 (CDNA4): the free-propagator builder and the chain
// rule to (mu, shift).  The dynamic-programme kernels are in cos_level.hip.
#include "cos_internal.hpp"

namespace libcos {

// ---------------------------------------------------------------------------
// free propagator (Methods, square-lattice dispersion; imaginary-time
// propagator with tau = 0 read as 0^-)
//
// What bounds it is the exponential of every (entry, momentum) pair, so the sum
// over the L^2 momenta is folded onto the lattice's symmetries: xi is even in
// both components and symmetric under their exchange, so one term per pair
// q <= p <= L / 2 remains, 15 instead of 64 at L = 8 and 45 instead of 256 at
// L = 16, and its phases become products of two cosines.  A workgroup serves
// g0_chunk configurations (short orders fill less than a workgroup) and all
// matrices, and forms the tables, which do not depend on the configuration,
// once.
// Measured, whole passes with the sums that follow: 8192 configurations of order
// 5, L = 8, 112 -> 53 us; 4096 of order 8 693 -> 667 us; 333 of order 6, L = 8,
// three matrices, with dG/dxi, 274 -> 249 us.  Against the sum over all momenta
// in extended precision the rms error of an entry is smaller: 1.5e-17 (was
// 2.6e-17) of the largest entry at L = 8, 1.2e-17 (2.7e-17) at L = 16.
// ---------------------------------------------------------------------------
constexpr int kG0Chunk = 8;                  // most configurations of a workgroup
constexpr size_t kG0TableBytes = 48 << 10;   // LDS for the tables; more matrices are served in turns

struct G0Params {
    double mu[COS_FMAX], alpha[COS_FMAX];
    double t, beta;
    int L, nmat, nconf, chunk, mper;   // configurations and (at a time) matrices of a workgroup
};

// The entries of a workgroup's configurations, one after another: off[i] is
// where those of configuration c0 + i begin (unit: entries of one matrix).
struct G0Items {
    int off[kG0Chunk + 1];
};

// n^2 entries per configuration, summed by one thread (chunk <= 8)
__device__ __forceinline__ void g0_items(G0Items &it, const int32_t *nvec, int c0, int chunk, int nconf) {
    if (threadIdx.x == 0) {
        int x = 0;
        for (int i = 0; i < chunk; ++i) {
            it.off[i] = x;
            const int n = c0 + i < nconf ? nvec[c0 + i] : 0;
            x += n * n;
        }
        it.off[chunk] = x;
    }
}

// the configuration of the workgroup that holds entry e
__device__ __forceinline__ int g0_config(const G0Items &it, int chunk, int e) {
    int i = 0;
    for (int k = 1; k < chunk; ++k) i += e >= it.off[k] ? 1 : 0;
    return i;
}

__device__ __forceinline__ int wrap(int x, int L) {   // x mod L, in [0, L)
    x %= L;
    return x < 0 ? x + L : x;
}

// x mod L for 0 <= x <= 2 (L - 1)^2, L <= 32; rcp = ceil(2^16 / L) (exact:
// x (L - 1) < 2^16)
__device__ __forceinline__ int small_mod(int x, int L, uint32_t rcp) {
    return x - L * (int)(((uint32_t)x * rcp) >> 16);
}

// Per momentum k the propagator term is -e^{-xi d} (1 - n_F) for d > 0 and
// e^{xi s} n_F for d = -s <= 0.  Written with every exponent non-positive,
// each case is +-exp(E) R_k with R_k = 1 / (1 + e^{-beta |xi_k|}) (the same
// factor for both signs of xi) and E one of -xi d, xi (beta - d), xi s or
// -xi (beta - s): one exponential per term, R_k shared by the entries.
// dG/dxi follows from the same term: g (beta n_F - d), resp. g (beta n_F -
// beta - d).  The momenta (+-p, +-q) and (+-q, +-p) share the term, with the
// phases m_p m_q (cos(p dx) cos(q dy) + cos(q dx) cos(p dy)), m_p = 1 where p
// and -p are the same momentum, else 2, and one of the two products at p = q.
template <bool DG>
__global__ void __launch_bounds__(512) g0_kernel(const int32_t *__restrict__ nvec, const int64_t *__restrict__ voff,
                                                 const int32_t *__restrict__ sites, const double *__restrict__ tau,
                                                 const int64_t *__restrict__ Goff, double *__restrict__ Gout,
                                                 double *__restrict__ dGout, const G0Params p) {
    extern __shared__ double sm[];
    __shared__ G0Items items;
    const int L = p.L, H = L / 2, NP = (H + 1) * (H + 2) / 2;
    double *cs = sm;        // [L] cos(2 pi j / L)
    double *tab = sm + L;   // [mper][NP] xi, 1 / (1 + e^{-beta |xi|}), n_F(xi)
    const int c0 = blockIdx.x * p.chunk;
    const double beta = p.beta;
    for (int j = threadIdx.x; j < L; j += blockDim.x) cs[j] = cospi(2.0 * (double)j / (double)L);
    g0_items(items, nvec, c0, p.chunk, p.nconf);
    for (int g0 = 0; g0 < p.nmat; g0 += p.mper) {
        const int gn = min(p.mper, p.nmat - g0);
        __syncthreads();
        for (int i = threadIdx.x; i < gn * NP; i += blockDim.x) {
            const int g = i / NP;
            int k = i - g * NP, a = 0;
            while (k > a) k -= ++a;   // momentum pair (a, k), k <= a
            const double e = -2.0 * p.t * (cs[a] + cs[k]) - p.mu[g0 + g] + p.alpha[g0 + g];
            const double q = exp(-beta * fabs(e)), r = 1.0 / (1.0 + q);
            tab[3 * i] = e;
            tab[3 * i + 1] = r;
            tab[3 * i + 2] = (e >= 0.0) ? q * r : r;   // Fermi function without overflow
        }
        __syncthreads();
        const int total = items.off[p.chunk];
        for (int i = threadIdx.x; i < total * gn; i += blockDim.x) {
            const int g = i / total, e0 = i - g * total, ci = g0_config(items, p.chunk, e0);
            const int c = c0 + ci, n = nvec[c], e = e0 - items.off[ci], a = e / n, b = e - a * n;
            const int64_t va = voff[c] + a, vb = voff[c] + b;
            const int dx = wrap(sites[2 * va] - sites[2 * vb], L), dy = wrap(sites[2 * va + 1] - sites[2 * vb + 1], L);
            const double d = tau[va] - tau[vb];
            const bool fwd = d > 0.0;
            // exponent coefficients for xi >= 0 and xi < 0, sign, dG offset
            const double cpos = fwd ? -d : -(beta + d), cneg = fwd ? beta - d : -d;
            const double sgn = fwd ? -1.0 : 1.0, doff = fwd ? -d : -beta - d;
            double sg = 0.0, sd = 0.0;
            const double *tk = tab + 3 * g * NP;
            int px = 0, py = 0;   // p dx, p dy mod L
            for (int kp = 0; kp <= H; ++kp) {
                const double mp = (kp == 0 || 2 * kp == L) ? 1.0 : 2.0;
                const double cxp = mp * cs[px], cyp = mp * cs[py];
                int qx = 0, qy = 0;
                for (int kq = 0; kq <= kp; ++kq, tk += 3) {
                    const double mq = (kq == 0 || 2 * kq == L) ? 1.0 : 2.0;
                    const double x = tk[0];
                    const double gk = exp(x * (x >= 0.0 ? cpos : cneg)) * tk[1];
                    double ph = cxp * cs[qy];
                    if (kq < kp) ph = __builtin_fma(cyp, cs[qx], ph);
                    const double wk = mq * ph;
                    sg = __builtin_fma(wk, gk, sg);
                    if (DG) sd = __builtin_fma(wk * gk, __builtin_fma(beta, tk[2], doff), sd);
                    qx += dx;
                    qx -= qx >= L ? L : 0;
                    qy += dy;
                    qy -= qy >= L ? L : 0;
                }
                px += dx;
                px -= px >= L ? L : 0;
                py += dy;
                py -= py >= L ? L : 0;
            }
            const double inv = sgn / (double)(L * L);
            const int64_t at = Goff[c] + (int64_t)(g0 + g) * n * n + e;
            Gout[at] = sg * inv;
            if (DG) dGout[at] = sd * inv;
        }
    }
}

// configurations of a workgroup: more than one only where there are workgroups
// enough to fill the chip (2048 of two wavefronts), and then as many as make a
// short order's n^2 entries fill its threads
static int g0_chunk(int nconf) { return std::max(1, std::min(kG0Chunk, nconf / 2048)); }

hipError_t launch_g0(int nconf, const int32_t *n, const int64_t *voff, const int32_t *sites,
                     const double *tau, int L, double t, double beta, int nmat, const double *mu,
                     const double *alpha, const int64_t *Goff, double *G, double *dG, hipStream_t s) {
    G0Params p;
    for (int g = 0; g < COS_FMAX; ++g) {
        p.mu[g] = g < nmat ? mu[g] : 0.0;
        p.alpha[g] = g < nmat ? alpha[g] : 0.0;
    }
    p.t = t; p.beta = beta; p.L = L; p.nmat = nmat; p.nconf = nconf;
    p.chunk = g0_chunk(nconf);
    const int H = L / 2;
    const size_t per = (size_t)((H + 1) * (H + 2) / 2) * 3 * sizeof(double);   // 3.7 KB at L = 32
    p.mper = (int)std::min<size_t>(nmat, kG0TableBytes / per);
    const size_t shm = p.mper * per + L * sizeof(double);
    const dim3 grid((nconf + p.chunk - 1) / p.chunk), block(128 * std::min(nmat, 4));
    if (dG)
        hipLaunchKernelGGL(g0_kernel<true>, grid, block, shm, s, n, voff, sites, tau, Goff, G, dG, p);
    else
        hipLaunchKernelGGL(g0_kernel<false>, grid, block, shm, s, n, voff, sites, tau, Goff, G, dG, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// free propagator of the honeycomb lattice (Methods, honeycomb Bloch
// Hamiltonian): per flavour H(k) = [[Delta - (mu - alpha), eps], [eps*,
// -Delta - (mu - alpha)]], eps(k) = -t (1 + e^{i k.b1} + e^{i k.b2}).  With
// H = d0 + d.sigma, |d| = r: f(H) = (f(d0 + r) + f(d0 - r)) / 2 + (f(d0 + r) -
// f(d0 - r)) / 2 * d.sigma / r, so per k two eigenvalues and the unit vector
// d / r (in LDS) give every sublattice entry.  Thread per vertex pair, four
// sublattice entries each.
// dG/dxi for a uniform move H -> H + xi (xi = -(mu - alpha)) shifts both
// eigenvalues and keeps d / r, so it is the same sum with f replaced by f'.
//
// Two exponentials per (vertex pair, momentum) bound it.  eps(k) is symmetric in
// (k1, k2) and eps(-k) = eps*(k), and every entry is a real part, so the four
// momenta +-(k1, k2), +-(k2, k1) share their term: 73 instead of 256 at L = 16.
// Workgroups as for the square lattice.
// Measured, 600 configurations of order 7, two matrices, with dG/dxi: a pass with
// gradients 4480 -> 4350 us; rms error 9.5e-18 of the largest entry (was
// 2.6e-17).
// ---------------------------------------------------------------------------
struct HcParams {
    double mu[COS_FMAX], alpha[COS_FMAX], delta[COS_FMAX];
    double t, beta;
    int L, nmat, nconf, chunk, mper;
};

// Fermi function without overflow
__device__ __forceinline__ double fermi(double x, double beta) {
    return (x >= 0.0) ? exp(-beta * x) / (1.0 + exp(-beta * x)) : 1.0 / (exp(beta * x) + 1.0);
}

// imaginary-time factor of one eigenvalue x with Fermi factor nF for the time
// difference d, as in g0_kernel: +-exp(E) R with every exponent E non-positive
// and R = 1 / (1 + e^{-beta |x|}) = (x >= 0 ? 1 - nF : nF); cpos, cneg and sgn
// are the entry's exponent coefficients and sign.
__device__ __forceinline__ double g0_branch(double x, double nF, double cpos, double cneg, double sgn) {
    const bool pos = x >= 0.0;
    return sgn * exp(x * (pos ? cpos : cneg)) * (pos ? 1.0 - nF : nF);
}

// number of classes of momenta under inversion and exchange (fixed points of
// the four operations, over four)
static int hc_classes(int L) { return (L * L + (L % 2 ? 1 : 4) + 2 * L) / 4; }

__global__ void __launch_bounds__(512) g0_honeycomb_kernel(const int32_t *__restrict__ nvec,
                                                           const int64_t *__restrict__ voff,
                                                           const int32_t *__restrict__ cells,
                                                           const double *__restrict__ tau,
                                                           const int64_t *__restrict__ Goff,
                                                           double *__restrict__ Gout, double *__restrict__ dGout,
                                                           const HcParams p, int NC) {
    extern __shared__ double sm[];
    __shared__ G0Items items;
    const int L = p.L, L2 = L * L;
    const uint32_t rcp = (65536u + L - 1) / L;
    double *cs = sm, *sn = sm + L;   // cos / sin (2 pi j / L)
    double *tab = sm + 2 * L;        // [mper][NC] the eigenvalues, their Fermi factors, d / r
    int *cls = (int *)(tab + (int64_t)p.mper * NC * 7);   // [NC] m1 | m2 << 8 | momenta of the class << 16
    const int c0 = blockIdx.x * p.chunk, lane = threadIdx.x & 63;
    for (int j = threadIdx.x; j < L; j += blockDim.x) {
        cs[j] = cospi(2.0 * (double)j / (double)L);
        sn[j] = sinpi(2.0 * (double)j / (double)L);
    }
    g0_items(items, nvec, c0, p.chunk, p.nconf);
    if (threadIdx.x < 64) {   // the first momentum of every class, in order
        int cnt = 0;
        for (int k0 = 0; k0 < L2; k0 += 64) {
            const int k = k0 + lane, m2 = k / L, m1 = k - m2 * L;
            const int i1 = m1 ? L - m1 : 0, i2 = m2 ? L - m2 : 0;
            const int ks = m1 * L + m2, ki = i2 * L + i1, kis = i1 * L + i2;
            const bool own = k < L2 && k <= ks && k <= ki && k <= kis;
            const uint64_t m = __ballot(own);
            if (own) {
                const int size = 1 + (ks != k) + (ki != k && ki != ks) + (kis != k && kis != ks && kis != ki);
                cls[cnt + __popcll(m & ((1ull << lane) - 1ull))] = m1 | m2 << 8 | size << 16;
            }
            cnt += __popcll(m);
        }
    }
    for (int g0 = 0; g0 < p.nmat; g0 += p.mper) {
        const int gn = min(p.mper, p.nmat - g0);
        __syncthreads();
        for (int i = threadIdx.x; i < gn * NC; i += blockDim.x) {
            const int g = i / NC, kc = cls[i - g * NC], m1 = kc & 255, m2 = (kc >> 8) & 255;
            const double er = -p.t * (1.0 + cs[m1] + cs[m2]), ei = -p.t * (sn[m1] + sn[m2]);
            const double d0 = -(p.mu[g0 + g] - p.alpha[g0 + g]), dz = p.delta[g0 + g];
            const double r = sqrt(er * er + ei * ei + dz * dz);
            const double inv = r > 0.0 ? 1.0 / r : 0.0;   // r = 0: both eigenvalues equal, f(H) = f(d0)
            double *tk = tab + (int64_t)i * 7;
            tk[0] = d0 + r;
            tk[1] = d0 - r;
            tk[2] = fermi(d0 + r, p.beta);
            tk[3] = fermi(d0 - r, p.beta);
            tk[4] = dz * inv;
            tk[5] = er * inv;
            tk[6] = ei * inv;
        }
        __syncthreads();
        const int total = items.off[p.chunk];
        for (int i = threadIdx.x; i < total * gn; i += blockDim.x) {
            const int g = i / total, e0 = i - g * total, ci = g0_config(items, p.chunk, e0);
            const int c = c0 + ci, n = nvec[c], e = e0 - items.off[ci], a = e / n, b = e - a * n, D = 2 * n;
            const int64_t va = voff[c] + a, vb = voff[c] + b;
            const int r1 = wrap(cells[2 * va] - cells[2 * vb], L), r2 = wrap(cells[2 * va + 1] - cells[2 * vb + 1], L);
            const double d = tau[va] - tau[vb], beta = p.beta;
            const bool fwd = d > 0.0;
            const double cpos = fwd ? -d : -(beta + d), cneg = fwd ? beta - d : -d, sgn = fwd ? -1.0 : 1.0;
            // d/dx of the branch factor: d > 0: f (beta nF - d); d <= 0: f (beta nF - beta - d)
            const double dsh = fwd ? -d : -beta - d;
            double acc[2][4] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};   // [G, dG/dxi][aa, bb, ab, ba]
            const double *tk = tab + (int64_t)g * NC * 7;
            for (int k = 0; k < NC; ++k, tk += 7) {
                const int kc = cls[k], m1 = kc & 255, m2 = (kc >> 8) & 255;
                const int ph = small_mod(m1 * r1 + m2 * r2, L, rcp), ps = small_mod(m2 * r1 + m1 * r2, L, rcp);
                const double wt = 0.5 * (double)(kc >> 16);   // each of the two phases, with its inverse
                const double ck = wt * (cs[ph] + cs[ps]), sk = wt * (sn[ph] + sn[ps]);
                const double gp = g0_branch(tk[0], tk[2], cpos, cneg, sgn);
                const double gm = g0_branch(tk[1], tk[3], cpos, cneg, sgn);
                const double fpv[2] = {gp, gp * __builtin_fma(beta, tk[2], dsh)};
                const double fmv[2] = {gm, gm * __builtin_fma(beta, tk[3], dsh)};
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (q == 1 && !dGout) break;
                    const double S = 0.5 * (fpv[q] + fmv[q]), Dd = 0.5 * (fpv[q] - fmv[q]);
                    acc[q][0] = __builtin_fma(ck, __builtin_fma(Dd, tk[4], S), acc[q][0]);
                    acc[q][1] = __builtin_fma(ck, __builtin_fma(-Dd, tk[4], S), acc[q][1]);
                    // Re[e^{i phi} Dd (ex + i ey)] and Re[e^{i phi} Dd (ex - i ey)]
                    const double xr = Dd * tk[5], xi = Dd * tk[6];
                    acc[q][2] = __builtin_fma(ck, xr, __builtin_fma(-sk, xi, acc[q][2]));
                    acc[q][3] = __builtin_fma(ck, xr, __builtin_fma(sk, xi, acc[q][3]));
                }
            }
            const double inv = 1.0 / (double)L2;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                double *base = q == 0 ? Gout : dGout;
                if (!base) continue;
                double *out = base + Goff[c] + (int64_t)(g0 + g) * D * D;
                out[(2 * a) * D + 2 * b] = acc[q][0] * inv;
                out[(2 * a) * D + 2 * b + 1] = acc[q][2] * inv;
                out[(2 * a + 1) * D + 2 * b] = acc[q][3] * inv;
                out[(2 * a + 1) * D + 2 * b + 1] = acc[q][1] * inv;
            }
        }
    }
}

hipError_t launch_g0_honeycomb(int nconf, const int32_t *n, const int64_t *voff, const int32_t *cells,
                               const double *tau, int L, double t, double beta, int nmat, const double *mu,
                               const double *alpha, const double *delta, const int64_t *Goff, double *G,
                               double *dG, hipStream_t s) {
    HcParams p;
    for (int g = 0; g < COS_FMAX; ++g) {
        p.mu[g] = g < nmat ? mu[g] : 0.0;
        p.alpha[g] = g < nmat ? alpha[g] : 0.0;
        p.delta[g] = g < nmat ? delta[g] : 0.0;
    }
    p.t = t; p.beta = beta; p.L = L; p.nmat = nmat; p.nconf = nconf;
    p.chunk = g0_chunk(nconf);
    const int nc = hc_classes(L);
    const size_t per = (size_t)nc * 7 * sizeof(double);   // 15 KB at L = 32
    p.mper = (int)std::min<size_t>(nmat, kG0TableBytes / per);
    const size_t shm = p.mper * per + 2 * L * sizeof(double) + nc * sizeof(int);
    hipLaunchKernelGGL(g0_honeycomb_kernel, dim3((nconf + p.chunk - 1) / p.chunk), dim3(64 * std::min(nmat, 8)), shm, s, n,
                       voff, cells, tau, Goff, G, dG, p, nc);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// chain rule to mu and the shift: x = sum_jk dS/dG[j][k] dG/dxi[j][k] per
// (configuration, matrix), mu_bar = -x, alpha_bar = x + sigma_bar / U.  One
// wavefront per (configuration, matrix): the lanes read the n^2 entries
// coalesced and a butterfly over the 64 lanes sums their partial products
// (a fixed order, so repeated calls agree bit for bit).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) chain_kernel(int nconf, const int32_t *__restrict__ nvec, int nmat,
                                                    const int64_t *__restrict__ Goff, const double *__restrict__ Gb,
                                                    const double *__restrict__ dG, const double *__restrict__ sb,
                                                    int nstub, double U, double *__restrict__ mub,
                                                    double *__restrict__ alb) {
    const int lane = threadIdx.x & 63;
    const int64_t nw = (int64_t)nconf * nmat, stride = (int64_t)gridDim.x * (blockDim.x >> 6);
    // wid is uniform in a wavefront: whole wavefronts leave the loop together
    for (int64_t wid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; wid < nw; wid += stride) {
        const int c = (int)(wid / nmat), g = (int)(wid % nmat);
        const int n = nvec[c];
        const int64_t base = Goff[c] + (int64_t)g * n * n;
        double x = 0.0;
        for (int e = lane; e < n * n; e += 64) x = __builtin_fma(Gb[base + e], dG[base + e], x);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
        if (lane == 0) {
            mub[wid] = -x;
            alb[wid] = x + (sb ? sb[(int64_t)c * nstub + (nstub == 1 ? 0 : g)] / U : 0.0);
        }
    }
}

hipError_t launch_chain(int nconf, const int32_t *n, int nmat, const int64_t *Goff, const double *Gb,
                        const double *dG, const double *sb, int nstub, double U, double *mub,
                        double *alb, hipStream_t s) {
    const int64_t blocks = ((int64_t)nconf * nmat + 3) / 4;   // four wavefronts per workgroup
    hipLaunchKernelGGL(chain_kernel, dim3((unsigned)std::min<int64_t>(blocks, 1 << 20)), dim3(256), 0, s, nconf, n,
                       nmat, Goff, Gb, dG, sb, nstub, U, mub, alb);
    return hipGetLastError();
}

}  // namespace libcos

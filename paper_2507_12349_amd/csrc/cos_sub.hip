// Sublattice-summed forward levels (bipartite lattices): the connected sum over
// every assignment of a sublattice label to each vertex, in one pass over the
// labelled state space (Results, four-state interaction mask; Alg. 1/2).
//
// Same organisation as the unlabelled level kernels: one configuration per
// lane, wave-uniform control flow from scalar mask records, one launch per
// level.  A row (m, u, s_u) holds 2n slots (v, s_v); the 2n x 2n matrix of the
// workgroup's flavour sits in LDS as [2n][2n][lane] ((2n)^2 x 512 B, 128 KB at
// n = 8: one workgroup of 16 wavefronts per CU), so the reads of G and the time
// to load it weigh as much as the states.  Hence the two rows of a head, which
// differ in the head's label alone, are taken together: one read of G serves
// both, and in the reverse one LDS add per (i, j).
//
// Measured against one row at a time and the flavours in turn (two flavours):
// n = 8, 1024 configurations, forward 8.8 -> 7.45 ms (best levels 3.6 -> 4.1 TB/s
// of states); n = 7, 600 configurations, forward 1.71 -> 1.0 ms and reverse
// 2.66 -> 1.57 ms (3.7 to 4 TB/s on the large levels).
//
// Rules per row (m, u, s_u), current slots f[(v, s_v)], acc = f . G (formed
// output by output, only for the outputs the row uses):
//   a once-unvisited w is reached on either label: child (m + (w, s)), slot
//   (w, s) = 2 acc[(w, s)] (first visit: either point of w);
//   a once-visited w keeps its label s: child (m with w twice), slot (w, s) =
//   acc[(w, s)];
//   close: t_m = W sum_rows acc[(u, s_u)]; the next cycle opens at the lowest
//   once-visited vertex h with its label s_h (slot (h, s_h) of row (m', h, s_h)),
//   or S = t_m at the full mask.
// Mask-only rules (SU(2), Alg. 1 with its labels): the two planes are the spin
// blocks, as in the unlabelled level kernels: a first visit has weight 1, the
// head point is never reached by an extension, rows (m, 0, s) use plane 0
// while m_0 is once-visited and plane 1 afterwards (the other plane is
// skipped), and the first cycle's successor opens on plane 1 only.
#include "cos_device.hpp"

namespace libcos {

template <int N>
struct SubRec {
    int code, rb;
    uint32_t ones, twos, subb;
    int crb[2 * N];
};

template <int N>
__device__ __forceinline__ SubRec<N> load_sub_rec(const DevPlan &P, int gi) {
    const cint32 *r = (const cint32 *)(P.mrec + (int64_t)gi * kSubRecInts);
    SubRec<N> m;
    m.code = r[0];
    const uint32_t info = (uint32_t)r[1];
    m.ones = info & 0xffffu;
    m.twos = info >> 16;
    m.rb = r[2];
    m.subb = (uint32_t)r[3];
#pragma unroll
    for (int i = 0; i < 2 * N; ++i) m.crb[i] = r[4 + i];
    return m;
}

// child row base for visiting slot i = 2w + s (i wave-uniform; select chain
// keeps the record in scalar registers)
template <int N>
__device__ __forceinline__ int sub_child_base(const SubRec<N> &M, int i) {
    int rb = 0;
#pragma unroll
    for (int k = 0; k < 2 * N; ++k) rb = (k == i) ? M.crb[k] : rb;
    return rb;
}

// bytes of a row
template <int N> constexpr uint32_t kRowB = 2u * N * 512u;

// The states, slots [i0, i0 + NI), of R rows of a mask with head u: row `row`
// (byte offset; label su) alone, or with R = 2 the rows of both labels, which
// follow one another (su = 0).  cs: their current slots from bit 0, returned;
// zeros elsewhere.  MULTI: a cycle opens on slot (u, s_u) with the sum of every
// flavour's part, which lie on that slot of the planes, for u = 0 on its
// neighbour (0, 1 - s_0), which is never current, while the slot itself holds
// this flavour's extension.
template <int N, int R, int NI, bool MULTI, bool MASK>
__device__ __forceinline__ void sub_states(double (&f)[R][NI], uint32_t (&cs)[R], const SubRec<N> &M, int u, int su,
                                           uint32_t row, bool start, plane_t own, const Planes &all, uint32_t lane8,
                                           int i0) {
    const int jc = 2 * u + su;
    const uint32_t c0 = sub_current(N, u, su, M.ones, M.twos, M.subb);
    cs[0] = c0;
    if (R == 2) cs[1] = (c0 & ~(3u << (2 * u))) | ((c0 & (1u << (2 * u))) << 1);
    uint32_t ld[R];   // slots loaded from the own plane
    double y[R], z[R];
    const bool open = MULTI && ((c0 >> jc) & 1u) && (u || (M.twos & 1u));   // wave-uniform
    const uint32_t oat = row + (uint32_t)(u ? jc : jc ^ 1) * 512u, ostep = u ? kRowB<N> + 512u : kRowB<N> - 512u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        ld[r] = start ? 0u : cs[r];
        y[r] = start ? 1.0 : 0.0;   // start: vertex 0 on label s_u
        z[r] = 0.0;
        if (!open) continue;
        if (u || MASK) ld[r] &= ~(1u << (jc + r));
        y[r] = slot_ld(make_plane(all.base), lane8, oat + r * ostep);
        // mask-only: the first cycle's parts lie in plane 0 alone, and vertex 0
        // is not reached by an extension
        if (!MASK || u) z[r] = slot_ld(make_plane(all.base + all.stride), lane8, oat + r * ostep);
    }
#pragma unroll
    for (int k = 0; k < NI; ++k) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            f[r][k] = 0.0;
            if ((ld[r] >> (i0 + k)) & 1u) f[r][k] = state_ld<true>(own, lane8, row + r * kRowB<N> + (i0 + k) * 512u);
        }
    }
    if (open) {
        for (int p = 2; p < all.n; ++p)
#pragma unroll
            for (int r = 0; r < R; ++r) y[r] += slot_ld(make_plane(all.base + p * all.stride), lane8, oat + r * ostep);
    }
    // (one flavour: nothing opens elsewhere, and the start row is no pair.  Adding
    // zeros all the same, which the compiler must keep, made every load wait for
    // the one before it: 64 configurations of n = 8, forward 646 us, without 451;
    // 1000 4407 and 3350; of n = 6 306 and 226)
    if (!MULTI && R == 2) return;
    // (selects: branches here made the compiler keep the reads of G in registers
    // across the two instances, and spill)
#pragma unroll
    for (int k = 0; k < NI; ++k)
#pragma unroll
        for (int r = 0; r < R; ++r) f[r][k] += (i0 + k == jc + r) ? y[r] + z[r] : 0.0;
}

// R rows as in sub_states: every G read serves both.  Adds their closes to T.
template <int N, int R, bool MULTI, bool MASK>
__device__ __forceinline__ void sub_fwd_rows(const SubRec<N> &M, uint32_t gaddr, plane_t own, const Planes &all,
                                             plane_t nxt, uint32_t lane8, int u, int su, uint32_t row, bool start,
                                             double &T, double &dext) {
    constexpr int D = 2 * N;
    const uint32_t ones = M.ones, twos = M.twos, subb = M.subb;
    double f[R][D];
    uint32_t cs[R];
    sub_states<N, R, D, MULTI, MASK>(f, cs, M, u, su, row, start, own, all, lane8, 0);
    // G comes from LDS for every row: a base that is opaque from here on keeps
    // the reads behind the loads of the states
    asm volatile("" : "+v"(gaddr));
    const lds_double *Gs = (const lds_double *)(uintptr_t)gaddr;
#pragma unroll
    for (int w = 0; w < N; ++w) {
        const uint32_t bit = 1u << w;
        if ((twos & bit) && w != u) continue;   // wave-uniform
        const bool once = ones & bit;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int j = 2 * w + s;
            // both labels of an unvisited w, the kept label of a once-visited w
            const bool ext = !(twos & bit) && (!once || (int)((subb >> w) & 1u) == s);
            if (!ext && w != u) continue;
            double a[R];
#pragma unroll
            for (int r = 0; r < R; ++r) a[r] = 0.0;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const double g = Gs[(i * D + j) * 64];
#pragma unroll
                for (int r = 0; r < R; ++r) a[r] = __builtin_fma(f[r][i], g, a[r]);
            }
            if (w == u) {   // the close of the row with label s
                if (R == 2 || s == su) T += a[R == 2 ? s : 0];
                // vertex 0 once visited: the next cycle opens on this same slot
                // (mask-only: the head point itself, not an extension)
                if (R == 1 && !MASK && ext) dext = a[0];
                continue;
            }
            const uint32_t dst = (uint32_t)(M.crb[j] + sub_head_slot(u, su, once ? (twos | bit) : twos)) * kRowB<N> + j * 512u;
#pragma unroll
            for (int r = 0; r < R; ++r)
                state_st<true>(nxt, lane8, dst + r * kRowB<N>, (once || MASK) ? a[r] : 2.0 * a[r]);
        }
    }
}

// opens the next cycle of a mask with this flavour's part of t_m
template <int N, bool MULTI, bool MASK>
__device__ __forceinline__ void sub_fwd_close(const SubRec<N> &M, plane_t nxt, uint32_t lane8, double t, double dext) {
    if (!M.ones) return;
    const int h = __builtin_ctz(M.ones);
    const int sh = (M.subb >> h) & 1u, j = 2 * h + sh;
    const uint32_t row = (uint32_t)(sub_child_base<N>(M, j) + sub_head_slot(h, sh, M.twos | (1u << h))) * kRowB<N>;
    if (!MULTI) {
        slot_st(nxt, lane8, row + j * 512u, t + (h == 0 ? dext : 0.0));
        return;
    }
    slot_st(nxt, lane8, row + (h ? j : j ^ 1) * 512u, t);
    if (!MASK && h == 0) slot_st(nxt, lane8, row + j * 512u, dext);
}

// row pairs of a mask (its one row while vertex 0 is once visited)
__device__ __forceinline__ int sub_pairs(uint32_t twos) { return (twos & 1u) ? 1 + __builtin_popcount(twos & ~1u) : 1; }

// A workgroup serves one group of 64 configurations, one flavour and a block of
// masks, whose wavefronts claim the masks one at a time from an LDS counter (a
// wavefront that drew masks with few rows takes more).  Levels with few masks
// (A.split): the items are (mask, row pair), and the close sums of a mask's
// pairs wait in LDS until one wavefront adds them up, in order.  The last level
// is one mask: one workgroup per group takes the flavours in turn.
template <int N, bool MULTI, bool MASK>
__global__ void __launch_bounds__(1024) sub_fwd_kernel(const LvlArgs A) {
    constexpr int D = 2 * N;
    extern __shared__ double lds[];
    double *Gs_all = lds;               // [D * D][64]
    double *Ts = lds + D * D * 64;      // close sums [item][64] (split)
    __shared__ int next_item, nlist;
    __shared__ uint16_t item_list[kSubSplitMasks * N];
    const int lane = threadIdx.x & 63, wave = COS_RF(threadIdx.x >> 6);   // wave index: uniform
    const int wpb = blockDim.x >> 6;
    const DevPlan &P = A.plan;
    BlockAt at;
    if (!xcd_block(A, at)) return;
    const int gl = at.group, g = A.group0 + gl, nfs = MULTI ? A.nfs : 1;
    const bool last = A.level == 2 * N, start = A.level == 1, each = MULTI && !last;
    const int blk = each ? at.x / nfs : at.x, lam0 = each ? at.x - blk * nfs : 0, lam1 = each ? lam0 + 1 : nfs;
    const int mb0 = blk * A.mpb, nm = min(A.mpb, A.nmasks - mb0);
    const Planes all{A.cur + gl * A.cur_gstride + (int64_t)A.cur_row0 * D * 64, A.cur_frows * D * 64, nfs};
    double *nxt = A.nxt + gl * A.nxt_gstride + (int64_t)A.nxt_row0 * D * 64;
    const uint32_t lane8 = work_lane(A, g, lane) * 8u;
    const uint32_t gaddr = lds_addr(Gs_all) + lane8;
    if (A.split && wave == 0) {
        int cnt = 0;
        if (lane < nm) cnt = sub_pairs((uint32_t)P.mrec[(int64_t)(A.mask0 + mb0 + lane) * kSubRecInts + 1] >> 16);
        int end = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int x = __shfl_up(end, d);
            if (lane >= d) end += x;
        }
        for (int k = 0; k < cnt; ++k) item_list[end - cnt + k] = (uint16_t)(lane << 4 | k);
        if (lane == 63) nlist = end;
    }
    double S = 0.0;
    for (int lam = lam0; lam < lam1; ++lam) {
        if (lam > lam0) __syncthreads();
        if (threadIdx.x == 0) next_item = wpb;   // the first wpb items go to the waves in order
        stage_slots(Gs_all, A.GT + (int64_t)(g * nfs + lam) * D * D * 64, D * D);
        __syncthreads();
        const plane_t own = make_plane(all.base + lam * all.stride), nxtL = make_plane(nxt + lam * (A.nxt_frows * D * 64));
        const int ni = A.split ? COS_RF(nlist) : nm;
        for (int it = wave; it < ni; it = claim(&next_item, lane)) {
            const int word = A.split ? COS_RF((int)item_list[it]) : it << 4;
            const SubRec<N> M = load_sub_rec<N>(P, A.mask0 + mb0 + (word >> 4));
            const bool full0 = M.twos & 1u;   // vertex 0 visited twice: rows come in label pairs
            // mask-only: rows of head vertex 0 use one plane (plane 0 while m_0 is once-visited)
            if (MASK && !full0 && lam != 0) continue;
            int k = word & 15;
            const int k1 = A.split ? k + 1 : sub_pairs(M.twos);
            uint32_t hs = M.twos & ~1u;   // heads >= 1, ascending
            for (int q = 1; q < k; ++q) hs &= hs - 1u;
            double T = 0.0, dext = 0.0;
            if (!full0) {
                sub_fwd_rows<N, 1, MULTI, MASK>(M, gaddr, own, all, nxtL, lane8, 0, (int)(M.subb & 1u),
                                                (uint32_t)M.rb * kRowB<N>, start, T, dext);
            } else {
                for (; k < k1; ++k) {
                    int u = 0;
                    if (k) {
                        u = __builtin_ctz(hs);
                        hs &= hs - 1u;
                    }
                    if (MASK && u == 0 && lam == 0) continue;
                    double t = 0.0;   // pair by pair, as with A.split: the same sum at every batch size
                    sub_fwd_rows<N, 2, MULTI, MASK>(M, gaddr, own, all, nxtL, lane8, u, 0,
                                                    (uint32_t)(M.rb + 2 * k) * kRowB<N>, false, t, dext);
                    T += t;
                }
            }
            if (A.split && full0) Ts[it * 64 + lane] = T;
            else sub_fwd_close<N, MULTI, MASK>(M, nxtL, lane8, A.W * T, dext);
        }
        if (!A.split) continue;
        __syncthreads();
        int i0 = 0;
        for (int m = 0; m < nm; ++m) {
            const SubRec<N> M = load_sub_rec<N>(P, A.mask0 + mb0 + m);
            const int cnt = sub_pairs(M.twos);
            if ((M.twos & 1u) && m % wpb == wave) {
                double T = 0.0;
                for (int i = i0; i < i0 + cnt; ++i) T += Ts[i * 64 + lane];
                if (last) S += T;
                else sub_fwd_close<N, MULTI, MASK>(M, nxtL, lane8, A.W * T, 0.0);
            }
            i0 += cnt;
        }
    }
    if (last && wave == 0) {
        const int cfg = A.lane_cfg[g * 64 + lane];
        if (cfg >= 0 && A.out) A.out[cfg] = A.W * S;
    }
}

// ---------------------------------------------------------------------------
// reverse: B = dS/dF of the labelled states at `level` from B at level + 1,
// the transpose of the forward rules above:
//   a[(w, s)] = c B(child)[(w, s)] for every output the row extends to
//   (c = 2 on a first visit, 1 otherwise and in mask-only mode), plus
//   W tbar_m on the row's close slot (u, s_u);
//   tbar_m = sum_l B(m', h, s_h, l)[(h, s_h)] of the slot the next cycle opens
//   on (1 at the full mask), B(m, u, s_u)[i] = sum_j G[i][j] a[j] over the
//   current slots i, and dS/dG[i][j] += f[i] a[j].
// A wavefront takes the two rows of a head (its two labels) together.  The
// workgroup keeps the rows i of its flavour's G that it needs and their dS/dG
// accumulator for its 64 configurations in LDS ([i][j][lane]), and adds the
// accumulator to the packed gradient at its end.  Up to n = 6 one workgroup owns
// every row i (2 x 72 KB at n = 6); at n = 7, 8 the two matrices would not fit (2 x
// 128 KB at n = 8), so two workgroups, next to each other in the grid, share a block
// of masks, each owning half of the rows i: both read the child adjoints a, each
// reads its half of the states and writes its half of B.
// ---------------------------------------------------------------------------
template <int N>
struct SubAdjShape {
    static constexpr int D = 2 * N;
    static constexpr bool SPLIT = 2 * D * D * 64 * 8 > 160 * 1024;
    static constexpr int RI = SPLIT ? N : D;   // rows i owned by one workgroup
};

// R rows as in sub_states: every G read serves both, and their terms of dS/dG
// are added up before they go to the accumulator
template <int N, int R, bool MULTI, bool MASK>
__device__ __forceinline__ void sub_adj_rows(const SubRec<N> &M, uint32_t gaddr, uint32_t gbaddr, plane_t F,
                                             const Planes &Fall, plane_t Bn, plane_t Bc, uint32_t lane8, int u, int su,
                                             uint32_t row, bool start, double tb, int i0) {
    constexpr int D = 2 * N, RI = SubAdjShape<N>::RI;
    const uint32_t ones = M.ones, twos = M.twos, subb = M.subb;
    double f[R][RI], a[R][D];
    uint32_t need = 0;   // outputs j with a[j] possibly nonzero (wave-uniform)
#pragma unroll
    for (int w = 0; w < N; ++w) {
        const uint32_t bit = 1u << w;
        const bool once = ones & bit;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int j = 2 * w + s;
            bool ext = !(twos & bit) && (!once || (int)((subb >> w) & 1u) == s);
            if (MASK && once && w == 0 && u == 0) ext = false;   // the head point itself
#pragma unroll
            for (int r = 0; r < R; ++r) a[r][j] = 0.0;
            if (!ext) continue;   // wave-uniform
            need |= 1u << j;
            const uint32_t at = (uint32_t)(M.crb[j] + sub_head_slot(u, su, once ? (twos | bit) : twos)) * kRowB<N> + j * 512u;
#pragma unroll
            for (int r = 0; r < R; ++r) a[r][j] = slot_ld(Bn, lane8, at + r * kRowB<N>);
        }
    }
    uint32_t cs[R];
    sub_states<N, R, RI, MULTI, MASK>(f, cs, M, u, su, row, start, F, Fall, lane8, i0);
#pragma unroll
    for (int j = 0; j < D; ++j) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!MASK) a[r][j] *= (((ones | twos) >> (j >> 1)) & 1u) ? 1.0 : 2.0;   // first visit: 2
            a[r][j] += (j == 2 * u + su + r) ? tb : 0.0;   // the row's close slot
        }
    }
    need |= (R == 2 ? 3u : 1u) << (2 * u + su);
    asm volatile("" : "+v"(gaddr));
    asm volatile("" : "+v"(gbaddr));
    const lds_double *Gs = (const lds_double *)(uintptr_t)gaddr;
    lds_double *Gb = (lds_double *)(uintptr_t)gbaddr;
#pragma unroll
    for (int k = 0; k < RI; ++k) {
        uint32_t any = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) any |= cs[r];
        if (!((any >> (i0 + k)) & 1u)) continue;   // wave-uniform
        // every output j, a[j] = 0 where nothing is needed: straight-line LDS
        // reads that issue together and are waited for once, rather than one
        // read-and-wait per needed output behind a branch
        double b[R];
#pragma unroll
        for (int r = 0; r < R; ++r) b[r] = 0.0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const double g = Gs[(k * D + j) * 64];
#pragma unroll
            for (int r = 0; r < R; ++r) b[r] = __builtin_fma(g, a[r][j], b[r]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if ((cs[r] >> (i0 + k)) & 1u) state_st<true>(Bc, lane8, row + r * kRowB<N> + (i0 + k) * 512u, b[r]);
#pragma unroll
        for (int j = 0; j < D; ++j) {
            if (!((need >> j) & 1u)) continue;   // wave-uniform
            double x = f[0][k] * a[0][j];
            if (R == 2) x = __builtin_fma(f[R - 1][k], a[R - 1][j], x);
            __hip_atomic_fetch_add(Gb + (k * D + j) * 64, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
}

// A workgroup serves one group, one flavour and a block of items, which its
// wavefronts claim one at a time: masks, or on levels of few masks (A.row_items)
// (mask, row pair), item i = n m + k standing for pair k of mask m, so that the
// pairs of a mask run side by side.
template <int N, bool MULTI, bool MASK>
__global__ void __launch_bounds__(64 * kSubAdjWaves) sub_adj_kernel(const LvlArgs A) {
    constexpr int D = 2 * N, RI = SubAdjShape<N>::RI;
    extern __shared__ double lds[];
    double *Gs_all = lds;                      // [RI][D][64]  the owned rows of G
    double *Gb_all = lds + RI * D * 64;        // [RI][D][64]  dS/dG of the owned rows, this workgroup
    __shared__ int next_item;
    const int lane = threadIdx.x & 63, wave = COS_RF(threadIdx.x >> 6);   // wave index: uniform
    const int wpb = blockDim.x >> 6;
    const DevPlan &P = A.plan;
    BlockAt at;
    if (!xcd_block(A, at)) return;
    constexpr int Z = SubAdjShape<N>::SPLIT ? 2 : 1;
    const int gl = at.group, g = A.group0 + gl, nfs = MULTI ? A.nfs : 1;
    const int i0 = (at.x % Z) * RI;   // first owned row i
    const int blk = at.x / Z / nfs, lam = at.x / Z - blk * nfs;
    const int nitems = A.row_items ? A.nmasks * N : A.nmasks;
    const int blk0 = blk * A.mpb, ni = min(A.mpb, nitems - blk0);
    const Planes Fall{A.F + gl * A.F_gstride + (int64_t)A.F_row0 * D * 64, A.F_frows * D * 64, nfs};
    const Planes Bn{A.cur + gl * A.cur_gstride, A.cur_frows * D * 64, nfs};   // level + 1
    double *Bc = A.nxt + gl * A.nxt_gstride;                                   // level
    const uint32_t wl = work_lane(A, g, lane), lane8 = wl * 8u;
    const double obar = A.out_bar[A.lane_cfg[g * 64 + wl]];
    const uint32_t gaddr = lds_addr(Gs_all) + lane8, gbaddr = lds_addr(Gb_all) + lane * 8u;
    const bool top = A.level == 2 * N;

    if (threadIdx.x == 0) next_item = wpb;   // the first wpb items go to the waves in order
    for (int i = threadIdx.x; i < RI * D * 64; i += blockDim.x) Gb_all[i] = 0.0;
    stage_slots(Gs_all, A.GT + ((int64_t)(g * nfs + lam) * D + i0) * D * 64, RI * D);
    __syncthreads();
    const plane_t FL = make_plane(Fall.base + lam * Fall.stride), BnL = make_plane(Bn.base + lam * Bn.stride),
                  BcL = make_plane(Bc + lam * (A.nxt_frows * D * 64));
    for (int it = wave; it < ni; it = claim(&next_item, lane)) {
        const int item = blk0 + it, mi = A.row_items ? item / N : item;
        int k = A.row_items ? item - mi * N : 0;
        const SubRec<N> M = load_sub_rec<N>(P, A.mask0 + mi);
        const uint32_t ones = M.ones, twos = M.twos;
        const bool full0 = twos & 1u;
        const int pairs = sub_pairs(twos), k1 = A.row_items ? k + 1 : pairs;
        if (k >= pairs) continue;   // the mask has fewer pairs
        // mask-only: the planes that rows of head vertex 0 use
        if (MASK && !full0 && lam != 0) continue;
        double tb = 0.0;
        if (top) {
            tb = obar;
        } else if (ones) {
            const int h = __builtin_ctz(ones);
            const int sh = (M.subb >> h) & 1u;
            const uint32_t to = (uint32_t)(sub_child_base<N>(M, 2 * h + sh) + sub_head_slot(h, sh, twos | (1u << h))) * kRowB<N> +
                                (2 * h + sh) * 512u;
            // mask-only: the first cycle's successor lives on plane 1 only
            for (int p = (MASK && h == 0 ? 1 : 0); p < nfs; ++p) tb += slot_ld(make_plane(Bn.base + p * Bn.stride), lane8, to);
        }
        tb *= A.W;
        if (!full0) {
            sub_adj_rows<N, 1, MULTI, MASK>(M, gaddr, gbaddr, FL, Fall, BnL, BcL, lane8, 0, (int)(M.subb & 1u),
                                            (uint32_t)M.rb * kRowB<N>, A.level == 1, tb, i0);
            continue;
        }
        uint32_t hs = twos & ~1u;   // heads >= 1, ascending
        for (int q = 1; q < k; ++q) hs &= hs - 1u;
        for (; k < k1; ++k) {
            int u = 0;
            if (k) {
                u = __builtin_ctz(hs);
                hs &= hs - 1u;
            }
            if (MASK && u == 0 && lam == 0) continue;
            sub_adj_rows<N, 2, MULTI, MASK>(M, gaddr, gbaddr, FL, Fall, BnL, BcL, lane8, u, 0,
                                            (uint32_t)(M.rb + 2 * k) * kRowB<N>, false, tb, i0);
        }
    }
    __syncthreads();
    double *__restrict__ gb = A.Gbar_T + ((int64_t)(g * nfs + lam) * D + i0) * D * 64;
    const bool own = g * 64 + lane < A.count;
    for (int i = threadIdx.x; i < RI * D * 64; i += blockDim.x) {
        const double x = Gb_all[i];   // (i's column is this lane's)
        if (x != 0.0 && own) atomicAdd(gb + i, x);
    }
}

static hipError_t allow_sub_lds(const void *fn, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// workgroups of a launch, gridx per group, dealt to the XCDs by xcd_block
static dim3 sub_grid(LvlArgs &a, int gridx, int ngroups) {
    a.gridx = gridx;
    a.ngroups = ngroups;
    return dim3((unsigned)(((int64_t)gridx * ngroups + 7) / 8 * 8));
}

hipError_t launch_sub_level(LvlArgs a, int ngroups, int wpb, hipStream_t s) {
    const int n = a.plan.n;
    if (wpb < 1 || wpb > 16 || (a.split && a.mpb > kSubSplitMasks)) return hipErrorInvalidValue;
    const bool multi = a.nfs > 1, last = a.level == 2 * n;
    if (last && !a.split) return hipErrorInvalidValue;
    const size_t shm = (size_t)(4 * n * n + (a.split ? a.mpb * n : 0)) * 64 * sizeof(double);
    const dim3 grid = sub_grid(a, a.nblocks * (last ? 1 : a.nfs), ngroups);
    switch (n) {
#define COS_SUB_CASE(K)                                                                                  \
    case K: {                                                                                            \
        void (*fn)(LvlArgs) = a.mask_only ? sub_fwd_kernel<K, true, true>                                \
                              : multi     ? sub_fwd_kernel<K, true, false>                               \
                                          : sub_fwd_kernel<K, false, false>;                             \
        hipError_t e = allow_sub_lds((const void *)fn, shm);                                             \
        if (e != hipSuccess) return e;                                                                   \
        hipLaunchKernelGGL(fn, grid, dim3(64 * wpb), shm, s, a);                                         \
        break;                                                                                           \
    }
        COS_SUB_CASE(1) COS_SUB_CASE(2) COS_SUB_CASE(3) COS_SUB_CASE(4)
        COS_SUB_CASE(5) COS_SUB_CASE(6) COS_SUB_CASE(7) COS_SUB_CASE(8)
#undef COS_SUB_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_sub_adj_level(LvlArgs a, int ngroups, hipStream_t s) {
    const int n = a.plan.n;
    const size_t mat = (size_t)(4 * n * n) * 64 * sizeof(double);
    const bool multi = a.nfs > 1;
    const bool halves = 2 * mat > 160 * 1024;   // as SubAdjShape: two workgroups per block of masks
    const size_t shm = halves ? mat : 2 * mat;  // owned rows of G and of the accumulator
    const dim3 grid = sub_grid(a, a.nblocks * a.nfs * (halves ? 2 : 1), ngroups);
    switch (n) {
#define COS_SUBADJ_CASE(K)                                                                               \
    case K: {                                                                                            \
        void (*fn)(LvlArgs) = a.mask_only ? sub_adj_kernel<K, true, true>                                \
                              : multi     ? sub_adj_kernel<K, true, false>                               \
                                          : sub_adj_kernel<K, false, false>;                             \
        hipError_t e = allow_sub_lds((const void *)fn, shm);                                             \
        if (e != hipSuccess) return e;                                                                   \
        hipLaunchKernelGGL(fn, grid, dim3(64 * kSubAdjWaves), shm, s, a);                                \
        break;                                                                                           \
    }
        COS_SUBADJ_CASE(1) COS_SUBADJ_CASE(2) COS_SUBADJ_CASE(3) COS_SUBADJ_CASE(4)
        COS_SUBADJ_CASE(5) COS_SUBADJ_CASE(6) COS_SUBADJ_CASE(7) COS_SUBADJ_CASE(8)
#undef COS_SUBADJ_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace libcos

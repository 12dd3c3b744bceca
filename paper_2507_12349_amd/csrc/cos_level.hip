// Level kernels: one configuration per lane, 64 configurations per wavefront.
//
// The state tables (which rows, heads and currents exist at each level) are
// the same for every configuration of an order n, so a wavefront walks them
// with wave-uniform control flow: mask codes, row bases and current sets sit
// in SGPRs, and every DP state access reads or writes 64 consecutive doubles
// (one per lane), a single 512-byte transaction.  Each lane's own propagator
// matrix sits in LDS.  The launches of a batch run back to back on one stream
// (and can be captured in a graph).
//
// Tiles.  The last vertex b = n - 1 is kept out of the level structure: a mask
// here is the visited counts of the other n - 1 vertices, a level is their
// sum, and a wavefront takes the three states m_b = 0, 1, 2 of a (mask, head)
// together, as a tile of three rows.  The slots whose current vertex is b are
// reached and left inside the tile, so they stay in registers and never pass
// through memory (a slot is written once, by the visit of its current vertex);
// the other slots of the three rows are read and written as before.  Against
// one row at a time this moves a part 1/(n - 1/2) fewer bytes (10% at n = 10),
// takes 2(n - 1) launches instead of 2n, keeps three times the loads in flight
// per wavefront and reads each element of G from LDS once per three rows.
// What bounds them: a tile moves about 3 (n - 1) slots in and out for 3 n (n - 1)
// FMAs, so the large levels run at the memory rate (4.7-4.8 TB/s of states at
// n = 10, against 5.0 TB/s of a plain copy of that size; with the arithmetic
// taken out the reverse gained 10%), the small ones at the latency of a launch
// and of a few tiles in turn.
// Measured (defaults, before -> after, whole levels): forward n = 10, 2048
// configurations, 4.20 -> 3.60 ms; n = 8, 4096, 0.77 -> 0.64 ms; with the reverse
// n = 10, 2048, 10.9 -> 9.5 ms.
//
// Packed layouts (lane fastest):
//   GT   [group][flavour][v][w][64]      propagators
//   sigT [group][flavour][64]            shift weights
//   state buffers [group][flavour][row][v < n - 1][64]
// Rows of a mask m, in order: head 0 (three rows, m_b = 0, 1, 2), then when
// m_0 = 2 each head h >= 1 visited twice (three rows each) and last the one
// row of head b (m_b = 2).  A tile is stored slot by slot ([v][j][64]).
//
// Flavours meet only in t_m, and every flavour has workgroups of its own: each
// stores its own part W sum_u acc[u] of t_m in its own plane, and whoever reads
// a slot on which a cycle opens adds up the parts of all planes.  For head
// h >= 1 the part is the slot (h, h) itself; for head 0, whose slot also takes
// vertex 0's extension, it is a slot of its own in front of the mask's rows
// (batches of one flavour add both and have no such slot).  For head b, which
// opens only in a "special" mask (m_0 = 2, no vertex but b visited once): the
// part is kept in slot 0 of the mask's own head-b row (never a current slot) for
// the reverse sweep, and in slot 0 of the head-b row of every child m + e_w,
// which then adds the opened cycle's first step, 2 t G[b][w], to its slot w.  So
// no part of a level waits for another.  Against the flavours in turn in one
// workgroup: three flavours, n = 10, 1024 configurations, forward 5.94 -> 5.28 ms;
// n = 6, 333, with gradients 531 -> 274 us.
//
// Forward rules per row (m, u) and flavour l (Results; Alg. 2/3):
//   acc = f . G_l;  extension to w (m_w < 2): child (m + e_w, u)[w] = c_w acc[w]
//   (c_w = 2 on a first visit); shift head on the partner of a vertex just
//   reached for the first time: + (-sigma_l) f[w] (doubled on the start row);
//   close: t_m = W sum_{u,l} acc[u]; the next cycle opens at
//   h = min{k : m_k = 1} with value t_m in every flavour, or S = t_m at the
//   full mask.
//
// Mask-only rules (SU(2), w = -1; Results, the variant without cycle factors;
// Alg. 1): the states are (head point, current point, mask) with points, not
// vertices.  They fill the same rows with the two spin blocks as the two
// planes: row (m, 0) holds the head on the up point of vertex 0 (plane 0)
// while m_0 = 1, and on its down point (plane 1) once m_0 = 2; rows (m, h),
// h >= 1, hold both.  The other plane of a row (m, 0) stays empty and is
// skipped.  A point is reached with weight 1 (no factor 2), never onto the
// head point; after the first cycle the next one can open only on the down
// point of vertex 0 (the head is not repeated), later cycles on either end.
#include <algorithm>

#include "cos_device.hpp"

namespace libcos {

// one mask of a level: its vertices visited once and twice, the byte offset of
// its first row inside a flavour plane and those of its children's
template <int N>
struct MaskRec {
    static constexpr int NB = N - 1;
    uint32_t ones, twos, rb;
    uint32_t crb[NB];   // first row of m + e_w; valid where m_w < 2
};

template <int N>
__device__ __forceinline__ MaskRec<N> load_rec(const DevPlan &P, int gi) {
    const cint32 *r = (const cint32 *)(P.mrec + (int64_t)gi * kRecInts);
    MaskRec<N> m;
    const uint32_t info = (uint32_t)r[0];
    m.ones = info & 0xffffu;
    m.twos = info >> 16;
    m.rb = (uint32_t)r[1];
#pragma unroll
    for (int w = 0; w < N - 1; ++w) m.crb[w] = (uint32_t)r[2 + w];
    return m;
}

// first row of the child by vertex h (h is wave-uniform; a select chain keeps
// the record in scalar registers)
template <int N>
__device__ __forceinline__ uint32_t child_rows(const MaskRec<N> &M, int h) {
    uint32_t rb = 0;
#pragma unroll
    for (int w = 0; w < N - 1; ++w) rb = (w == h) ? M.crb[w] : rb;
    return rb;
}

// bytes of a tile's slot (three rows of 64 lanes) and of a tile
constexpr uint32_t kSlotB = 3u * 512u;
template <int N> constexpr uint32_t kTileB = (N - 1) * kSlotB;

// vertex 0 visited twice and no other vertex (but b) visited once
__device__ __forceinline__ bool special_mask(uint32_t ones, uint32_t twos) { return (twos & 1u) && ones == 0u; }

// byte offset, inside the rows of a mask, of the slot on which the next cycle
// opens (head h, current h); h < n - 1
template <int N>
__device__ __forceinline__ uint32_t open_slot(int h, uint32_t twos) {
    return (uint32_t)head_slot(h, twos | (1u << h)) * kTileB<N> + (uint32_t)h * kSlotB;
}

// mask-only: the plane of row (m, 0) that holds no head point
__device__ __forceinline__ bool empty_plane(int u, int lam, uint32_t twos) {
    return u == 0 && ((lam == 0) == ((twos & 1u) != 0u));
}

// ---------------------------------------------------------------------------
// packing: caller layout -> per-lane layout (zeros in padding lanes)
// ---------------------------------------------------------------------------
__global__ void pack_kernel(const PackArgs A) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int N = A.n, nfs = A.nfs;
    const int64_t per_group = (int64_t)nfs * N * N * 64;
    if (i >= per_group * A.ngroups) return;
    const int lane = (int)(i & 63);
    int64_t rest = i >> 6;
    const int w = (int)(rest % N); rest /= N;
    const int v = (int)(rest % N); rest /= N;
    const int l = (int)(rest % nfs); rest /= nfs;
    const int g = (int)rest;
    const int slot = g * 64 + lane;
    const int c = slot < A.count ? A.order[slot] : -1;
    double x = 0.0;
    if (c >= 0) {
        const int64_t off = A.Goff ? A.Goff[c] : (int64_t)c * A.nmat * N * N;
        x = A.G[off + ((int64_t)(A.variant ? l : 0) * N + v) * N + w];
    }
    A.GT[i] = x;
    if (v == 0 && w == 0) {
        const int64_t si = ((int64_t)g * nfs + l) * 64 + lane;
        if (A.sigT) A.sigT[si] = (c >= 0 && A.stub) ? A.stub[(int64_t)c * A.nstub + (A.variant ? l : 0)] : 0.0;
        if (l == 0) A.lane_cfg[slot] = c;
    }
}

// ---------------------------------------------------------------------------
// forward: level -> level + 1
// ---------------------------------------------------------------------------
// The states of a tile: rows (m, m_b = j), head u, j = 0, 1, 2, at byte offset
// `row`; zeros where v is not current (wave-uniform).  MULTI: the slot that the
// tile's cycle opens on is the sum of every plane's part (for head 0 the parts
// lie in front of the mask's rows, and the slot holds this flavour's extension).
template <int N, bool MULTI, bool MASK, bool STREAM>
__device__ __forceinline__ void tile_states(double (&f)[3][N - 1], const MaskRec<N> &M, uint32_t cm, int u, uint32_t row,
                                            bool start, plane_t own, const Planes &all, const uint32_t (&off)[3]) {
    uint32_t ld = start ? 0u : cm;   // slots read from the own plane
    double y[3] = {0.0, 0.0, 0.0}, z[3] = {0.0, 0.0, 0.0};
    const bool open = MULTI && ((ld >> u) & 1u) && (u || (M.twos & 1u));
    const uint32_t oat = u ? row + (uint32_t)u * kSlotB : M.rb - kSlotB;
    if (open) {
        // mask-only: the first cycle's parts lie in plane 0 alone, and vertex 0
        // is not reached by an extension
        if (u || MASK) ld &= ~(1u << u);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            y[j] = slot_ld(make_plane(all.base), off[j], oat);
            if (!MASK || u) z[j] = slot_ld(make_plane(all.base + all.stride), off[j], oat);
        }
    }
#pragma unroll
    for (int v = 0; v < N - 1; ++v) {
        f[0][v] = f[1][v] = f[2][v] = 0.0;
        if (!((ld >> v) & 1u)) continue;
        const uint32_t at = row + v * kSlotB;
#pragma unroll
        for (int j = 0; j < 3; ++j) f[j][v] = state_ld<STREAM>(own, off[j], at);
    }
    if (MULTI) {
        if (open && !MASK) {
            for (int k = 2; k < all.n; ++k) {
                const plane_t p = make_plane(all.base + k * all.stride);
#pragma unroll
                for (int j = 0; j < 3; ++j) y[j] += slot_ld(p, off[j], oat);
            }
        }
        // (selects: branches here made the compiler spill)
#pragma unroll
        for (int v = 0; v < N - 1; ++v)
#pragma unroll
            for (int j = 0; j < 3; ++j) f[j][v] += v == u ? y[j] + z[j] : 0.0;
    }
    if (start) f[0][0] = 1.0;   // mask-only: plane 0 only (plane 1 skipped)
}

// The states of the row of head b, at byte offset `row`: where exactly one
// vertex w is visited once, the cycle opened in m - e_w adds its first step.
// Returns G in LDS.
template <int N, bool MASK, bool STREAM>
__device__ __forceinline__ const lds_double *brow_states(double (&f)[N - 1], const MaskRec<N> &M, uint32_t row,
                                                         uint32_t gaddr, plane_t own, const Planes &all, uint32_t off) {
    constexpr int NB = N - 1;
    const uint32_t cm = (M.ones | M.twos) & ~1u;
    int w = 31;
    double y = 0.0;
    if (M.ones && (M.ones & (M.ones - 1u)) == 0u) {
        w = __builtin_ctz(M.ones);
        y = (MASK ? 1.0 : 2.0) * all.sum(off, row) * ((const lds_double *)(uintptr_t)gaddr)[(NB * N + w) * 64];
    }
    asm volatile("" : "+v"(y));
#pragma unroll
    for (int v = 0; v < NB; ++v) {
        f[v] = v == w ? y : 0.0;   // wave-uniform
        if ((cm >> v) & 1u) f[v] += state_ld<STREAM>(own, off, row + v * 512u);
    }
    asm volatile("" : "+v"(gaddr));   // as in fwd_tile
    const lds_double *Gs = (const lds_double *)(uintptr_t)gaddr;
    return Gs;
}

// One tile.  own, nxt: this flavour's planes; hb: byte offset of the tile in its
// mask's rows.  Adds the close to T[j] and returns in dext[j] the extension of
// vertex 0 to its second visit while m_0 = 1 (the next cycle opens on that same
// slot).
template <int N, bool MULTI, bool MASK, bool STREAM>
__device__ __forceinline__ void fwd_tile(const MaskRec<N> &M, uint32_t gaddr, plane_t own, const Planes &all, plane_t nxt,
                                         const uint32_t (&off)[3], int u, uint32_t hb, bool start, double sg,
                                         double (&T)[3], double (&dext)[3]) {
    constexpr int NB = N - 1;
    const uint32_t ones = M.ones, twos = M.twos;
    const uint32_t cm = current_set(u, ones, twos);   // the same for the three rows (on the start row: j = 0 only)
    double f[3][NB];
    tile_states<N, MULTI, MASK, STREAM>(f, M, cm, u, M.rb + hb, start, own, all, off);
    // G comes from LDS for every tile: a base that is opaque from here on keeps
    // the N^2 reads behind the loads of the states, instead of in N^2 registers
    asm volatile("" : "+v"(gaddr));
    const lds_double *Gs = (const lds_double *)(uintptr_t)gaddr;
    // vertex b first: the slots with current b of rows j = 1, 2
    double fb1, fb2;
    {
        double a0 = 0.0, a1 = 0.0;
#pragma unroll
        for (int v = 0; v < NB; ++v) {
            const double g = Gs[(v * N + NB) * 64];
            a0 = __builtin_fma(f[0][v], g, a0);
            a1 = __builtin_fma(f[1][v], g, a1);
        }
        fb1 = MASK ? a0 : 2.0 * a0;
        a1 = __builtin_fma(fb1, (double)Gs[(NB * N + NB) * 64], a1);
        fb2 = __builtin_fma(-sg, fb1, a1);
    }
    const double sgx = start ? 2.0 * sg : sg;
#pragma unroll
    for (int w = 0; w < NB; ++w) {
        const uint32_t bit = 1u << w;
        if ((twos & bit) && w != u) continue;   // wave-uniform: output not needed
        double a[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < NB; ++v) {
            const double g = Gs[(v * N + w) * 64];
#pragma unroll
            for (int j = 0; j < 3; ++j) a[j] = __builtin_fma(f[j][v], g, a[j]);
        }
        {
            const double g = Gs[(NB * N + w) * 64];
            a[1] = __builtin_fma(fb1, g, a[1]);
            a[2] = __builtin_fma(fb2, g, a[2]);
        }
        if (w == u) {
#pragma unroll
            for (int j = 0; j < 3; ++j) T[j] += a[j];
        }
        if (twos & bit) continue;
        const bool first = !(ones & bit);
        if (MASK && w == 0 && u == 0) continue;   // the head point itself: not an extension
        if (first) {
#pragma unroll
            for (int j = 0; j < 3; ++j) a[j] *= MASK ? 1.0 : 2.0;
        } else if (cm & bit) {
#pragma unroll
            for (int j = 0; j < 3; ++j) a[j] = __builtin_fma(-sgx, f[j][w], a[j]);
        }
        if (w == 0 && u == 0 && !(twos & 1u)) {
#pragma unroll
            for (int j = 0; j < 3; ++j) dext[j] = a[j];
            continue;
        }
        // a second visit below the head moves the child's head one tile up
        const uint32_t dst = M.crb[w] + hb + ((!first && w < u) ? kTileB<N> : 0u) + w * kSlotB;
#pragma unroll
        for (int j = 0; j < 3; ++j) state_st<STREAM>(nxt, off[j], dst, a[j]);
    }
}

// the row of head b (m_b = 2) at byte offset hb of its mask's rows; returns its
// close
template <int N, bool MASK, bool STREAM>
__device__ __forceinline__ double fwd_brow(const MaskRec<N> &M, uint32_t gaddr, plane_t own, const Planes &all,
                                           plane_t nxt, uint32_t off, uint32_t hb, double sg) {
    constexpr int NB = N - 1;
    const uint32_t ones = M.ones, twos = M.twos;
    const uint32_t cm = (ones | twos) & ~1u;
    double f[NB], close = 0.0;
    const lds_double *Gs = brow_states<N, MASK, STREAM>(f, M, M.rb + hb, gaddr, own, all, off);
#pragma unroll
    for (int w = 0; w < N; ++w) {
        const uint32_t bit = 1u << w;
        if (w < NB && (twos & bit)) continue;
        double a = 0.0;
#pragma unroll
        for (int v = 0; v < NB; ++v) a = __builtin_fma(f[v], Gs[(v * N + w) * 64], a);
        if (w == NB) {
            close = a;
            continue;
        }
        const bool first = !(ones & bit);
        if (first) a *= MASK ? 1.0 : 2.0;
        else if (cm & bit) a = __builtin_fma(-sg, f[w < NB ? w : 0], a);
        state_st<STREAM>(nxt, off, M.crb[w < NB ? w : 0] + hb + (first ? 0u : kTileB<N>) + w * 512u, a);
    }
    return close;
}

// Opens the next cycle of a mask that is not full with this flavour's part of
// t_m (T: sums over its heads).
template <int N, bool MULTI, bool MASK>
__device__ __forceinline__ void close_mask(const MaskRec<N> &M, double W, plane_t own, plane_t nxt,
                                           const uint32_t (&off)[3], const double (&T)[3], const double (&dext)[3]) {
    constexpr int NB = N - 1;
    if (special_mask(M.ones, M.twos)) {   // head b, m_b = 1
        const uint32_t brow = (1u + (uint32_t)__builtin_popcount(M.twos & ~1u)) * kTileB<N>;
        const double x = W * T[1];
        slot_st(own, off[0], M.rb + brow, x);
#pragma unroll
        for (int w = 0; w < NB; ++w)
            if (!((M.twos >> w) & 1u)) slot_st(nxt, off[0], M.crb[w] + brow, x);
        return;
    }
    const int h = __builtin_ctz(M.ones);   // some vertex but b is visited once
    const uint32_t base = child_rows<N>(M, h), dst = base + open_slot<N>(h, M.twos);
    if (!MULTI) {
#pragma unroll
        for (int j = 0; j < 3; ++j) slot_st(nxt, off[j], dst, __builtin_fma(W, T[j], h == 0 ? dext[j] : 0.0));
        return;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) slot_st(nxt, off[j], h ? dst : base - kSlotB, W * T[j]);
    if (!MASK && h == 0) {
#pragma unroll
        for (int j = 0; j < 3; ++j) slot_st(nxt, off[j], dst, dext[j]);
    }
}

// head of slot k of a mask with `heads` (the heads >= 1)
__device__ __forceinline__ int head_of(uint32_t heads, int k) {
    for (int s = 1; s < k; ++s) heads &= heads - 1u;
    return k ? __builtin_ctz(heads) : 0;
}

// head slots of a mask: its tiles, and the head-b row
__device__ __forceinline__ int head_slots(uint32_t twos) {
    return (twos & 1u) ? 2 + __builtin_popcount(twos & ~1u) : 1;
}

// lists the items (mask << 4 | head slot) of a block of `nm` <= 64 masks, mask
// by mask, heads in order: lane m of one wavefront takes mask m.  Returns their
// number in lane 63.
__device__ __forceinline__ int list_items(uint16_t *list, const int32_t *mrec, int nm, int lane) {
    const int cnt = lane < nm ? head_slots((uint32_t)mrec[(int64_t)lane * kRecInts] >> 16) : 0;
    int end = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int x = __shfl_up(end, d);
        if (lane >= d) end += x;
    }
    for (int k = 0; k < cnt; ++k) list[end - cnt + k] = (uint16_t)(lane << 4 | k);
    return end;
}

// The last level: the full mask alone.  One workgroup per group, its heads
// spread over the wavefronts, flavour after flavour; wavefront 0 adds up the
// closes.  (A kernel of its own: inside level_fwd_kernel a further copy of the
// tile made the compiler spill.)
template <int N, bool MULTI, bool MASK>
__global__ void __launch_bounds__(1024) level_last_kernel(const LvlArgs A) {
    constexpr int NB = N - 1;
    extern __shared__ double lds[];
    double *Gs_all = lds, *Ts = lds + N * N * 64;   // G, close sums [head][3][64]
    const int lane = threadIdx.x & 63, wave = COS_RF(threadIdx.x >> 6), wpb = blockDim.x >> 6;
    const int gl = blockIdx.x, g = A.group0 + gl, nfs = MULTI ? A.nfs : 1;
    const Planes all{A.cur + gl * A.cur_gstride + (int64_t)A.cur_row0 * 64, A.cur_frows * 64, nfs};
    const plane_t nxt = make_plane(A.nxt);   // (nothing is open: never written)
    const uint32_t wl = work_lane(A, g, lane), lane8 = wl * 8u;
    const uint32_t off[3] = {lane8, lane8 + 512u, lane8 + 1024u};
    const MaskRec<N> M = load_rec<N>(A.plan, A.mask0);
    const uint32_t heads = M.twos & ~1u, brow = (uint32_t)NB * kTileB<N>;
    const uint32_t gaddr = lds_addr(Gs_all) + lane8;
    double T1 = 0.0, T2 = 0.0, gbb = 0.0;
    for (int lam = 0; lam < nfs; ++lam) {
        if (MULTI && lam) __syncthreads();
        stage_slots(Gs_all, A.GT + (int64_t)(g * nfs + lam) * N * N * 64, N * N);
        __syncthreads();
        const double sg = A.stubs ? A.sigT[(int64_t)(g * nfs + lam) * 64 + wl] : 0.0;
        const plane_t own = make_plane(all.base + lam * all.stride);
        for (int k = wave; k <= NB; k += wpb) {
            double T[3] = {0.0, 0.0, 0.0}, dext[3] = {0.0, 0.0, 0.0};
            const int u = head_of(heads, min(k, NB - 1));
            if (k == NB) T[2] = fwd_brow<N, MASK, true>(M, gaddr, own, all, nxt, lane8, brow, sg);
            else if (!(MASK && empty_plane(u, lam, M.twos)))
                fwd_tile<N, MULTI, MASK, true>(M, gaddr, own, all, nxt, off, u, (uint32_t)k * kTileB<N>, false, sg, T, dext);
#pragma unroll
            for (int j = 0; j < 3; ++j) Ts[(k * 3 + j) * 64 + lane] = T[j];
        }
        __syncthreads();
        if (wave) continue;
        double s1 = 0.0, s2 = 0.0;
        for (int k = 0; k <= NB; ++k) {
            s1 += Ts[(k * 3 + 1) * 64 + lane];
            s2 += Ts[(k * 3 + 2) * 64 + lane];
        }
        T1 += A.W * s1;   // the parts of the cycle of head b, as the other masks store them
        T2 += s2;
        gbb += Gs_all[(NB * N + NB) * 64 + lane];
        slot_st(own, lane8, M.rb + brow, A.W * s1);
    }
    // the cycle of head b closes at once
    const int cfg = A.lane_cfg[g * 64 + lane];
    if (wave == 0 && cfg >= 0 && A.out) A.out[cfg] = A.W * __builtin_fma(T1, gbb, T2);
}

// A workgroup serves one group of 64 configurations, one flavour and a block of
// masks.  G_l of the 64 lanes sits in LDS ([v][w][lane], conflict-free: the
// lanes read consecutive words), loaded once by the whole workgroup.
//   Levels of many masks: the wavefronts claim the block's masks one at a time
// from an LDS counter (a wavefront that drew masks with few heads takes more)
// and take a mask's heads in turn.
//   Levels with fewer masks than wavefronts that fit the chip (A.split): the
// heads of a mask go to different wavefronts, and the close sums of the heads
// wait in LDS until one wavefront adds them up, in the same order.
template <int N, bool MULTI, bool MASK>
__global__ void __launch_bounds__(1024) level_fwd_kernel(const LvlArgs A) {
    extern __shared__ double lds[];
    double *Gs_all = lds;                      // [N * N][64]
    double *Ts = lds + N * N * 64;             // close sums of heads [item][3][64] (split)
    __shared__ int next_mask, nitems;
    __shared__ uint16_t item_list[kSplitMasks * N];
    const int lane = threadIdx.x & 63, wave = COS_RF(threadIdx.x >> 6);   // wave index: uniform
    const int wpb = blockDim.x >> 6;
    const DevPlan &P = A.plan;
    BlockAt at;
    if (!xcd_block(A, at)) return;
    const int gl = at.group, g = A.group0 + gl;
    const int nfs = MULTI ? A.nfs : 1;
    // wave-uniform bases; the lane's word is added at each access.  States are
    // stored by flavour plane: [flavour][row][v][lane], planes of *_frows slots
    const Planes all{A.cur + gl * A.cur_gstride + (int64_t)A.cur_row0 * 64, A.cur_frows * 64, nfs};
    double *nxt = A.nxt + gl * A.nxt_gstride + (int64_t)A.nxt_row0 * 64;
    const uint32_t wl = work_lane(A, g, lane), lane8 = wl * 8u;
    const uint32_t off[3] = {lane8, lane8 + 512u, lane8 + 1024u};
    const uint32_t gaddr = lds_addr(Gs_all) + lane8;
    const bool start = A.level == 1;
    const double *GT = A.GT + (int64_t)g * nfs * N * N * 64, *sigT = A.stubs ? A.sigT + (int64_t)g * nfs * 64 : nullptr;

    const int blk = MULTI ? at.x / nfs : at.x, lam = MULTI ? at.x - blk * nfs : 0;
    const int mb0 = blk * A.mpb, mb1 = min(mb0 + A.mpb, A.nmasks);
    if (A.split && wave == 0) {
        const int n = list_items(item_list, P.mrec + (int64_t)(A.mask0 + mb0) * kRecInts, mb1 - mb0, lane);
        if (lane == 63) nitems = n;
    }
    if (threadIdx.x == 0) next_mask = mb0 + wpb;   // the first wpb masks go to the waves in order
    stage_slots(Gs_all, GT + (int64_t)lam * N * N * 64, N * N);
    __syncthreads();
    const double sg = sigT ? sigT[lam * 64 + wl] : 0.0;
    const plane_t own = make_plane(all.base + lam * all.stride), nxtL = make_plane(nxt + lam * (A.nxt_frows * 64));
    if (A.split) {
        const int ni = COS_RF(nitems);
        for (int i = wave; i < ni; i += wpb) {
            const int word = COS_RF((int)item_list[i]), k = word & 15;
            const MaskRec<N> M = load_rec<N>(P, A.mask0 + mb0 + (word >> 4));
            const uint32_t heads = (M.twos & 1u) ? (M.twos & ~1u) : 0u, hb = (uint32_t)k * kTileB<N>;
            double T[3] = {0.0, 0.0, 0.0}, dext[3] = {0.0, 0.0, 0.0};
            if (k == 1 + __builtin_popcount(heads)) {
                T[2] = fwd_brow<N, MASK, true>(M, gaddr, own, all, nxtL, lane8, hb, sg);
            } else {
                const int u = head_of(heads, k);
                if (!(MASK && empty_plane(u, lam, M.twos)))
                    fwd_tile<N, MULTI, MASK, true>(M, gaddr, own, all, nxtL, off, u, hb, start, sg, T, dext);
            }
            if (!(M.twos & 1u)) {   // the mask's only head
                close_mask<N, MULTI, MASK>(M, A.W, own, nxtL, off, T, dext);
            } else {
#pragma unroll
                for (int j = 0; j < 3; ++j) Ts[(i * 3 + j) * 64 + lane] = T[j];
            }
        }
        __syncthreads();
        int i0 = 0;
        for (int m = 0; m < mb1 - mb0; ++m) {
            const MaskRec<N> M = load_rec<N>(P, A.mask0 + mb0 + m);
            const int cnt = head_slots(M.twos);
            if ((M.twos & 1u) && m % wpb == wave) {
                double T[3] = {0.0, 0.0, 0.0};
                const double dext[3] = {0.0, 0.0, 0.0};
                for (int i = i0; i < i0 + cnt; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) T[j] += Ts[(i * 3 + j) * 64 + lane];
                close_mask<N, MULTI, MASK>(M, A.W, own, nxtL, off, T, dext);
            }
            i0 += cnt;
        }
        return;
    }
    for (int mi = mb0 + wave; mi < mb1; mi = claim(&next_mask, lane)) {
        const MaskRec<N> M = load_rec<N>(P, A.mask0 + mi);
        const uint32_t twos = M.twos;
        uint32_t hs = (twos & 1u) ? (twos & ~1u) : 0u;   // heads >= 1, ascending
        int u = 0;
        uint32_t hb = 0;
        double T[3] = {0.0, 0.0, 0.0}, dext[3] = {0.0, 0.0, 0.0};
        while (true) {
            if (!(MASK && empty_plane(u, lam, twos)))
                fwd_tile<N, MULTI, MASK, true>(M, gaddr, own, all, nxtL, off, u, hb, start, sg, T, dext);
            hb += kTileB<N>;
            if (!hs) break;
            u = __builtin_ctz(hs);
            hs &= hs - 1u;
        }
        if (twos & 1u) T[2] += fwd_brow<N, MASK, true>(M, gaddr, own, all, nxtL, lane8, hb, sg);
        close_mask<N, MULTI, MASK>(M, A.W, own, nxtL, off, T, dext);
    }
}

// ---------------------------------------------------------------------------
// reverse: B = dS/dF at level `level` from B at level + 1.
//   a[w] = c_w B(m + e_w, u)[w] (open w) + [w == u] W tbar_m,
//   tbar_m = sum_l B(m + e_h, h, l)[h] (1 at the full mask, 0 when dropped),
//   B(m, u)[v] = sum_w G[v][w] a[w] + [m_v = 1, v current] (-sigma) a'[v]
//   (a' = a without the close term), Gbar[v][w] += f[v] a[w],
//   sigmabar += -f[w] B(m + e_w, u)[w] on the shift edges.
//
// The tiles of the forward, backwards: of the three rows the adjoints of the
// slots with current b are formed from j = 2 down and stay in registers, and
// the forward's values of those slots (which dS/dG needs) are formed again
// from the slots read.  The dS/dG accumulator of the 64 configurations of the
// workgroup lives in LDS next to G ([v][w][lane], the lanes add to consecutive
// words) and is added to the packed gradient once per workgroup and flavour; a
// tile sums its three rows' terms in registers first, so the accumulator takes
// one LDS add per touched (v, w) pair and tile.
// ---------------------------------------------------------------------------
// How a tile adds to the LDS accumulator: at once, in whatever order the
// wavefronts come (Unordered), or (InTurn) only once every item before it has
// added its terms, so that the order of summation is that of the items.  A
// wavefront takes its items in ascending order, so the one with the lowest
// item left never waits and every turn comes.  The accumulator's rows v have
// kTurns turns, so that an item adds to the first rows while the one before it
// is still at the later ones.  A turn orders LDS accesses alone: its adds have
// arrived (lgkmcnt) before the next item's turn is stored, while the item's
// stores of adjoints to memory may still be on their way.
constexpr int kTurns = 3;
__device__ __forceinline__ void lds_add(lds_double *p, double x) {
    __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <int N>
__device__ __forceinline__ constexpr int first_row(int stage) { return (stage * N + kTurns - 1) / kTurns; }
struct Unordered {
    static constexpr bool kDefer = false;
    __device__ __forceinline__ void wait(int) const {}
    __device__ __forceinline__ void done(int) const {}
    __device__ __forceinline__ void last(lds_double *, double) const {}
};
struct InTurn {
    static constexpr bool kDefer = true;
    lds_int *turn;   // the item whose turn it is, for each part of the rows
    int item, stubs;
    __device__ __forceinline__ void wait(int stage) const {
        while (COS_RF(__hip_atomic_load(turn + stage, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != item)
            __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
    }
    __device__ __forceinline__ void done(int stage) const {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __hip_atomic_store(turn + stage, item + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // the end of an item: its shift terms too
    __device__ __forceinline__ void last(lds_double *sig, double s) const {
        if (stubs) lds_add(sig, s);
        done(kTurns - 1);
    }
};

template <int N, bool MULTI, bool MASK, bool STREAM, class Order>
__device__ __forceinline__ void adj_tile(const MaskRec<N> &M, uint32_t gaddr, uint32_t gbaddr, plane_t F,
                                         const Planes &Fall, plane_t Bn, plane_t Bc, const uint32_t (&off)[3], int u,
                                         uint32_t hb, bool start, const double (&tb)[3], double sg, double &sacc,
                                         const Order &order) {
    constexpr int NB = N - 1;
    const uint32_t ones = M.ones, twos = M.twos;
    const uint32_t cm = current_set(u, ones, twos);
    const uint32_t row = M.rb + hb;
    // only the open slots' child adjoints and the current slots' forward states
    // are loaded (wave-uniform branches around the loads)
    double a[3][N], f[3][NB];
#pragma unroll
    for (int w = 0; w < NB; ++w) {
        const uint32_t bit = 1u << w;
        const bool first = !(ones & bit);
        if (!(twos & bit)) {
            const uint32_t at = M.crb[w] + hb + ((!first && w < u) ? kTileB<N> : 0u) + w * kSlotB;
#pragma unroll
            for (int j = 0; j < 3; ++j) a[j][w] = slot_ld(Bn, off[j], at);
        } else {
#pragma unroll
            for (int j = 0; j < 3; ++j) a[j][w] = 0.0;
        }
    }
    tile_states<N, MULTI, MASK, STREAM>(f, M, cm, u, row, start, F, Fall, off);
    const double sgx = start ? 2.0 * sg : sg, sc = start ? 2.0 : 1.0;
#pragma unroll
    for (int w = 0; w < NB; ++w) {
        const uint32_t bit = 1u << w;
        if (!MASK && !((ones | twos) & bit)) {   // first visit
#pragma unroll
            for (int j = 0; j < 3; ++j) a[j][w] *= 2.0;
        }
        if (MASK && w == 0 && u == 0) {   // no extension onto the head point
#pragma unroll
            for (int j = 0; j < 3; ++j) a[j][w] = 0.0;
        }
        if ((ones & bit) && (cm & bit)) {   // shift edges
#pragma unroll
            for (int j = 0; j < 3; ++j) sacc = __builtin_fma(-sc * f[j][w], a[j][w], sacc);
        }
        // the close of this row feeds t_m: dS/dacc[u] gains W tbar
#pragma unroll
        for (int j = 0; j < 3; ++j) a[j][w] += w == u ? tb[j] : 0.0;   // (a branch here made the compiler spill)
    }
    const uint32_t need = (~twos | (1u << u)) & ((1u << NB) - 1u);   // w < b with a[w] != 0 possible
    asm volatile("" : "+v"(gaddr));
    asm volatile("" : "+v"(gbaddr));
    const lds_double *Gs = (const lds_double *)(uintptr_t)gaddr;
    lds_double *Gb = (lds_double *)(uintptr_t)gbaddr;
    // vertex b: adjoints of its slots in rows 2 and 1, which are the child
    // adjoints a[b] of rows 1 and 0
    const double gbb = Gs[(NB * N + NB) * 64];
    {
        double b2 = 0.0, b1 = 0.0;
#pragma unroll
        for (int w = 0; w < NB; ++w) {
            const double g = Gs[(NB * N + w) * 64];
            b2 = __builtin_fma(g, a[2][w], b2);
            b1 = __builtin_fma(g, a[1][w], b1);
        }
        b1 = __builtin_fma(gbb, b2, b1);
        b1 = __builtin_fma(-sg, b2, b1);   // the shift edge out of (m_b = 1, b)
        a[0][NB] = MASK ? b1 : 2.0 * b1;
        a[1][NB] = b2;
        a[2][NB] = 0.0;
    }
    // dS/dG[v][*] of the three rows
    auto add_row = [&](int v) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < N; ++w) {
            if (w < NB && !(need & (1u << w))) continue;   // wave-uniform
            double x = f[0][v] * a[0][w];
            x = __builtin_fma(f[1][v], a[1][w], x);
            if (w < NB) x = __builtin_fma(f[2][v], a[2][w], x);
            lds_add(Gb + (v * N + w) * 64, x);
        }
    };
    double c0 = 0.0, c1 = 0.0;   // f . G[.][b] of rows 0 and 1
#pragma unroll
    for (int v = 0; v < NB; ++v) {
        const uint32_t bit = 1u << v;
        if (!(cm & bit)) continue;   // wave-uniform
        double b[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int w = 0; w < N; ++w) {
            const double g = Gs[(v * N + w) * 64];
#pragma unroll
            for (int j = 0; j < 3; ++j) b[j] = __builtin_fma(g, a[j][w], b[j]);
            if (w == NB) {
                c0 = __builtin_fma(f[0][v], g, c0);
                c1 = __builtin_fma(f[1][v], g, c1);
            }
        }
        if (ones & bit) {
            // shift edge out of this slot: child adjoint, without the close term
#pragma unroll
            for (int j = 0; j < 3; ++j) b[j] = __builtin_fma(-sgx, (v == u) ? a[j][v] - tb[j] : a[j][v], b[j]);
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) state_st<STREAM>(Bc, off[j], row + v * kSlotB, b[j]);
        if (!Order::kDefer) add_row(v);
    }
    // the forward's slots with current b, formed again, and their row of dS/dG
    const double fb1 = MASK ? c0 : 2.0 * c0;
    const double fb2 = __builtin_fma(-sg, fb1, __builtin_fma(fb1, gbb, c1));
    sacc = __builtin_fma(-fb1, a[1][NB], sacc);   // its shift edge
    if (Order::kDefer) {
#pragma unroll
        for (int stage = 0; stage < kTurns; ++stage) {
            order.wait(stage);
#pragma unroll
            for (int v = first_row<N>(stage); v < NB && v < first_row<N>(stage + 1); ++v)
                if ((cm >> v) & 1u) add_row(v);
            if (stage < kTurns - 1) order.done(stage);
        }
    }
#pragma unroll
    for (int w = 0; w < N; ++w) {
        if (w < NB && !(need & (1u << w))) continue;
        double x = fb1 * a[1][w];
        if (w < NB) x = __builtin_fma(fb2, a[2][w], x);
        lds_add(Gb + (NB * N + w) * 64, x);
    }
    order.last(Gb + N * N * 64, sacc);
}

// the row of head b; tb: W times the adjoint of its close.  In special masks
// the cycle that opens there adds its own terms to dS/dG (its adjoint is formed
// by close_adjoint).
template <int N, bool MASK, bool STREAM, class Order>
__device__ __forceinline__ void adj_brow(const MaskRec<N> &M, uint32_t gaddr, uint32_t gbaddr, plane_t F,
                                         const Planes &Fall, plane_t Bn, plane_t Bc, uint32_t off, uint32_t hb, double tb,
                                         double sg, double &sacc, const Order &order) {
    constexpr int NB = N - 1;
    const uint32_t ones = M.ones, twos = M.twos;
    const uint32_t cm = (ones | twos) & ~1u;
    const uint32_t row = M.rb + hb;
    double a[N], f[NB];
    double fi = 0.0;
    if (special_mask(ones, twos)) fi = Fall.sum(off, row);
    const lds_double *Gs = brow_states<N, MASK, STREAM>(f, M, row, gaddr, F, Fall, off);
#pragma unroll
    for (int w = 0; w < NB; ++w) {
        const uint32_t bit = 1u << w;
        const bool first = !(ones & bit);
        a[w] = 0.0;
        if (!(twos & bit)) a[w] = slot_ld(Bn, off, M.crb[w] + hb + (first ? 0u : kTileB<N>) + w * 512u);
    }
    asm volatile("" : "+v"(gbaddr));
    lds_double *Gb = (lds_double *)(uintptr_t)gbaddr;
#pragma unroll
    for (int w = 0; w < NB; ++w) {
        const uint32_t bit = 1u << w;
        if (!MASK && !((ones | twos) & bit)) a[w] *= 2.0;
        if ((ones & bit) && (cm & bit)) sacc = __builtin_fma(-f[w], a[w], sacc);
    }
    a[NB] = tb;
#pragma unroll
    for (int stage = 0; stage < kTurns; ++stage) order.wait(stage);   // (a head-b row is short: it takes all turns at once)
#pragma unroll
    for (int v = 0; v < N; ++v) {
        const uint32_t bit = 1u << v;
        if (v < NB ? !(cm & bit) : !special_mask(ones, twos)) continue;
        if (v < NB) {
            double b = 0.0;
#pragma unroll
            for (int w = 0; w < N; ++w) b = __builtin_fma(Gs[(v * N + w) * 64], a[w], b);
            if (ones & bit) b = __builtin_fma(-sg, a[v < NB ? v : 0], b);
            state_st<STREAM>(Bc, off, row + v * 512u, b);
        }
        const double fv = v < NB ? f[v < NB ? v : 0] : fi;
#pragma unroll
        for (int w = 0; w < N; ++w)
            if (w == NB || !((twos >> w) & 1u)) lds_add(Gb + (v * N + w) * 64, fv * a[w]);   // wave-uniform
    }
#pragma unroll
    for (int stage = 0; stage < kTurns - 1; ++stage) order.done(stage);
    order.last(Gb + N * N * 64, sacc);
}

// W tbar of a mask's three rows.  Special masks: row 1 opens the cycle of head
// b, whose adjoint in flavour l is sum_w G_l[b][w] a_l[w] over the head-b row's
// outputs (the children's slots, its close); row 2 is the result at the full
// mask.  grow(l, w): G_l[b][w].
template <int N, bool MASK, class RowB>
__device__ __forceinline__ void close_adjoint(const MaskRec<N> &M, const Planes &Bn, const RowB &grow,
                                              const uint32_t (&off)[3], double W, double obar, double (&tb)[3]) {
    constexpr int NB = N - 1;
    const uint32_t ones = M.ones, twos = M.twos;
    tb[0] = tb[1] = tb[2] = 0.0;
    if (special_mask(ones, twos)) {
        const uint32_t brow = (1u + (uint32_t)__builtin_popcount(twos & ~1u)) * kTileB<N>;
        const bool full = twos == (1u << NB) - 1u;
        for (int k = 0; k < Bn.n; ++k) {
            const plane_t p = make_plane(Bn.base + k * Bn.stride);
#pragma unroll
            for (int w = 0; w < NB; ++w)
                if (!((twos >> w) & 1u))
                    tb[1] = __builtin_fma((MASK ? 1.0 : 2.0) * slot_ld(p, off[0], M.crb[w] + brow + w * 512u),
                                          grow(k, w), tb[1]);
            if (full) tb[1] = __builtin_fma(W * obar, grow(k, NB), tb[1]);
        }
        if (full) tb[2] = obar;
    } else {
        const int h = __builtin_ctz(ones);
        const uint32_t at = child_rows<N>(M, h) + open_slot<N>(h, twos);
        for (int k = 0; k < Bn.n; ++k) {
            if (MASK && h == 0 && k == 0) continue;
            const plane_t p = make_plane(Bn.base + k * Bn.stride);
#pragma unroll
            for (int j = 0; j < 3; ++j) tb[j] += slot_ld(p, off[j], at);
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) tb[j] *= W;
}

// the head slots [s0, s1) of a mask, backwards
template <int N, bool MULTI, bool MASK, bool STREAM, class Order>
__device__ __forceinline__ void adj_heads(const MaskRec<N> &M, uint32_t gaddr, uint32_t gbaddr, plane_t F,
                                          const Planes &Fall, plane_t Bn, plane_t Bc, const uint32_t (&off)[3], int lam,
                                          int s0, int s1, bool start, const double (&tb)[3], double sg, double &sacc,
                                          const Order &order) {
    const uint32_t twos = M.twos;
    const int nh = (twos & 1u) ? 1 + __builtin_popcount(twos & ~1u) : 1;
    uint32_t hs = (twos & 1u) ? (twos & ~1u) : 0u;   // heads >= 1, ascending
    for (int k = 1; k < s0; ++k) hs &= hs - 1u;
    for (int k = s0; k < s1 && k < nh; ++k) {
        int u = 0;
        if (k > 0) {
            u = __builtin_ctz(hs);
            hs &= hs - 1u;
        }
        if (!(MASK && empty_plane(u, lam, twos))) {
            adj_tile<N, MULTI, MASK, STREAM, Order>(M, gaddr, gbaddr, F, Fall, Bn, Bc, off, u, (uint32_t)k * kTileB<N>, start, tb,
                                             sg, sacc, order);
        } else {
#pragma unroll
            for (int stage = 0; stage < kTurns; ++stage) {
                order.wait(stage);
                order.done(stage);
            }
        }
    }
    if ((twos & 1u) && s1 > nh)   // the close of the head-b row feeds row 2
        adj_brow<N, MASK, STREAM, Order>(M, gaddr, gbaddr, F, Fall, Bn, Bc, off[0], (uint32_t)nh * kTileB<N>, tb[2], sg,
                                         sacc, order);
}

// A workgroup serves one group, one flavour and a block of masks.  Its
// wavefronts claim masks one at a time from an LDS counter, so that a wavefront
// that drew masks with few heads takes more.  On levels of few masks the items
// are (mask, head) pairs instead (A.row_items: blocks of mpb masks, their items
// listed in LDS), so that the heads of a mask run side by side.
template <int N, bool MULTI, bool MASK>
__global__ void __launch_bounds__(64 * kAdjWaves) level_adj_kernel(const LvlArgs A) {
    extern __shared__ double lds[];
    double *Gs_all = lds;                     // [N * N][64]  G of the flavour
    double *Gb_all = lds + N * N * 64;        // [N * N][64]  dS/dG of the flavour, this workgroup
    __shared__ int next_item, nlist;
    __shared__ uint16_t item_list[kAdjListMasks * N];
    const int lane = threadIdx.x & 63, wave = COS_RF(threadIdx.x >> 6);   // wave index: uniform
    const int wpb = blockDim.x >> 6;
    const DevPlan &P = A.plan;
    BlockAt at;
    if (!xcd_block(A, at)) return;
    const int nfs = MULTI ? A.nfs : 1, blk = at.x / nfs, lam = at.x - blk * nfs;
    const int blk0 = blk * A.mpb, nm = min(A.mpb, A.nmasks - blk0);
    const int gl = at.group, g = A.group0 + gl;
    // wave-uniform bases; the lane's word is added at each access; flavour planes
    const Planes Fall{A.F + gl * A.F_gstride + (int64_t)A.F_row0 * 64, A.F_frows * 64, nfs};
    const Planes Bn{A.cur + gl * A.cur_gstride, A.cur_frows * 64, nfs};   // level + 1
    double *Bc = A.nxt + gl * A.nxt_gstride;                               // level
    const uint32_t wl = work_lane(A, g, lane), lane8 = wl * 8u;
    const uint32_t off[3] = {lane8, lane8 + 512u, lane8 + 1024u};
    const double obar = A.out_bar[A.lane_cfg[g * 64 + wl]];
    const uint32_t gaddr = lds_addr(Gs_all) + lane8, gbaddr = lds_addr(Gb_all) + lane * 8u;
    const double *GT = A.GT + (int64_t)g * nfs * N * N * 64;
    const auto grow = [&](int l, int w) {
        return slot_ld(make_plane(GT + (l * N + N - 1) * N * 64), lane8, (uint32_t)w * 512u);
    };

    if (A.row_items && wave == 0) {
        const int n = list_items(item_list, P.mrec + (int64_t)(A.mask0 + blk0) * kRecInts, nm, lane);
        if (lane == 63) nlist = n;
    }
    if (threadIdx.x == 0) next_item = wpb;   // the first wpb items go to the waves in order
    for (int i = threadIdx.x; i < N * N * 64; i += blockDim.x) Gb_all[i] = 0.0;
    stage_slots(Gs_all, GT + lam * N * N * 64, N * N);
    __syncthreads();
    const double sg = A.stubs ? A.sigT[(int64_t)(g * nfs + lam) * 64 + wl] : 0.0;
    const plane_t FL = make_plane(Fall.base + lam * Fall.stride), BnL = make_plane(Bn.base + lam * Bn.stride),
                  BcL = make_plane(Bc + lam * (A.nxt_frows * 64));
    const int nitems = A.row_items ? COS_RF(nlist) : nm;
    double sacc = 0.0;
    bool any = false;
    for (int it = wave; it < nitems; it = claim(&next_item, lane)) {
        any = true;
        const int word = A.row_items ? COS_RF((int)item_list[it]) : it << 4, k = word & 15;
        const MaskRec<N> M = load_rec<N>(P, A.mask0 + blk0 + (word >> 4));
        double tb[3];
        close_adjoint<N, MASK>(M, Bn, grow, off, A.W, obar, tb);
        // this item's head slots: all of the mask's, or slot k alone
        adj_heads<N, MULTI, MASK, true, Unordered>(M, gaddr, gbaddr, FL, Fall, BnL, BcL, off, lam, A.row_items ? k : 0,
                                            A.row_items ? k + 1 : 16, A.level == 1, tb, sg, sacc, {});
    }
    if (A.stubs && any) atomicAdd(A.sbar_T + (int64_t)(g * nfs + lam) * 64 + lane, sacc);
    __syncthreads();
    double *__restrict__ gb = A.Gbar_T + (int64_t)(g * nfs + lam) * N * N * 64;
    const bool own = g * 64 + lane < A.count;
    for (int i = threadIdx.x; i < N * N * 64; i += blockDim.x) {
        const double x = Gb_all[i];   // (i's column is this lane's)
        if (x != 0.0 && own) atomicAdd(gb + i, x);
    }
}

// ---------------------------------------------------------------------------
// reverse, deterministic: the same tiles, with an order of summation that
// depends on nothing but the order n.  A level's masks are cut into parts (a mask
// each, or more where there are more than kDetParts); one workgroup takes one or
// several parts of one group and flavour, lists their (mask, head) items, deals
// them to its wavefronts in turn (item i to wavefront i mod kAdjWaves), and lets
// the items of a part add their dS/dG terms to the part's LDS accumulator in the
// order of the list (InTurn): everything else of a tile, 9/10 of its time, still
// overlaps with other tiles.  The accumulators are added to their parts' own
// slots of a partial buffer (no atomics: one workgroup per slot and level, the
// levels follow one another on the stream), and det_reduce_kernel sums the parts
// in order.
// Measured (n = 9, 1024 configurations, the reverse levels): 2.87 -> 1.76 ms
// against one wavefront per slot v, which read every child adjoint n times and
// kept one row of dS/dG in registers; 1.53 ms with three turns per item that
// order LDS accesses alone (1.54 with five, 1.58 with nine; the default reverse
// takes 1.00).  Eight loads in flight per thread where the accumulators are added
// to the partial buffer: the whole pass 2.17 -> 2.08 ms.
// ---------------------------------------------------------------------------
// first mask of part p
__device__ __forceinline__ int det_mask(const LvlArgs &A, int p) { return p * A.nmasks / A.det_parts; }

template <int N, bool MULTI, bool MASK>
__global__ void __launch_bounds__(64 * kAdjWaves) level_adj_det_kernel(const LvlArgs A) {
    extern __shared__ double lds[];
    double *Gs_all = lds, *Gb_all = lds + N * N * 64;   // G; per part dS/dG [N * N][64] and dS/dsigma [64]
    constexpr int kPart = (N * N + 1) * 64;
    __shared__ int turn[kDetPer][kTurns], nlist;
    __shared__ uint16_t item_list[kAdjListMasks * N];
    const int lane = threadIdx.x & 63, wave = COS_RF(threadIdx.x >> 6);   // wave index: uniform
    const DevPlan &P = A.plan;
    const int nfs = MULTI ? A.nfs : 1, blk0 = blockIdx.x / nfs, lam = blockIdx.x - blk0 * nfs;
    const int p0 = blk0 * A.det_per, np = min(A.det_per, A.det_parts - p0);
    const int lo = det_mask(A, p0), hi = det_mask(A, p0 + np);   // np > 1: at most kAdjListMasks masks
    const int gl = blockIdx.y, g = A.group0 + gl;
    const Planes Fall{A.F + gl * A.F_gstride + (int64_t)A.F_row0 * 64, A.F_frows * 64, nfs};
    const Planes Bn{A.cur + gl * A.cur_gstride, A.cur_frows * 64, nfs};   // level + 1
    double *Bc = A.nxt + gl * A.nxt_gstride;                               // level
    const uint32_t wl = work_lane(A, g, lane), lane8 = wl * 8u;
    const uint32_t off[3] = {lane8, lane8 + 512u, lane8 + 1024u};
    const double obar = A.out_bar[A.lane_cfg[g * 64 + wl]];
    const uint32_t gaddr = lds_addr(Gs_all) + lane8, gbaddr = lds_addr(Gb_all) + lane * 8u;
    const double *GT = A.GT + (int64_t)g * nfs * N * N * 64;
    const auto grow = [&](int l, int w) {
        return slot_ld(make_plane(GT + (l * N + N - 1) * N * 64), lane8, (uint32_t)w * 512u);
    };
    const plane_t FL = make_plane(Fall.base + lam * Fall.stride), BnL = make_plane(Bn.base + lam * Bn.stride),
                  BcL = make_plane(Bc + lam * (A.nxt_frows * 64));
    for (int i = threadIdx.x; i < np * kPart; i += blockDim.x) Gb_all[i] = 0.0;
    stage_slots(Gs_all, GT + lam * N * N * 64, N * N);
    const double sg = A.stubs ? A.sigT[(int64_t)(g * nfs + lam) * 64 + wl] : 0.0;
    for (int blk = lo; blk < hi; blk += kAdjListMasks) {
        __syncthreads();   // the previous block's list has been read
        if (wave == 0) {
            const int n = list_items(item_list, P.mrec + (int64_t)(A.mask0 + blk) * kRecInts, min(kAdjListMasks, hi - blk),
                                     lane);
            if (lane == 63) nlist = n;
            if (lane < kTurns) turn[0][lane] = 0;
            for (int j = 1; j < np; ++j) {   // the first turn of a part is that of its first item
                const int first = __shfl(n, det_mask(A, p0 + j) - lo - 1);
                if (lane < kTurns) turn[j][lane] = first;
            }
        }
        __syncthreads();
        const int nitems = COS_RF(nlist);
        for (int it = wave, j = 0; it < nitems; it += kAdjWaves) {
            const int word = COS_RF((int)item_list[it]), k = word & 15;
            while (j + 1 < np && (word >> 4) >= det_mask(A, p0 + j + 1) - lo) ++j;   // the item's part
            const MaskRec<N> M = load_rec<N>(P, A.mask0 + blk + (word >> 4));
            double tb[3], sacc = 0.0;   // (the shift terms go to the part's sums at the end of the item)
            close_adjoint<N, MASK>(M, Bn, grow, off, A.W, obar, tb);
            adj_heads<N, MULTI, MASK, true, InTurn>(M, gaddr, gbaddr + j * (kPart * 8), FL, Fall, BnL, BcL, off, lam, k, k + 1,
                                             A.level == 1, tb, sg, sacc, InTurn{(lds_int *)turn[j], it, A.stubs});
        }
    }
    __syncthreads();
    // the parts' slots of the partial sums (one workgroup per slot and level)
    for (int j = 0; j < np; ++j) {
        const int64_t slot = ((int64_t)(p0 + j) * A.det_groups + g) * nfs + lam;
        const double *gb = Gb_all + j * kPart;
        double *gp = A.Gbar_T + slot * N * N * 64;
        constexpr int kT = 64 * kAdjWaves, kU = 8;   // kU loads in flight per thread
        for (int i0 = threadIdx.x; i0 < N * N * 64; i0 += kU * kT) {
            double x[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) x[u] = i0 + u * kT < N * N * 64 ? gp[i0 + u * kT] : 0.0;
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (i0 + u * kT < N * N * 64) gp[i0 + u * kT] = x[u] + gb[i0 + u * kT];
        }
        if (A.stubs && wave == 0) A.sbar_T[slot * 64 + lane] += gb[N * N * 64 + lane];
    }
}

// sums the parts in order: GbT[i] = sum_p Gpart[p][i], sbT[g][l] = sum_p Spart[p][g][l]
__global__ void det_reduce_kernel(int parts, const double *__restrict__ Gpart, const double *__restrict__ Spart,
                                  int64_t gsize, int64_t ssize, double *__restrict__ GbT, double *__restrict__ sbT) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < gsize) {
        double x = 0.0;
#pragma unroll 8
        for (int p = 0; p < parts; ++p) x += Gpart[(int64_t)p * gsize + i];
        GbT[i] = x;
    }
    if (Spart && i < ssize) {   // i = (g * nfs + l) * 64 + lane
        const int64_t gl = i >> 6, lane = i & 63;
        double x = 0.0;
#pragma unroll 8
        for (int p = 0; p < parts; ++p) x += Spart[((int64_t)p * (ssize >> 6) + gl) * 64 + lane];
        sbT[i] = x;
    }
}

__global__ void zero_kernel(double *p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

__global__ void iota_kernel(int32_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = i;
}

// packed gradients -> caller layout
__global__ void unpack_kernel(const PackArgs A, const double *__restrict__ GbT, const double *__restrict__ sbT,
                              double *__restrict__ Gb, double *__restrict__ sb) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int N = A.n, nfs = A.nfs;
    const int64_t per_group = (int64_t)nfs * N * N * 64;
    if (i >= per_group * A.ngroups) return;
    const int lane = (int)(i & 63);
    int64_t rest = i >> 6;
    const int w = (int)(rest % N); rest /= N;
    const int v = (int)(rest % N); rest /= N;
    const int l = (int)(rest % nfs); rest /= nfs;
    const int g = (int)rest;
    const int slot = g * 64 + lane;
    if (slot >= A.count) return;
    const int c = A.order[slot];
    const int64_t off = A.Goff ? A.Goff[c] : (int64_t)c * A.nmat * N * N;
    Gb[off + ((int64_t)(A.variant ? l : 0) * N + v) * N + w] = GbT[i];
    if (v == 0 && w == 0 && sb) sb[(int64_t)c * A.nstub + (A.variant ? l : 0)] = sbT[((int64_t)g * nfs + l) * 64 + lane];
}

hipError_t launch_pack(const PackArgs &a, hipStream_t s) {
    const int64_t tot = (int64_t)a.ngroups * a.nfs * a.n * a.n * 64;
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_unpack(const PackArgs &a, const double *GbT, const double *sbT, double *Gb, double *sb,
                         hipStream_t s) {
    const int64_t tot = (int64_t)a.ngroups * a.nfs * a.n * a.n * 64;
    hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, a, GbT, sbT, Gb, sb);
    return hipGetLastError();
}

hipError_t launch_zero(double *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_iota(int32_t *p, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(iota_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// order 1: the start row (e_0, 0) and the row (m_0 = 2, 0) in closed form, one
// lane per configuration (forward, and with Gb the gradients in the packed
// layout).  F = t + G_l - 2 sigma_l with t = W sum_l G_l, S = W sum_l F_l G_l;
// mask-only: F lives on plane 1 alone and is t = W G_0.
// ---------------------------------------------------------------------------
__global__ void order1_kernel(const LvlArgs A, int nslots) {
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= nslots) return;
    const int cfg = A.lane_cfg[slot];
    if (cfg < 0) return;
    const int nfs = A.nfs, lane = slot & 63;
    const double *__restrict__ G = A.GT + (int64_t)(slot >> 6) * nfs * 64 + lane;
    const double *__restrict__ sig = A.stubs ? A.sigT + (int64_t)(slot >> 6) * nfs * 64 + lane : nullptr;
    double t = 0.0;
    for (int l = 0; l < (A.mask_only ? 1 : nfs); ++l) t += G[l * 64];
    t *= A.W;
    double s = 0.0, ft = 0.0;   // S / W; dS/dt / W
    for (int l = A.mask_only ? 1 : 0; l < nfs; ++l) {
        const double f = A.mask_only ? t : t + (G[l * 64] - (sig ? 2.0 * sig[l * 64] : 0.0));
        s = __builtin_fma(f, G[l * 64], s);
        ft += G[l * 64];
    }
    if (A.out) A.out[cfg] = A.W * s;
    if (!A.Gbar_T) return;
    const double ob = A.W * A.out_bar[cfg];
    double *__restrict__ Gb = A.Gbar_T + (int64_t)(slot >> 6) * nfs * 64 + lane;
    double *__restrict__ sb = A.sbar_T + (int64_t)(slot >> 6) * nfs * 64 + lane;
    for (int l = 0; l < nfs; ++l) {
        const double g = G[l * 64];
        if (A.mask_only) {
            Gb[l * 64] = l == 0 ? ob * A.W * ft : ob * t;
        } else {
            const double f = t + (g - (sig ? 2.0 * sig[l * 64] : 0.0));
            Gb[l * 64] = ob * (f + g + A.W * ft);
            if (sig) sb[l * 64] = -2.0 * ob * g;
        }
    }
}

hipError_t launch_order1(const LvlArgs &a, int ngroups, hipStream_t s) {
    hipLaunchKernelGGL(order1_kernel, dim3((unsigned)((ngroups * 64 + 255) / 256)), dim3(256), 0, s, a, ngroups * 64);
    return hipGetLastError();
}

// raise a kernel's dynamic-LDS limit when a launch needs more than 64 KB
static hipError_t allow_lds(const void *fn, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// LDS of a workgroup of the deterministic reverse: G, and per part the sums
size_t det_lds_bytes(int n, int per) { return ((size_t)n * n + per * ((size_t)n * n + 1)) * 512; }

hipError_t launch_level_det(const LvlArgs &a, int ngroups, hipStream_t s) {
    const int n = a.plan.n;
    const size_t shm = det_lds_bytes(n, a.det_per);
    if (a.det_per < 1 || a.det_per > kDetPer) return hipErrorInvalidValue;
    if (a.det_per > 1 && a.det_per * ((a.nmasks + a.det_parts - 1) / a.det_parts) > kAdjListMasks)
        return hipErrorInvalidValue;
    if (a.det_parts < 1 || a.det_parts > kDetParts) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((a.det_parts + a.det_per - 1) / a.det_per * a.nfs), (unsigned)ngroups), block(64 * kAdjWaves);
    switch (n) {
#define COS_DET_CASE(K)                                                                              \
    case K: {                                                                                        \
        void (*fn)(LvlArgs) = a.mask_only   ? level_adj_det_kernel<K, true, true>             \
                              : a.nfs > 1 ? level_adj_det_kernel<K, true, false>              \
                                          : level_adj_det_kernel<K, false, false>;            \
        hipError_t e = allow_lds((const void *)fn, shm);                                      \
        if (e != hipSuccess) return e;                                                        \
        hipLaunchKernelGGL(fn, grid, block, shm, s, a);                                       \
        break;                                                                                       \
    }
        COS_DET_CASE(2) COS_DET_CASE(3) COS_DET_CASE(4) COS_DET_CASE(5)
        COS_DET_CASE(6) COS_DET_CASE(7) COS_DET_CASE(8) COS_DET_CASE(9)
        COS_DET_CASE(10) COS_DET_CASE(11) COS_DET_CASE(12)
#undef COS_DET_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_det_reduce(int parts, const double *Gpart, const double *Spart, int64_t gsize, int64_t ssize,
                             double *GbT, double *sbT, hipStream_t s) {
    const int64_t tot = (Spart && ssize > gsize) ? ssize : gsize;
    if (tot <= 0) return hipSuccess;
    hipLaunchKernelGGL(det_reduce_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, parts, Gpart, Spart,
                       gsize, ssize, GbT, sbT);
    return hipGetLastError();
}

// the grid of xcd_block: gridx workgroups for each of the groups, padded to a
// multiple of 8
static dim3 xcd_grid(LvlArgs &a, int gridx, int ngroups) {
    a.gridx = gridx;
    a.ngroups = ngroups;
    return dim3((unsigned)(((int64_t)gridx * ngroups + 7) / 8 * 8));
}

hipError_t launch_level_adj(LvlArgs a, int ngroups, hipStream_t s) {
    const int n = a.plan.n, wpa = kAdjWaves;
    const size_t shm = 2 * (size_t)n * n * 64 * sizeof(double);
    if (a.row_items && a.mpb > kAdjListMasks) return hipErrorInvalidValue;
    const dim3 grid = xcd_grid(a, a.nblocks * a.nfs, ngroups);
    switch (n) {
#define COS_ADJ_CASE(K)                                                                           \
    case K: {                                                                                     \
        void (*fn)(LvlArgs) = a.mask_only   ? level_adj_kernel<K, true, true>              \
                              : a.nfs > 1 ? level_adj_kernel<K, true, false>               \
                                          : level_adj_kernel<K, false, false>;             \
        hipError_t e = allow_lds((const void *)fn, shm);                                   \
        if (e != hipSuccess) return e;                                                     \
        hipLaunchKernelGGL(fn, grid, dim3(64 * wpa), shm, s, a);                           \
        break;                                                                                    \
    }
        case 2:   // (other batches of order 2 run in one launch)
            if (a.nfs <= 2 || a.mask_only) return hipErrorInvalidValue;
            hipLaunchKernelGGL((level_adj_kernel<2, true, false>), grid, dim3(64 * wpa), shm, s, a);
            break;
        COS_ADJ_CASE(3) COS_ADJ_CASE(4) COS_ADJ_CASE(5)
        COS_ADJ_CASE(6) COS_ADJ_CASE(7) COS_ADJ_CASE(8) COS_ADJ_CASE(9)
        COS_ADJ_CASE(10) COS_ADJ_CASE(11) COS_ADJ_CASE(12)
#undef COS_ADJ_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// LDS of a forward workgroup: G, and the close sums of the heads of a split
// block (the last level's one mask: n head slots)
size_t fwd_lds_bytes(int n, int split_masks) { return ((size_t)n * n + 3 * (size_t)split_masks * n) * 512; }

hipError_t launch_level_fwd(LvlArgs a, int ngroups, int wpb, hipStream_t s) {
    const int n = a.plan.n;
    if (wpb < 1 || wpb > 16) return hipErrorInvalidValue;
    if (a.split && a.mpb > kSplitMasks) return hipErrorInvalidValue;
    const bool multi = a.nfs > 1;
    const bool last = a.level == 2 * (n - 1);
    const size_t shm = fwd_lds_bytes(n, last ? 1 : a.split ? a.mpb : 0);
    const dim3 grid = last ? dim3((unsigned)ngroups) : xcd_grid(a, a.nblocks * a.nfs, ngroups);
    const void *fn = nullptr;
    switch (n) {
#define COS_FWD_KERNEL(NAME, K)                                    \
    a.mask_only ? (const void *)NAME<K, true, true>                \
    : multi     ? (const void *)NAME<K, true, false>               \
                : (const void *)NAME<K, false, false>
#define COS_FWD_CASE(K)                                                                              \
    case K:                                                                                          \
        fn = last ? (COS_FWD_KERNEL(level_last_kernel, K)) : (COS_FWD_KERNEL(level_fwd_kernel, K));  \
        break;
        COS_FWD_CASE(2) COS_FWD_CASE(3) COS_FWD_CASE(4) COS_FWD_CASE(5)
        COS_FWD_CASE(6) COS_FWD_CASE(7) COS_FWD_CASE(8) COS_FWD_CASE(9)
        COS_FWD_CASE(10) COS_FWD_CASE(11) COS_FWD_CASE(12)
#undef COS_FWD_CASE
#undef COS_FWD_KERNEL
        default: return hipErrorInvalidValue;
    }
    hipError_t e = allow_lds(fn, shm);
    if (e != hipSuccess) return e;
    void *args[] = {(void *)&a};
    return hipLaunchKernel(fn, grid, dim3(64 * wpb), args, shm, s);
}

// ---------------------------------------------------------------------------
// small orders (2 <= n <= kSmallMax): a whole sweep in one launch
//
// At these orders a level of one group is at most a few dozen tiles, a launch
// per level costs more than the level's work (at n = 4 each launch ran 3-4 us
// for well under 1 us of work), and one group's states (0.25 MB for two levels
// at n = 5) stay in the caches.  So one workgroup of kSmallWaves wavefronts takes
// one group of 64 configurations through every level, with barriers instead of
// launches between them; it reads the caller's matrices and writes the
// caller's gradients itself, so that the packing, zeroing and unpacking
// launches go too.  G of every flavour stays in LDS, and in the reverse sweep
// the dS/dG accumulators beside it.
//
// The heads of a mask run side by side on different wavefronts: the forward
// works in rounds of at most kSmallItems (mask, head) items per flavour, whose
// close sums wait in LDS; after a barrier one wavefront per mask adds them up
// (heads in order, flavours in order, as the level kernels do, so that the sums
// agree bit for bit) and opens the next cycle.  The rounds come from a table
// made with the state tables (kSmallHeader and following).
//
// Measured, one flavour, 300 and 8192 configurations, against the level kernels:
// forward n = 4 26 / 28 -> 16 / 17 us, n = 5 43 / 54 -> 34 / 36 us; with the
// reverse n = 4 69 / 74 -> 32 / 34 us, n = 5 121 / 165 -> 79 / 95 us.  At n = 6
// one CU per group is too little (65 -> 96 us at 300 configurations, with the
// reverse 179 -> 334 us): the line lies at n = 5, and with three or more flavours
// at n = 4 for small batches.  At n <= 4 one launch took 0.26 to 0.86 of the level
// kernels' time for one to four flavours and 1 to 32768 configurations (forward of
// 100000 with one flavour: n = 2 21 us against 17, n = 3 42 and 39).
// ---------------------------------------------------------------------------
template <int N>
struct SmallCtx {
    const SmallArgs &A;
    cint32 *script;
    int nrounds, lane, wave, nfs, gl;
    uint32_t wl;             // as work_lane
    double *Gs, *Ts, *sig;   // LDS: G [nfs][N * N][64], close sums, shift weights [nfs][64]
    int cfg;
    uint32_t lane8;
    uint32_t off[3];
};

// states of level l: all levels kept (reverse sweep) or two windows
template <int N>
__device__ __forceinline__ double *small_level(const SmallCtx<N> &C, bool keep, int l, int64_t *plane) {
    if (keep) {
        *plane = C.A.plan.total_rows * 64;
        const cint32 *p = (const cint32 *)(C.A.plan.levels + l);
        return C.A.F + C.gl * C.A.F_gstride + (int64_t)p[0] * 64;
    }
    *plane = (int64_t)C.A.plan.max_rows * 64;
    return C.A.win + C.gl * C.A.win_gstride + (l & 1) * (*plane) * C.nfs;
}

// the workgroup's G (and shift weights) into LDS, straight from the caller's
// layout: the lanes of a wavefront read their own configurations' entries, and
// the lines they touch are used up within 16 entries
template <int N>
__device__ __forceinline__ void small_stage(const SmallCtx<N> &C) {
    const SmallArgs &A = C.A;
    const int n2 = C.nfs * N * N;
    const double *src = nullptr;
    if (C.cfg >= 0) src = A.G + (A.Goff ? A.Goff[C.cfg] : (int64_t)C.cfg * n2);
    const int wpb = blockDim.x >> 6;
    for (int e = C.wave; e < n2; e += wpb) C.Gs[e * 64 + C.lane] = src ? src[e] : 0.0;
    for (int l = C.wave; l < C.nfs; l += wpb)
        C.sig[l * 64 + C.lane] = (src && A.stub) ? A.stub[(int64_t)C.cfg * C.nfs + l] : 0.0;
}

// every forward level; writes S
template <int N, bool MULTI, bool MASK>
__device__ __forceinline__ void small_forward(const SmallCtx<N> &C, bool keep) {
    constexpr int NB = N - 1;
    const SmallArgs &A = C.A;
    const int wpb = blockDim.x >> 6, nfs = C.nfs, lane = C.lane;
    const cint32 *rounds = C.script + kSmallHeader, *items = rounds + C.nrounds * kSmallRoundInts;
    for (int r = 0; r < C.nrounds; ++r) {
        const cint32 *R = rounds + r * kSmallRoundInts;
        const int level = R[0], item0 = R[1], ni = R[2], close0 = R[3], nc = R[4];
        int64_t cpl, npl;
        double *cur = small_level<N>(C, keep, level, &cpl), *nxt = small_level<N>(C, keep, level + 1, &npl);
        const Planes all{cur, cpl, nfs};
        const bool start = level == 1;
        for (int q = C.wave; q < ni * nfs; q += wpb) {
            const int lam = q / ni, i = q - lam * ni;
            const uint32_t word = (uint32_t)items[item0 + i];
            const int k = (word >> 4) & 15, u = word & 15;
            const MaskRec<N> M = load_rec<N>(A.plan, (int)(word >> 8));
            const plane_t own = make_plane(cur + lam * cpl), nxtL = make_plane(nxt + lam * npl);
            const uint32_t gaddr = lds_addr(C.Gs + lam * N * N * 64) + C.lane8;
            const double sg = A.stub ? C.sig[lam * 64 + C.wl] : 0.0;
            double T[3] = {0.0, 0.0, 0.0}, dext[3] = {0.0, 0.0, 0.0};
            if (u == kSmallBrow) {
                T[2] = fwd_brow<N, MASK, false>(M, gaddr, own, all, nxtL, C.lane8, k * kTileB<N>, sg);
            } else if (!(MASK && empty_plane(u, lam, M.twos))) {
                fwd_tile<N, MULTI, MASK, false>(M, gaddr, own, all, nxtL, C.off, u, k * kTileB<N>, start, sg, T, dext);
            }
            if (!(M.twos & 1u)) {   // the mask's only head
                close_mask<N, MULTI, MASK>(M, A.W, own, nxtL, C.off, T, dext);
                continue;
            }
            double *t = C.Ts + (lam * kSmallItems + i) * 192 + lane;
#pragma unroll
            for (int j = 0; j < 3; ++j) t[j * 64] = T[j];
        }
        __syncthreads();
        // one wavefront per mask and flavour: W sum over its heads
        for (int q = C.wave; q < nc * nfs; q += wpb) {
            const int lam = q / nc, c = q - lam * nc;
            const uint32_t word = (uint32_t)items[close0 + c];
            const int first = (word >> 4) & 15, cnt = word & 15;
            const MaskRec<N> M = load_rec<N>(A.plan, (int)(word >> 8));
            if (!(M.twos & 1u)) continue;
            double T[3] = {0.0, 0.0, 0.0};
            const double dext[3] = {0.0, 0.0, 0.0};
            for (int i = first; i < first + cnt; ++i) {
                const double *t = C.Ts + (lam * kSmallItems + i) * 192 + lane;
#pragma unroll
                for (int j = 0; j < 3; ++j) T[j] += t[j * 64];
            }
            const plane_t own = make_plane(cur + lam * cpl), nxtL = make_plane(nxt + lam * npl);
            close_mask<N, MULTI, MASK>(M, A.W, own, nxtL, C.off, T, dext);
        }
        if (level == 2 * NB && C.wave == 0) {
            // the full mask: S / W, as level_last_kernel adds it up
            double T1 = 0.0, T2 = 0.0, gbb = 0.0;
            for (int lam = 0; lam < nfs; ++lam) {
                double s1 = 0.0, s2 = 0.0;
                for (int i = 0; i < ni; ++i) {
                    const double *t = C.Ts + (lam * kSmallItems + i) * 192 + lane;
                    s1 += t[64];
                    s2 += t[128];
                }
                T1 += A.W * s1;
                T2 += s2;
                gbb += C.Gs[(lam * N * N + NB * N + NB) * 64 + lane];
            }
            if (C.cfg >= 0 && A.out) A.out[C.cfg] = A.W * __builtin_fma(T1, gbb, T2);
        }
        __syncthreads();
    }
}

template <int N>
__device__ __forceinline__ SmallCtx<N> small_ctx(const SmallArgs &A, double *lds, uint32_t tail_doubles) {
    const int lane = threadIdx.x & 63, wave = COS_RF(threadIdx.x >> 6), g = A.group0 + (int)blockIdx.x;
    cint32 *script = (cint32 *)A.plan.script;
    const int slot = g * 64 + lane;
    const uint32_t wl = slot < A.count ? lane : 0, lane8 = wl * 8u;
    double *Ts = lds + (int64_t)A.nfs * N * N * 64;
    return SmallCtx<N>{A,  script, (int)script[0], lane, wave, A.nfs, (int)blockIdx.x, wl,
                       lds, Ts, Ts + tail_doubles, slot < A.count ? A.order[slot] : -1,
                       lane8, {lane8, lane8 + 512u, lane8 + 1024u}};
}

template <int N, bool MULTI, bool MASK>
__global__ void __launch_bounds__(64 * kSmallWaves) small_fwd_kernel(const SmallArgs A) {
    extern __shared__ double lds[];
    const SmallCtx<N> C = small_ctx<N>(A, lds, (uint32_t)A.nfs * kSmallItems * 192u);
    small_stage<N>(C);
    __syncthreads();
    small_forward<N, MULTI, MASK>(C, false);
}

// forward (every level kept) and reverse; writes S, dS/dG and dS/dsigma.  The
// accumulators take the place of the forward's close sums in LDS.  Both run in
// one launch; to be timed apart, in two (A.parts).
template <int N, bool MULTI, bool MASK>
__global__ void __launch_bounds__(64 * kSmallWaves) small_adj_kernel(const SmallArgs A) {
    constexpr int NB = N - 1;
    extern __shared__ double lds[];
    const uint32_t tail = (uint32_t)A.nfs * 64u * (N * N > 3 * kSmallItems ? N * N : 3 * kSmallItems);
    const SmallCtx<N> C = small_ctx<N>(A, lds, tail);
    const int wpb = blockDim.x >> 6, nfs = C.nfs, lane = C.lane;
    double *Gb = C.Ts, *sb = C.sig + nfs * 64;
    small_stage<N>(C);
    __syncthreads();
    if (A.parts & kSmallForward) small_forward<N, MULTI, MASK>(C, true);
    if (!(A.parts & kSmallReverse)) return;
    const int n2 = nfs * N * N;
    for (int e = C.wave; e < n2; e += wpb) Gb[e * 64 + lane] = 0.0;
    for (int l = C.wave; l < nfs; l += wpb) sb[l * 64 + lane] = 0.0;
    __syncthreads();
    const double obar = A.out_bar[A.order[(A.group0 + C.gl) * 64 + (int)C.wl]];
    const cint32 *items = C.script + kSmallHeader + C.nrounds * kSmallRoundInts, *lev = items + C.script[1];
    for (int l = 2 * NB; l >= 1; --l) {
        int64_t fpl, cpl, npl;
        const double *F = small_level<N>(C, true, l, &fpl);
        const double *B1 = small_level<N>(C, false, l + 1, &cpl);
        double *Bc = small_level<N>(C, false, l, &npl);
        const Planes Fall{F, fpl, nfs}, Bn{B1, cpl, nfs};
        const int item0 = lev[2 * l], ni = lev[2 * l + 1];
        for (int q = C.wave; q < ni * nfs; q += wpb) {
            const int lam = q / ni;
            const uint32_t word = (uint32_t)items[item0 + (q - lam * ni)];
            const int k = (word >> 4) & 15;
            const MaskRec<N> M = load_rec<N>(A.plan, (int)(word >> 8));
            const uint32_t gaddr = lds_addr(C.Gs + lam * N * N * 64) + C.lane8;
            const uint32_t gbaddr = lds_addr(Gb + lam * N * N * 64) + lane * 8u;
            const double sg = A.stub ? C.sig[lam * 64 + C.wl] : 0.0;
            double sacc = 0.0, tb[3];
            close_adjoint<N, MASK>(M, Bn, [&](int l, int w) { return C.Gs[((l * N + N - 1) * N + w) * 64 + C.wl]; }, C.off, A.W,
                                   obar, tb);
            adj_heads<N, MULTI, MASK, false, Unordered>(M, gaddr, gbaddr, make_plane(F + lam * fpl), Fall,
                                                 make_plane(B1 + lam * cpl), make_plane(Bc + lam * npl), C.off, lam, k,
                                                 k + 1, l == 1, tb, sg, sacc, {});
            if (A.stub) atomicAdd(sb + lam * 64 + lane, sacc);
        }
        __syncthreads();
    }
    if (C.cfg < 0) return;
    double *out = A.G_bar + (A.Goff ? A.Goff[C.cfg] : (int64_t)C.cfg * n2);
    for (int e = C.wave; e < n2; e += wpb) out[e] = Gb[e * 64 + lane];
    if (A.stub)
        for (int l = C.wave; l < nfs; l += wpb) A.stub_bar[(int64_t)C.cfg * nfs + l] = sb[l * 64 + lane];
}

size_t small_lds_bytes(int n, int nfs, bool reverse) {
    const size_t tail = reverse && n * n > 3 * kSmallItems ? (size_t)n * n : (size_t)3 * kSmallItems;
    return (size_t)nfs * 512 * (n * n + tail + (reverse ? 2 : 1));
}

hipError_t launch_small(const SmallArgs &a, bool reverse, int ngroups, hipStream_t s) {
    const size_t shm = small_lds_bytes(a.plan.n, a.nfs, reverse);
    const dim3 grid((unsigned)ngroups), block(64 * kSmallWaves);
    void (*fn)(SmallArgs) = nullptr;
    switch (a.plan.n) {
#define COS_SMALL_CASE(K)                                                                            \
    case K:                                                                                          \
        fn = reverse ? (a.mask_only ? small_adj_kernel<K, true, true>                                \
                        : a.nfs > 1 ? small_adj_kernel<K, true, false> : small_adj_kernel<K, false, false>)\
                     : (a.mask_only ? small_fwd_kernel<K, true, true>                                \
                        : a.nfs > 1 ? small_fwd_kernel<K, true, false> : small_fwd_kernel<K, false, false>);\
        break;
        COS_SMALL_CASE(2) COS_SMALL_CASE(3) COS_SMALL_CASE(4) COS_SMALL_CASE(5)
#undef COS_SMALL_CASE
        default: return hipErrorInvalidValue;
    }
    hipError_t e = allow_lds((const void *)fn, shm);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fn, grid, block, shm, s, a);
    return hipGetLastError();
}

}  // namespace libcos

// Fused limited LBGK step kernels for gfx950.
//
// Compiled once per population storage type (LBM_ST = 0..3).  A D2Q9 time
// step of every domain is one launch of the collision kernel and, when a
// limiter needs more than the node itself, one launch of the second pass
// (small domains take k_block2d, which does both, D1Q3 k_step1d):
//
//  collision: one thread per node, one workgroup per 256 consecutive nodes in
//    row-major order, so the whole grid streams through
//    a narrow band of rows at a time.  Free flight (pull form, read from
//    buffer `parity`), moments, f*, the collision (LBGK, or ELBM in its own
//    instantiation), Delta S', the trimming and positivity factors (they
//    depend on the node alone), and the store of the limited post-collision
//    state into the other buffer.  With the median filter or an
//    ensemble-dependent limiter on, Delta S' also goes to a plane of its own.
//    In steps whose sums may be read (the last of a captured sequence) each
//    workgroup leaves one partial of the reduction terms; the FP64 global sums
//    are formed from these on demand, when the stats are read.
//  second pass: the 3x3 median of that plane and the ensemble-dependent
//    factors (thresholds from this step's E(Delta S') and selections) decide
//    which nodes move further; after LBGK these are formed anew from the step's
//    input, after ELBM (whose f' needs the node's root) and far beyond the
//    last-level cache their stored limited states are rescaled in place.
//
// The collision kernel is a plain streaming pass with aligned loads and
// stores and no barrier before its epilogue, the access pattern that
// sustains the highest HBM bandwidth on this part.
#include <type_traits>

#include "lbm_device.h"

#ifndef LBM_ST
#define LBM_ST 1
#endif
#if LBM_ST == 0
using StT = double;
#define LBM_SUFFIX st0
#elif LBM_ST == 1
using StT = float;
#define LBM_SUFFIX st1
#elif LBM_ST == 2
using StT = _Float16;
#define LBM_SUFFIX st2
#else
using StT = __bf16;
#define LBM_SUFFIX st3
#endif
#define LBM_CAT2(a, b) a##_##b
#define LBM_CAT(a, b) LBM_CAT2(a, b)

namespace lbm {

// node classes of the cavity (Sec. 4.4.1): walls x = 0, x = nx-1, y = 0
// (corners included), lid y = ny-1, fluid elsewhere
enum { kNodeFluid = 0, kNodeWall = 1, kNodeLid = 2, kNodeNone = 3 };

template <int BC>
__device__ inline int node_class(int x, int y, int nx, int ny)
{
    if constexpr (BC != kCavity) {
        return kNodeFluid;
    } else {
        if (x == 0 || x == nx - 1 || y == 0) return kNodeWall;
        if (y == ny - 1) return kNodeLid;
        return kNodeFluid;
    }
}

// spatial tile of a workgroup: blocks are spread over the XCDs so that each
// XCD runs one contiguous stretch of tiles (rows sharing halo lines hit the
// same L2).  `first` is the block id of tile 0.
__device__ inline int tile_of_block(const StepArgs& a, int first)
{
    return xcd_spatial(int(blockIdx.x) - first, a.ntiles);
}

// FP64 partials: set 0 = the collision kernel's, per group (summed on demand; the
// D1Q3 kernel writes them per workgroup), set 1 = second pass, per tile (and every
// partial of the fused step and of the tile kernel)
__device__ inline double* partial_slot(const StepArgs& a, int set, int tile)
{
    return a.partials + ((long long)set * a.pstride + tile) * kNStat;
}

// The node of a thread of the collision kernel and of k_form2d: 64 consecutive
// nodes per wave.  `inner` (uniform in the wave) when all of them lie in rows
// 1 .. ny - 2 of a domain at least 64 wide, so that every neighbour is at a
// fixed distance (up to the wrap of the columns); the rest is the first and
// last rows and very narrow domains.
struct Node {
    unsigned n;
    int x, y;
    bool in, inner;
};
__device__ __forceinline__ Node node_of(const DomainDev& D, int block)
{
    const int nx = D.nx, ny = D.ny;
    const unsigned all = unsigned(nx) * unsigned(ny);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
    const unsigned nw = unsigned(block) * kThreads + unsigned(wave) * kWave;
    Node r;
    r.n = nw + (threadIdx.x & (kWave - 1));
    r.in = r.n < all;
    if (nx >= kWave) {
        const int yw = row_of_node(nw, nx, D.inv_nx);
        r.x = int(nw - unsigned(yw) * unsigned(nx)) + int(threadIdx.x & (kWave - 1));
        const bool next = r.x >= nx;
        r.x -= next ? nx : 0;
        r.y = yw + (next ? 1 : 0);
        r.inner = yw > 0 && nw + kWave <= all - unsigned(nx);
    } else {
        r.y = int(r.n / unsigned(nx));
        r.x = int(r.n - unsigned(r.y) * unsigned(nx));
        r.inner = false;
    }
    return r;
}

// trimming factor of one node (it depends on the node alone, Sec. 3.2/3.4)
template <class A, class DD>
__device__ __forceinline__ A trim_phi(const DD& D, A dpost, unsigned& mask)
{
    A phi = A(1);
    if ((D.limiter & kLimTrim) && dpost > A(D.delta_trim)) {
        mask |= kMaskTrim;
        phi = D.trim_mode ? A(0) : sqrt_(A(D.delta_trim) * rcp(dpost));
    }
    return phi;
}

// Columns of one thread: pull sources of movers with vx = +1, 0, -1 as byte
// offsets (periodic wrap), and the thread's own column.
template <class T, int BC>
struct Cols {
    unsigned m, c, p, own;
    int x;
    __device__ Cols(int x_, int nx) : x(x_)
    {
        constexpr unsigned es = sizeof(T);
        if constexpr (BC == kPeriodic) {
            m = es * unsigned(x == 0 ? nx - 1 : x - 1);
            p = es * unsigned(x == nx - 1 ? 0 : x + 1);
        } else {
            m = es * unsigned(x - 1);
            p = es * unsigned(x + 1);
        }
        c = es * unsigned(x);
        own = c;
    }
};

// pull free flight of node (x, y): population i arriving there left
// (x - vx, y - vy); off a non-periodic edge it is the node's own opposite
// population (reflection: free flight stays a permutation)
template <int BC, class T>
__device__ __forceinline__ void gather2d(gptr<const T> src, long long plane, int nx, int ny, const Cols<T, BC>& cl,
                                         int y, typename Store<T>::A (&g)[9])
{
    using L = Lat<kD2Q9>;
    if constexpr (BC == kPeriodic) {
        const long long r0 = (long long)y * nx;
        const long long rm = (long long)(y == 0 ? ny - 1 : y - 1) * nx;
        const long long rp = (long long)(y == ny - 1 ? 0 : y + 1) * nx;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const long long rs = L::vy(i) > 0 ? rm : (L::vy(i) < 0 ? rp : r0);
            const unsigned cs = L::vx(i) > 0 ? cl.m : (L::vx(i) < 0 ? cl.p : cl.c);
            g[i] = Store<T>::ld(at_bytes(src + (i * plane + rs), cs));
        }
    } else {
        // A wave covers one row (callers keep it so), so the source rows are
        // scalars, clamped at the domain's edges like the lanes' columns; the
        // loads are then those of the periodic case.  A source off the domain
        // (at wall and lid nodes only) is replaced by the node's own opposite
        // population, loaded afterwards for those lanes alone.
        const int yw = __builtin_amdgcn_readfirstlane(y);
        const long long r0 = (long long)yw * nx;
        const long long rm = yw > 0 ? r0 - nx : r0;
        const long long rp = yw < ny - 1 ? r0 + nx : r0;
        constexpr unsigned es = sizeof(T);
        const int x = cl.x;
        const unsigned cc = es * unsigned(x);
        const unsigned cm = x > 0 ? cc - es : cc;
        const unsigned cp = x < nx - 1 ? cc + es : cc;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const long long rs = L::vy(i) > 0 ? rm : (L::vy(i) < 0 ? rp : r0);
            const unsigned cs = L::vx(i) > 0 ? cm : (L::vx(i) < 0 ? cp : cc);
            g[i] = Store<T>::ld(at_bytes(src + (i * plane + rs), cs));
        }
        const bool xm = x > 0, xp = x < nx - 1, ym = yw > 0, yp = yw < ny - 1;
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const bool in = (L::vx(i) > 0 ? xm : (L::vx(i) < 0 ? xp : true)) &&
                            (L::vy(i) > 0 ? ym : (L::vy(i) < 0 ? yp : true));
            if (!in) g[i] = Store<T>::ld(at_bytes(src + (L::opp(i) * plane + r0), cc));
        }
    }
}

// The same into the node of a thread (Node): in inner waves the nine sources
// are three lane offsets (columns x - 1, x, x + 1) on scalar bases, else they
// are computed per lane.
template <int BC, class T>
__device__ __forceinline__ void gather_at(gptr<const T> src, long long plane, int nx, int ny, const Node& v,
                                          typename Store<T>::A (&g)[9])
{
    using L = Lat<kD2Q9>;
    constexpr unsigned es = sizeof(T);
    const int x = v.x, y = v.y;
    const bool xm = x > 0, xp = x < nx - 1;
    const unsigned c = es * v.n;
    if (v.inner) {
        unsigned m = c - es, p = c + es;
        if constexpr (BC == kPeriodic) {
            m += xm ? 0u : es * unsigned(nx);
            p -= xp ? 0u : es * unsigned(nx);
        }
        // (at a cavity's side walls these are the neighbouring rows' ends)
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const long long up = L::vy(i) > 0 ? -(long long)nx : (L::vy(i) < 0 ? (long long)nx : 0);
            g[i] = Store<T>::ld(at_bytes(src + (i * plane + up), L::vx(i) > 0 ? m : (L::vx(i) < 0 ? p : c)));
        }
    } else {
        int left = x - 1, right = x + 1, below = y - 1, top = y + 1;
        if constexpr (BC == kPeriodic) {
            left = xm ? left : nx - 1;
            right = xp ? right : 0;
            below = y > 0 ? below : ny - 1;
            top = y < ny - 1 ? top : 0;
        } else {
            left = xm ? left : 0;
            right = xp ? right : x;
            below = y > 0 ? below : 0;
            top = y < ny - 1 ? top : y;
        }
        const unsigned r0 = unsigned(y) * unsigned(nx), rm = unsigned(below) * unsigned(nx), rp = unsigned(top) * unsigned(nx);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const unsigned at = (L::vy(i) > 0 ? rm : (L::vy(i) < 0 ? rp : r0)) +
                                unsigned(L::vx(i) > 0 ? left : (L::vx(i) < 0 ? right : x));
            g[i] = Store<T>::ld(at_bytes(src + i * plane, es * at));
        }
    }
    if constexpr (BC != kPeriodic) {
        // a source off the domain (at wall and lid nodes only): the node's own
        // opposite population
        const bool ym = y > 0, yp = y < ny - 1;
        if (!(xm && xp && ym && yp)) {
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const bool in = (L::vx(i) > 0 ? xm : (L::vx(i) < 0 ? xp : true)) &&
                                (L::vy(i) > 0 ? ym : (L::vy(i) < 0 ? yp : true));
                if (!in) g[i] = Store<T>::ld(at_bytes(src + L::opp(i) * plane, c));
            }
        }
    }
}

// Mass and momentum of a wall or lid node's nine populations in FP64 (its
// share of the stats), in population order; each population enters the
// momentum sums only where its velocity component is nonzero.
template <class A>
__device__ __forceinline__ void moments_fp64(const A (&g)[9], double& dr, double& jx, double& jy)
{
    using L = Lat<kD2Q9>;
    dr = 0.0;
    jx = 0.0;
    jy = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double v = double(g[i]);
        dr += v;
        if (L::vx(i) > 0) jx += v;
        if (L::vx(i) < 0) jx -= v;
        if (L::vy(i) > 0) jy += v;
        if (L::vy(i) < 0) jy -= v;
    }
}

// STREAM: the nontemporal hint, for a wave whose 64 lanes write one whole
// aligned piece; a wave that writes a segment sharing its end sectors
// with another wave's (the fused step) stores plainly, so that L2 merges the
// two halves of a sector before it goes to HBM
template <class T, bool STREAM = true>
__device__ __forceinline__ void store_limited(gptr<T> dst, long long plane, long long row, unsigned own,
                                              const SiteState<kD2Q9, typename Store<T>::A>& S,
                                              typename Store<T>::A phi, typename Store<T>::A c)
{
    using A = typename Store<T>::A;
    const A k = phi * c;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        if constexpr (STREAM) Store<T>::st_stream(at_bytes(dst + (i * plane + row), own), S.gs[i] - k * S.d[i]);
        else Store<T>::st(at_bytes(dst + (i * plane + row), own), S.gs[i] - k * S.d[i]);
    }
}

// What leaves a wall or lid node (no collision).  Bounce-back: every population
// reversed.  Lid: f*(rho0, (u0, 0)).  Diffusive Maxwell walls (Sec. 4.4.2, the
// lid moves with (u0, 0), corners reflect): the populations pointing into the
// fluid become gamma f*_i(1, u_wall), gamma = (mass that arrived from the fluid)
// / (mass of those f*_i), the others keep what free flight brought.
template <int QE, class A, class DD>
__device__ __forceinline__ void wall_state(const DD& D, int cls, int x, int y, int nx, int ny, const A (&g)[9], A shift,
                                           A (&out)[9])
{
    using L = Lat<kD2Q9>;
    const bool corner = (x == 0 || x == nx - 1) && (y == 0 || y == ny - 1);
    if (D.diffusive && !corner) {
        const int my = y == 0 ? 1 : (y == ny - 1 ? -1 : 0);
        const int mx = my != 0 ? 0 : (x == 0 ? 1 : -1);
        A E[9] = {A(0), A(0), A(0), A(0), A(0), A(0), A(0), A(0), A(0)};    // a resting wall's f* is w_i
        if (y == ny - 1) eq_excess<kD2Q9, QE>(A(D.lid_ux), A(0), E);
        A sum_in = A(0), sum_arrived = A(0);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int d = L::vx(i) * mx + L::vy(i) * my;
            if (d > 0) sum_in += A(L::w(i)) * (A(1) + E[i]);
            if (d < 0) sum_arrived += A(L::w(i)) * shift + g[i];
        }
        const A gamma = sum_arrived / sum_in;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int d = L::vx(i) * mx + L::vy(i) * my;
            out[i] = d > 0 ? gamma * (A(L::w(i)) * (A(1) + E[i])) - A(L::w(i)) * shift : g[i];
        }
    } else if (cls == kNodeWall) {
#pragma unroll
        for (int i = 0; i < 9; ++i) out[i] = g[L::opp(i)];
    } else {
        A E[9];
        eq_excess<kD2Q9, QE>(A(D.lid_ux), A(0), E);
        const A r0 = A(D.rho0);
#pragma unroll
        for (int i = 0; i < 9; ++i) out[i] = A(L::w(i)) * ((r0 - shift) + r0 * E[i]);
    }
}

// The exact homothety of a node to Delta S = t as a real call (its root solve,
// needed by few nodes, would otherwise sit in the middle of every kernel).  The
// state goes by value: a caller's own copy then stays in registers.
template <class A>
__device__ __attribute__((noinline)) A exact_homothety_call(SiteState<kD2Q9, A> o, A shift, A t)
{
    return exact_homothety<kD2Q9>(o, shift, t, o.dpost);
}

// STATS: a step whose sums will be read.  The others (63 of 64 in a long run)
// leave the sums out, and with them a third of the instructions, the barrier
// and the partial at the end of every workgroup.
template <class T, int QE, int DS, int BC, bool ELBM, bool STATS>
__global__ void __launch_bounds__(kThreads, DS == kExact && !STATS && !ELBM ? 4 : 1) k_collide2d(StepArgs a)
{
    using A = typename Store<T>::A;
    constexpr int Q = 9;
    __shared__ double red[STATS ? 4 * kNStat : 1];
    // one node per thread, kThreads consecutive nodes per workgroup
    const Block t = a.blocks ? a.blocks[blockIdx.x] : Block{0, int(blockIdx.x)};
    const DomainDev& D = a.dom[t.domain];
    const int nx = D.nx, ny = D.ny;
    const long long plane = D.plane;
    const gptr<const T> src = to_global<T>(static_cast<const void*>(D.buf[a.parity]));
    const gptr<T> dst = to_global<T>(D.buf[1 - a.parity]);
    const gptr<A> dsb = to_global<A>(D.dsbuf);
    const A shift = A(D.shift), c = A(D.c);
    const bool record = STATS && (a.flags & kFlagRecord);
    const bool want_ent = STATS && (a.flags & kFlagEntropy);
    const bool keep_ds = D.limiter & (kLimMedian | kLimEns);
    const bool dense = !ELBM && D.dense;       // k_form2d stores the fluid nodes
    const long long step = a.counter[a.parity];
    // the index of the next step, read by the next launch (which reads buffer 1 - parity)
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counter[1 - a.parity] = step + 1;

    // The ensemble limiters and the GATE reading of the median use every
    // Delta S'.  The FLOOR median only needs the values above delta: its
    // threshold max(median, delta) and its decision are unchanged when every
    // value at or below delta is replaced by 0.  So there a wave with no node
    // above delta stores nothing, and the median pass reads its 64 nodes as
    // zeros (a.above records which waves stored).
    const bool every = (D.limiter & kLimEns) || D.median_mode != 0;
    AccT<A> acc;
    bool any_up = false;       // a fluid node of the wave is a median candidate
    const Node v = node_of(D, t.first);
    {
        const int x = v.x, y = v.y;
        const unsigned node = v.n, own = unsigned(sizeof(T)) * v.n;
        if (v.in) {
            A g[Q];
            gather_at<BC>(src, plane, nx, ny, v, g);
            const int cls = node_class<BC>(x, y, nx, ny);
            if (cls == kNodeFluid) {
                SiteState<kD2Q9, A> S;
                SiteScalars sc;
                collide_site<kD2Q9, QE, DS, ELBM>(g, shift, c, S, sc, STATS);
                if constexpr (STATS) {
                    acc.moments(sc);
                    acc.fluid_site(sc, S.dpost);
                }
                if (want_ent) {
                    const double e = entropy_site<kD2Q9>(g, shift);
                    if (isfinite(e)) acc.ent += A(e);
                }
                if (x == D.probe_x && y == D.probe_y) {
                    const gptr<float> p = to_global<float>(D.probe) + 2 * (step % D.probe_cap);
                    p[0] = sc.ux;
                    p[1] = sc.uy;
                }
                unsigned mask = 0;
                A phi = trim_phi(D, S.dpost, mask);
                if constexpr (DS == kExactHom) {
                    if (D.homothety && (mask & kMaskTrim) && !D.trim_mode && isfinite(S.dpost))
                        phi = exact_homothety_call(S, shift, A(D.delta_trim));
                }
                if (S.posrule) {
                    mask |= kMaskPos;
                    if constexpr (STATS) ++acc.pos;
                }
                if (D.limiter & kLimPos) {
                    const A pp = positivity_phi<kD2Q9>(S, shift);
                    if (pp < A(1)) {
                        mask |= kMaskPos;
                        if constexpr (STATS) ++acc.pos;
                        phi = fmin(phi, pp);
                    }
                }
                if (!dense) store_limited<T>(dst, plane, 0, own, S, phi, S.c);
                if (keep_ds) {
                    // NaN counts as above: such a wave always stores its values
                    const bool up = (D.limiter & kLimMedian) && !(S.dpost <= A(D.delta_median));
                    any_up = __ballot(up) != 0;
                    if (every || any_up) Store<A>::st(dsb + node, S.dpost);
                }
                if constexpr (STATS) {
                    if (mask & kMaskTrim) ++acc.trim;
                    if (phi < A(1) && isfinite(S.dpost))
                        acc.lim += S.dpost - delta_s_scaled<kD2Q9, DS>(S, shift, S.c, phi);
                    if (sc.nonpos) mask |= kMaskNonpos;
                }
                if (record) {
                    to_global<unsigned char>(D.mask)[node] = (unsigned char)mask;
                    to_global<double>(D.dS)[node] = double(S.dpost);
                }
            } else {
                A out[Q];
                wall_state<QE>(D, cls, x, y, nx, ny, g, shift, out);
#pragma unroll
                for (int i = 0; i < Q; ++i) Store<T>::st(at_bytes(dst + i * plane, own), out[i]);
                if constexpr (STATS) {
                    SiteScalars sc;
                    moments_fp64(g, sc.dr, sc.jx, sc.jy);
                    acc.moments(sc);
                }
                if (record) {
                    to_global<unsigned char>(D.mask)[node] = (unsigned char)kMaskNotFluid;
                    to_global<double>(D.dS)[node] = 0.0;
                }
            }
        }
    }
    const int wave = int(threadIdx.x) / kWave;
    const long long part = (long long)D.part_first + t.first;
    if (D.limiter & kLimMedian) {
        // which waves hold candidates; the lanes of wall nodes do not know
        const bool some = __ballot(any_up) != 0;
        if ((threadIdx.x & (kWave - 1)) == 0) to_global<unsigned char>(a.above + part)[wave] = some ? 1 : 0;
    }
    if constexpr (STATS) node_partial(acc, a.blockpart + part * kNStat, red);
}

// Second pass: median filter (Sec. 3.5; cavity stencils of Sec. 4.4) on the
// Delta S' plane written by the collision kernel, and the ensemble-dependent
// limiters.  A wave walks down 64 adjacent columns in chunks of kMedChunk rows
// (the loads of a chunk, one per row, are issued together; the neighbouring
// columns come from the adjacent lanes), decides which nodes move and lists
// them in LDS; after kListRows rows the listed nodes are moved, 64 at a time,
// with every lane busy and all their loads in flight together.
constexpr int kMedChunk = 4;
constexpr int kListRows = 8;                      // rows decided before their moved nodes are moved
constexpr int kListCap = kListRows * kWave;

// the filter's threshold and decision for a node with Delta S' = dc whose
// stencil median is med (FLOOR or GATE reading of the tolerance delta)
template <class A, class DD>
__device__ __forceinline__ bool median_decide(const DD& D, A dc, A med, A& thr)
{
    const A dmed = A(D.delta_median);
    if (D.median_mode) {
        thr = med;
        return dc > dmed && dc > med;
    }
    thr = fmax(med, dmed);
    return dc > thr;
}

// median threshold of a fluid node from its window (rows b, c, n = y-1, y, y+1;
// columns l, m, r = x-1, x, x+1); returns whether the filter hits the node
template <int BC, class A, class DD>
__device__ __forceinline__ bool median_hit(const DD& D, int x, int y, int nx, int ny, const A (&b)[3],
                                           const A (&c)[3], const A (&n)[3], A& thr)
{
    A med;
    if constexpr (BC == kPeriodic) {
        med = median9(b[0], b[1], b[2], c[0], c[1], c[2], n[0], n[1], n[2]);
    } else {
        // three nodes along a neighbouring wall; two inner axis neighbours
        // next to a corner; 3x3 elsewhere
        const bool wl = x == 1, wr = x == nx - 2, wb = y == 1, wt = y == ny - 2;
        if ((wl || wr) && (wb || wt))
            med = med3(c[1], wl ? c[2] : c[0], wb ? n[1] : b[1]);
        else if (wl || wr)
            med = med3(b[1], c[1], n[1]);
        else if (wb || wt)
            med = med3(c[0], c[1], c[2]);
        else
            med = median9(b[0], b[1], b[2], c[0], c[1], c[2], n[0], n[1], n[2]);
    }
    return median_decide(D, c[1], med, thr);
}

// Free flight into a fluid node whose row differs between the lanes of a wave
// (a fluid node of the cavity has all its sources inside): one 32-bit lane
// offset per population on a scalar base (Q nx ny < 2^31 elements, so a
// plane's bytes fit 32 bits).
template <int BC, class T>
__device__ __forceinline__ void gather_node(gptr<const T> src, long long plane, int nx, int ny, int x, int y,
                                            typename Store<T>::A (&g)[9])
{
    using L = Lat<kD2Q9>;
    constexpr unsigned es = sizeof(T);
    int xm = x - 1, xp = x + 1, ym = y - 1, yp = y + 1;
    if constexpr (BC == kPeriodic) {
        xm = x == 0 ? nx - 1 : xm;
        xp = x == nx - 1 ? 0 : xp;
        ym = y == 0 ? ny - 1 : ym;
        yp = y == ny - 1 ? 0 : yp;
    }
    const unsigned r0 = unsigned(y) * unsigned(nx), rm = unsigned(ym) * unsigned(nx), rp = unsigned(yp) * unsigned(nx);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const unsigned rs = L::vy(i) > 0 ? rm : (L::vy(i) < 0 ? rp : r0);
        const unsigned cs = unsigned(L::vx(i) > 0 ? xm : (L::vx(i) < 0 ? xp : x));
        g[i] = Store<T>::ld(at_bytes(src + i * plane, es * (rs + cs)));
    }
}

// The limited state of a node after LBGK collisions, formed anew by a second
// pass from the populations g that arrived there (the buffer the step reads
// still holds them), f* - phi c d with phi the smallest of its factors, as the
// fused step forms it.  Returns phi; `lim` (0 unless wanted) is the limiter's
// entropy production beyond what the collision kernel counted for the node.
template <class T, int QE, int DS, class DD>
__device__ __forceinline__ typename Store<T>::A form_state(const DD& D, const typename Store<T>::A (&g)[9],
                                                           typename Store<T>::A dc, typename Store<T>::A tgt,
                                                           typename Store<T>::A fac, bool want_lim,
                                                           SiteState<kD2Q9, typename Store<T>::A>& S, double& lim)
{
    using A = typename Store<T>::A;
    constexpr int Q = 9;
    const A inf = A(__builtin_huge_val());
    const A shift = A(D.shift), c = A(D.c);
    unsigned tmask = 0;
    A pt = trim_phi(D, dc, tmask);     // the factor the collision kernel applied
    A dr, jx, jy, rho, ux, uy;
    moments_equilibrium<kD2Q9, QE>(g, shift, dr, jx, jy, rho, ux, uy, S.gs);
#pragma unroll
    for (int i = 0; i < Q; ++i) S.d[i] = g[i] - S.gs[i];
    S.dpost = dc;
    S.c = c;
    S.posrule = false;
    A phi = pt;
    bool done = false;
    if constexpr (DS == kExactHom) {
        if (D.homothety && isfinite(dc)) {
            // targets reached exactly (Sec. 3.6); the smallest one decides
            const bool hom = (tmask & kMaskTrim) && !D.trim_mode;
            if (hom) pt = exact_homothety_call(S, shift, A(D.delta_trim));
            phi = fmin(pt, fac);
            if (tgt < inf && !(hom && tgt >= A(D.delta_trim))) phi = fmin(phi, exact_homothety_call(S, shift, tgt));
            done = true;
        }
    }
    if (!done) phi = fmin(pt, fmin(fac, tgt < inf ? sqrt_(tgt * rcp(dc)) : A(1)));
    lim = 0.0;
    if (want_lim && isfinite(dc) && phi < pt) {
        if constexpr (DS == kQuad) {
            lim = double(dc * (pt * pt - phi * phi));
        } else {
            const A before = pt < A(1) ? delta_s_scaled<kD2Q9, DS>(S, shift, c, pt) : dc;
            lim = double(before - delta_s_scaled<kD2Q9, DS>(S, shift, c, phi));
        }
    }
    return phi;
}

// one node of a wave's list
template <class T, int QE, int DS, int BC, class DD>
__device__ __forceinline__ double form_node(const DD& D, gptr<const T> src, gptr<T> dst, long long plane, int x, int y,
                                            typename Store<T>::A dc, typename Store<T>::A tgt,
                                            typename Store<T>::A fac, bool want_lim)
{
    using A = typename Store<T>::A;
    A g[9];
    gather_node<BC>(src, plane, D.nx, D.ny, x, y, g);
    SiteState<kD2Q9, A> S;
    double lim;
    const A k = form_state<T, QE, DS>(D, g, dc, tgt, fac, want_lim, S, lim) * S.c;
    const unsigned own = unsigned(sizeof(T)) * (unsigned(y) * unsigned(D.nx) + unsigned(x));
#pragma unroll
    for (int i = 0; i < 9; ++i) Store<T>::st(at_bytes(dst + i * plane, own), S.gs[i] - k * S.d[i]);
    return lim;
}

// The same after ELBM collisions, whose f' - f* = -(alpha beta - 1) d would
// need the node's entropy root again, and in FP32 and FP64 domains beyond the
// last-level cache (in_place): the limited state that the collision
// kernel stored is rescaled toward its f*, rebuilt from the state's own
// moments (the limiter kept them): f* + r (f_stored - f*), r = pq / pt (the new
// factor over the applied one).  With the exact homothety the stored state's
// deviation e = pt x is scaled to the target directly, and a direct factor is
// taken relative to f' = f* + e / pt.
template <class T, int QE, int DS, class DD>
__device__ __forceinline__ double rescale_node(const DD& D, gptr<T> buf, long long plane, int x, int y,
                                               typename Store<T>::A dc, typename Store<T>::A tgt,
                                               typename Store<T>::A fac)
{
    using A = typename Store<T>::A;
    constexpr int Q = 9;
    const A inf = A(__builtin_huge_val());
    const A shift = A(D.shift);
    const gptr<const T> lsrc = buf;
    const unsigned own = unsigned(sizeof(T)) * (unsigned(y) * unsigned(D.nx) + unsigned(x));
    A gl[Q], gs[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) gl[i] = Store<T>::ld(at_bytes(lsrc + i * plane, own));
    A dr, jx, jy, rho, ux, uy;
    moments_equilibrium<kD2Q9, QE>(gl, shift, dr, jx, jy, rho, ux, uy, gs);
    unsigned tmask = 0;
    const A pt = trim_phi(D, dc, tmask);
    A r = fmin(fac, tgt < inf ? sqrt_(tgt * rcp(dc)) : A(1)) * rcp(pt);
    A fs[Q], e[Q];
    if constexpr (DS != kQuad) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            fs[i] = A(Lat<kD2Q9>::w(i)) * shift + gs[i];
            e[i] = (gl[i] - gs[i]) * rcp(fs[i]);
        }
    }
    if constexpr (DS == kExactHom) {
        A emin = A(0);
#pragma unroll
        for (int i = 0; i < Q; ++i) emin = fmin(emin, e[i]);
        if (D.homothety && isfinite(dc)) {
            const A ds_s = kull_sum<false>(fs, e, A(1));
            r = A(1);
            if (ds_s > A(0)) {
                if (tgt < ds_s) r = kullback_scale<Q>(fs, e, tgt, sqrt_(tgt * rcp(ds_s)), A(0), A(1));
                if (fac < A(1)) {
                    const A lmax = emin < A(0) ? A(-1) / emin : inf;
                    const A lam = pt < A(1) ? kullback_scale<Q>(fs, e, dc, sqrt_(dc * rcp(ds_s)), A(1), lmax) : A(1);
                    r = fmin(r, fac * lam);
                }
            }
        }
    }
    if (!(r < A(1))) return 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) Store<T>::st(at_bytes(buf + i * plane, own), gs[i] + r * (gl[i] - gs[i]));
    if (!isfinite(dc)) return 0.0;
    if constexpr (DS == kQuad) return double(pt * pt * dc * (A(1) - r * r));
    return double(kull_sum<false>(fs, e, A(1)) - kull_sum<false>(fs, e, r));
}

template <class T, int QE, int DS, int BC, bool ENS, bool STORED>
__device__ __forceinline__ void second_pass2d(const StepArgs& a)
{
    using A = typename Store<T>::A;
    __shared__ double red[4 * kNStat];
    // nodes to move, per wave: row and lane, smallest homothety target and
    // (ensemble limiters) smallest factor given as phi itself
    __shared__ unsigned short list_id[kThreads / kWave][kListCap];
    __shared__ A list_tgt[kThreads / kWave][kListCap], list_fac[ENS ? kThreads / kWave : 1][ENS ? kListCap : 1];
    const int tidx = tile_of_block(a, 0);
    const Tile t = a.tiles[tidx];
    const DomainDev& D = a.dom[t.domain];
    if constexpr (!ENS) {
        // no median filter in this domain: an empty partial
        if (!(D.limiter & kLimMedian)) {
            if (threadIdx.x < kNStat) partial_slot(a, 1, tidx)[threadIdx.x] = 0.0;
            return;
        }
    } else {
        if (D.dense) return;          // k_form2d's
    }
    AccT<A, double> acc;
    const int nx = D.nx, ny = D.ny;
    // rows y0-1 .. y1 are read; y1 <= ny, so one wrap keeps them in range
    auto row_of = [&](int y) -> int {
        if constexpr (BC == kPeriodic)
            return y < 0 ? y + ny : (y >= ny ? y - ny : y);
        else
            return y < 0 ? 0 : (y >= ny ? ny - 1 : y);
    };
    // FLOOR median only: the 64 consecutive nodes of a collision wave in which
    // no node exceeded delta hold no Delta S' of this step and read as zeros.
    // Which waves stored is staged in LDS for the tile's rows and halo rows:
    // [0] and [kFlagSlots - 1] the waves of the columns left and right of the
    // tile, between them those of its columns (at most five).
    const bool sparse = !((D.limiter & kLimEns) || D.median_mode != 0);
    constexpr int kFlagSlots = 8;
    __shared__ unsigned char sflag[kMaxTileH + 2][kFlagSlots];
    int xl = t.x0 - 1, xr = t.x1;      // the columns beside the tile
    if constexpr (BC == kPeriodic) {
        xl = xl < 0 ? nx - 1 : xl;
        xr = xr == nx ? 0 : xr;
    } else {
        xl = xl < 0 ? 0 : xl;
        xr = xr == nx ? nx - 1 : xr;
    }
    const auto wave_flags = reinterpret_cast<const unsigned char*>(a.above + D.part_first);
    // The filter's threshold is never below delta (FLOOR: max(median, delta);
    // GATE: only nodes above delta), so a tile none of whose nodes has
    // Delta S' > delta (the collision kernel counted them, in the same
    // precision) has nothing to filter and skips the medians.
    // The ensemble limiters use this step's E(Delta S') and thresholds;
    // threshold-type ones skip tiles whose largest Delta S' is at or below
    // the threshold (and that hold no infinite value), the smooth ones move
    // every node with Delta S' > 0.
    bool active = false;
    double ensv[kNEns] = {0.0, 0.0, 0.0, 0.0};
    if constexpr (ENS) {
        if (D.limiter & kLimEns) {
#pragma unroll
            for (int k = 0; k < kNEns; ++k) ensv[k] = D.ens[k];
        }
    }
    if (D.limiter & (kLimMedian | kLimEns)) {
        const int rows = t.y1 - t.y0;
        bool cand = false;
        if (D.limiter & kLimMedian) {
            for (int idx = int(threadIdx.x); idx < (rows + 2) * kFlagSlots; idx += kThreads) {
                const int ry = idx / kFlagSlots, slot = idx % kFlagSlots;
                const unsigned r = unsigned(row_of(t.y0 - 1 + ry)) * unsigned(nx);
                const unsigned first = (r + unsigned(t.x0)) / kWave, last = (r + unsigned(t.x1 - 1)) / kWave;
                const unsigned at = slot == 0 ? (r + unsigned(xl)) / kWave
                                              : (slot == kFlagSlots - 1 ? (r + unsigned(xr)) / kWave : first + unsigned(slot - 1));
                const bool own = slot > 0 && slot < kFlagSlots - 1;
                const unsigned char f = own && at > last ? 0 : wave_flags[at];
                sflag[ry][slot] = f;
                // (a wave may reach into the neighbouring tiles' columns)
                cand = cand || (f && own && ry > 0 && ry <= rows);
            }
        }
        if constexpr (ENS) {
            // the collision workgroups of a row's columns: at most two
            if (int(threadIdx.x) < 2 * rows) {
                const unsigned r = unsigned(t.y0 + int(threadIdx.x) / 2) * unsigned(nx);
                const unsigned b = (threadIdx.x & 1) ? (r + unsigned(t.x1 - 1)) / kThreads : (r + unsigned(t.x0)) / kThreads;
                const double* rp = a.blockpart + ((long long)D.part_first + b) * kNStat;
                const A mx = A(rp[kSMax]);
                const bool inf = rp[kSNonpos] > 0.0;
                if (D.limiter & (kLimEnsSmooth | kLimEnsRational)) cand = cand || rp[kSFluid] > 0.0;
                if (D.limiter & kLimEnsThresh) cand = cand || inf || mx > A(ensv[kEThresh]);
                if (D.limiter & kLimEnsBudget) cand = cand || inf || mx > A(ensv[kEBudget]);
                if (D.limiter & kLimTopK) cand = cand || inf || mx > A(D.delta_trim);
            }
        }
        active = __syncthreads_or(cand || (a.flags & kFlagAllTiles));
    }
    // nothing to filter in this tile: its partial is zero (no reduction)
    if (!active) {
        if (threadIdx.x < kNStat) partial_slot(a, 1, tidx)[threadIdx.x] = 0.0;
        return;
    }
    const int wave = int(threadIdx.x) >> 6;
    const int lane = int(threadIdx.x) & (kWave - 1);
    const int xw = t.x0 + wave * kWave;        // the wave's first column
    if (xw < t.x1) {                           // uniform per wave
        const long long plane = D.plane;
        const gptr<const A> dsb = to_global<A>(static_cast<const void*>(D.dsbuf));
        const gptr<T> dst = to_global<T>(D.buf[1 - a.parity]);
        const bool record = (a.flags & kFlagRecord) && (a.flags & kFlagStats);
        // lanes past the tile's last column repeat it and decide nothing
        const bool in = xw + lane < t.x1;
        const int x = in ? xw + lane : t.x1 - 1;
        int xm, xp;
        if constexpr (BC == kPeriodic) {
            xm = x == 0 ? nx - 1 : x - 1;
            xp = x == nx - 1 ? 0 : x + 1;
        } else {
            // cavity: columns off the grid are never part of a fluid stencil
            xm = x > 0 ? x - 1 : x;
            xp = x < nx - 1 ? x + 1 : x;
        }
        // Each lane loads its own column (one aligned load per row); the
        // columns x -+ 1 come from the neighbouring lanes.  Only the first
        // lane of a wave and the lane at the right end of a wave or of the
        // tile load their outside neighbour themselves.
        const bool own_l = lane == 0;
        const bool own_r = lane == kWave - 1 || x == t.x1 - 1;
        auto load_raw = [&](int y, A (&r)[3]) {
            const int yy = row_of(y);
            const long long rr = (long long)yy * nx;
            r[1] = Store<A>::ld(dsb + (rr + x));
            if (own_l) r[0] = Store<A>::ld(dsb + (rr + xm));
            if (own_r) r[2] = Store<A>::ld(dsb + (rr + xp));
        };
        // zeros for the columns of waves that stored nothing (FLOOR median),
        // then the columns x -+ 1 from the neighbouring lanes
        auto complete = [&](int y, A (&r)[3]) {
            if (sparse) {
                const unsigned char* f = sflag[y - (t.y0 - 1)];
                const unsigned r0 = unsigned(row_of(y)) * unsigned(nx), first = (r0 + unsigned(t.x0)) / kWave;
                auto slot = [&](int xs) { return f[1 + int((r0 + unsigned(xs)) / kWave - first)]; };
                if (!slot(x)) r[1] = A(0);
                if (own_l && !(x == t.x0 ? f[0] : slot(x - 1))) r[0] = A(0);
                if (own_r && !(x == t.x1 - 1 ? f[kFlagSlots - 1] : slot(x + 1))) r[2] = A(0);
            }
            // every lane takes part in the shifts (no branch around them)
            const A l = lane_shift<-1>(r[1]), rr = lane_shift<+1>(r[1]);
            r[0] = own_l ? r[0] : l;
            r[2] = own_r ? r[2] : rr;
        };
        // w[k] holds row yb - 1 + k of the current chunk; the rows of the next
        // chunk are loaded into nw before the current chunk's nodes are moved,
        // so waiting for them does not wait for those stores
        A w[kMedChunk + 2][3], nw[kMedChunk][3];
#pragma unroll
        for (int k = 0; k < kMedChunk + 2; ++k) w[k][0] = w[k][2] = A(0);
#pragma unroll
        for (int k = 0; k < kMedChunk; ++k) nw[k][0] = nw[k][1] = nw[k][2] = A(0);
        load_raw(t.y0 - 1, w[0]);
        load_raw(t.y0, w[1]);
        complete(t.y0 - 1, w[0]);
        complete(t.y0, w[1]);
#pragma unroll
        for (int k = 0; k < kMedChunk; ++k)
            if (t.y0 + k + 1 <= t.y1) load_raw(t.y0 + k + 1, nw[k]);
        int listed = 0;                // nodes in the wave's list (uniform)
        int ylist = t.y0;              // row of its first entries
        for (int yb = t.y0; yb < t.y1; yb += kMedChunk) {
#pragma unroll
            for (int k = 0; k < kMedChunk; ++k)
                if (yb + k + 1 <= t.y1) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) w[k + 2][q] = nw[k][q];
                    complete(yb + k + 1, w[k + 2]);
                }
#pragma unroll
            for (int k = 0; k < kMedChunk; ++k) {
                const int y = yb + k;
                if (y >= t.y1) break;
                const A dc = w[k + 1][1];
                const bool fluid = in && node_class<BC>(x, y, nx, ny) == kNodeFluid;
                // smallest homothety target and smallest direct factor of the
                // limiters that act on this node (relative to f')
                A tgt = A(__builtin_huge_val()), fac = A(1), thr;
                SecondHit h;
                if ((D.limiter & kLimMedian) && fluid && median_hit<BC>(D, x, y, nx, ny, w[k], w[k + 1], w[k + 2], thr)) {
                    h.bits |= kMaskMedian;
                    tgt = thr;
                }
                if constexpr (ENS) {
                    if ((D.limiter & kLimEns) && fluid) ens_terms(D, ensv, dc, tgt, fac, h);
                }
                bool moves = false;
                if (h.bits) {
                    if (h.bits & kMaskMedian) ++acc.filt;
                    acc.ens += h.ens;
                    acc.trim += h.trim;
                    if (record)
                        to_global<unsigned char>(D.mask)[unsigned(y) * unsigned(nx) + unsigned(x)] |= (unsigned char)h.bits;
                    // further than the collision kernel's trimming moved it;
                    // the exact homothety decides by its roots
                    unsigned tmask = 0;
                    const A pt = trim_phi(D, dc, tmask);
                    moves = fmin(fac, tgt < A(__builtin_huge_val()) ? sqrt_(tgt * rcp(dc)) : A(1)) < pt;
                    if constexpr (DS == kExactHom) moves = moves || (D.homothety && isfinite(dc) && pt > A(0));
                }
                const unsigned long long b = __ballot(moves);
                if (moves) {
                    const int at = listed + int(__builtin_amdgcn_mbcnt_hi(unsigned(b >> 32),
                                                                        __builtin_amdgcn_mbcnt_lo(unsigned(b), 0)));
                    list_id[wave][at] = (unsigned short)((y - ylist) * kWave + lane);
                    list_tgt[wave][at] = tgt;
                    if constexpr (ENS) list_fac[wave][at] = fac;
                }
                listed += __popcll(b);
            }
            {
                const int yn = yb + kMedChunk;
#pragma unroll
                for (int k = 0; k < kMedChunk; ++k)
                    if (yn < t.y1 && yn + k + 1 <= t.y1) load_raw(yn + k + 1, nw[k]);
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                w[0][q] = w[kMedChunk][q];
                w[1][q] = w[kMedChunk + 1][q];
            }
            if (yb + kMedChunk - ylist < kListRows && yb + kMedChunk < t.y1) continue;
            // the list is the wave's own: its LDS accesses stay in order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int e = lane; e < listed; e += kWave) {
                const int id = list_id[wave][e];
                const int xn = xw + (id & (kWave - 1)), yn = ylist + (id >> 6);
                const A tgt = list_tgt[wave][e];
                A fac = A(1);
                if constexpr (ENS) fac = list_fac[wave][e];
                const A dc = Store<A>::ld(dsb + (unsigned(yn) * unsigned(nx) + unsigned(xn)));
                if constexpr (STORED)
                    acc.lim += rescale_node<T, QE, DS>(D, dst, plane, xn, yn, dc, tgt, fac);
                else
                    acc.lim += form_node<T, QE, DS, BC>(D, to_global<T>(static_cast<const void*>(D.buf[a.parity])), dst,
                                                        plane, xn, yn, dc, tgt, fac, a.flags & kFlagStats);
            }
            __builtin_amdgcn_wave_barrier();
            listed = 0;
            ylist = yb + kMedChunk;
        }
    }
    if (a.flags & kFlagStats) store_partial(acc, partial_slot(a, 1, tidx), red);
}

// the second D2Q9 pass without and with ensemble-dependent limiters (the
// latter needs more registers), forming the moved nodes anew or, after ELBM and
// beyond the last-level cache, from the stored states
template <class T, int QE, int DS, int BC, bool STORED>
__global__ void __launch_bounds__(kThreads) k_median2d(StepArgs a)
{
    second_pass2d<T, QE, DS, BC, false, STORED>(a);
}

template <class T, int QE, int DS, int BC, bool STORED>
__global__ void __launch_bounds__(kThreads) k_median_ens2d(StepArgs a)
{
    second_pass2d<T, QE, DS, BC, true, STORED>(a);
}

// Second pass of the domains whose every node it moves (the smooth and the
// rational factor).  The collision kernel stored their Delta S' and no
// populations, and this pass forms each fluid node's state once, one node per
// thread over the same nodes: 36 + 4 and 40 + 36 bytes per FP32 node in
// the two passes, where storing the trimmed state and rescaling it in place
// moved 36 + 40 and 40 + 36 and waited for the stored state besides.  Its
// terms of the sums join the workgroup's partial.
template <class T, int QE, int DS, int BC>
__global__ void __launch_bounds__(kThreads) k_form2d(StepArgs a)
{
    using A = typename Store<T>::A;
    __shared__ double red[4 * kNStat];
    const Block t = a.blocks ? a.blocks[blockIdx.x] : Block{0, int(blockIdx.x)};
    const DomainDev& D = a.dom[t.domain];
    if (!D.dense) return;
    const int nx = D.nx, ny = D.ny;
    const long long plane = D.plane;
    const gptr<const T> src = to_global<T>(static_cast<const void*>(D.buf[a.parity]));
    const gptr<T> dst = to_global<T>(D.buf[1 - a.parity]);
    const gptr<const A> dsb = to_global<A>(static_cast<const void*>(D.dsbuf));
    const bool record = a.flags & kFlagRecord;
    double ensv[kNEns];
#pragma unroll
    for (int k = 0; k < kNEns; ++k) ensv[k] = D.ens[k];
    AccT<A, double> acc;
    const Node v = node_of(D, t.first);
    const int x = v.x, y = v.y, lane = int(threadIdx.x) & (kWave - 1);
    if (v.in) {
        const unsigned n = v.n;
        // (first: they are in flight while the window below is put together)
        A g[9];
        gather_at<BC>(src, plane, nx, ny, v, g);
        A w[3][3];
        if (D.limiter & kLimMedian) {
            // rows y - 1, y, y + 1 of Delta S'; the columns beside come from the
            // neighbouring lanes, the wave's end lanes and the row's end nodes
            // load theirs (clamped at a cavity's edges, where no fluid node
            // reads them), the left one mostly: a second load serves a lane that
            // needs the right one
            const unsigned all = unsigned(nx) * unsigned(ny);
            const bool end_l = x == 0, end_r = x == nx - 1;
            const unsigned wrap = BC == kPeriodic ? unsigned(nx) : 1u;
            const bool own_l = lane == 0 || end_l, own_r = lane == kWave - 1 || end_r;
            const unsigned to_l = end_l ? wrap - 1 : ~0u, to_r = end_r ? 1u - wrap : 1u;   // offsets mod 2^32
            unsigned r[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                r[k] = k == 0 ? n - unsigned(nx) : (k == 1 ? n : n + unsigned(nx));
                if (k == 0 && y == 0) r[k] = BC == kPeriodic ? n + all - unsigned(nx) : n;
                if (k == 2 && y == ny - 1) r[k] = BC == kPeriodic ? n + unsigned(nx) - all : n;
                w[k][1] = Store<A>::ld(dsb + r[k]);
            }
            A beside[3] = {A(0), A(0), A(0)};
            if (own_l || own_r) {
#pragma unroll
                for (int k = 0; k < 3; ++k) beside[k] = Store<A>::ld(dsb + (r[k] + (own_l ? to_l : to_r)));
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const A l = lane_shift<-1>(w[k][1]), rr = lane_shift<+1>(w[k][1]);
                w[k][0] = own_l ? beside[k] : l;
                w[k][2] = own_r ? beside[k] : rr;
            }
            if (own_l && own_r) {      // a row's end at a wave's end
#pragma unroll
                for (int k = 0; k < 3; ++k) w[k][2] = Store<A>::ld(dsb + (r[k] + to_r));
            }
        } else {
            w[1][1] = Store<A>::ld(dsb + n);
        }
        if (node_class<BC>(x, y, nx, ny) == kNodeFluid) {
            const A dc = w[1][1];
            A tgt = A(__builtin_huge_val()), fac = A(1), thr;
            SecondHit h;
            if ((D.limiter & kLimMedian) && median_hit<BC>(D, x, y, nx, ny, w[0], w[1], w[2], thr)) {
                h.bits |= kMaskMedian;
                tgt = thr;
                acc.filt = 1;
            }
            ens_terms(D, ensv, dc, tgt, fac, h);
            acc.ens = h.ens;
            acc.trim = h.trim;
            if (record && h.bits) to_global<unsigned char>(D.mask)[n] |= (unsigned char)h.bits;
            SiteState<kD2Q9, A> S;
            A phi = form_state<T, QE, DS>(D, g, dc, tgt, fac, true, S, acc.lim);
            // Delta S' is infinite where the positivity rule acts, and none of the
            // factors above need do so there: E(Delta S') is 0 where no node has a
            // positive finite value, and a median may be infinite too
            // (with the quadratic form the rule and these factors cannot be combined)
            if constexpr (DS != kQuad) {
                if (D.limiter & kLimPos) phi = fmin(phi, positivity_phi<kD2Q9>(S, A(D.shift)));
            }
            store_limited<T>(dst, plane, 0, unsigned(sizeof(T)) * n, S, phi, S.c);
        }
    }
    // one value per wave and term, then added to the workgroup's partial
    // (nobody else's: the atomic add only spares the wait for the old value)
    const int wave = int(threadIdx.x) >> 6;
    const double lim = wave_reduce<false>(acc.lim);
    auto count = [](bool b) { return double(unsigned(__popcll(__ballot(b)))); };
    const double nt = count(acc.trim != 0), nf = count(acc.filt != 0), ne = count(acc.ens != 0);
    if (lane == kWave - 1) {
        red[wave * 4] = lim;
        red[wave * 4 + 1] = nt;
        red[wave * 4 + 2] = nf;
        red[wave * 4 + 3] = ne;
    }
    __syncthreads();
    const int k = int(threadIdx.x);
    if (k < 4) {
        const double s = (red[k] + red[4 + k]) + (red[8 + k] + red[12 + k]);
        const int slot = k == 0 ? kSLim : (k == 1 ? kSTrim : (k == 2 ? kSFilt : kSEns));
        unsafeAtomicAdd(a.blockpart + ((long long)D.part_first + t.first) * kNStat + slot, s);
    }
}

// The domain fields the fused step reads in its row loop.
struct FusedDom {
    int nx, ny, limiter, trim_mode, median_mode, homothety, diffusive, probe_x, probe_y, probe_cap;
    double delta_trim, delta_median, lid_ux, rho0;
    float* probe;
    unsigned char* mask;
    double* dS;
};

// Fused D2Q9 step: collision, trimming, positivity and the median filter of
// Sec. 3.5 (cavity stencils of Sec. 4.4) in one pass, for domains without
// ensemble-dependent limiters.  Each wave walks down 64 adjacent columns of a
// tile, lane l on column xw - 1 + l: lanes 1..62 own the wave's columns, lanes
// 0 and 63 compute the neighbours that the owned columns' stencils read (their
// Delta S' reaches the owned lanes by DPP lane shifts), and the rows above
// and below the tile are computed for their Delta S' only.  A row is decided
// one row later, when the Delta S' of the row below it is known; meanwhile
// it keeps f* and the nonequilibrium part, so that its final state
// f* - phi c d is formed once, phi the smallest of the trimming, positivity
// and median factors (as in eq. (LimGenF) with the factors of Sec. 3).  The
// gathers of the next row are issued before the current row is computed.  No
// Delta S' plane is written; one FP64 partial per tile goes to set 1.
template <class T, int QE, int DS, int BC, bool STATS>
__global__ void __launch_bounds__(kThreads) k_fused2d(StepArgs a)
{
    using A = typename Store<T>::A;
    constexpr int Q = 9;
    __shared__ double red[STATS ? 4 * kNStat : 1];
    // the pending row's f* and nonequilibrium part, one column per thread
    // (each thread reads back only its own slots)
    __shared__ A pend[2 * Q][kThreads];
    const int tidx = tile_of_block(a, 0);
    const Tile t = a.tiles[tidx];
    // the fields the walk reads, copied once: held in scalar registers (read
    // through the table they would be reloaded, each time with a wait for
    // every load in flight, after each store)
    const DomainDev& Dt = a.dom[t.domain];
    const FusedDom D{Dt.nx, Dt.ny, Dt.limiter, Dt.trim_mode, Dt.median_mode, Dt.homothety, Dt.diffusive,
                     Dt.probe_x, Dt.probe_y, Dt.probe_cap, Dt.delta_trim, Dt.delta_median, Dt.lid_ux, Dt.rho0,
                     Dt.probe, Dt.mask, Dt.dS};
    const int nx = D.nx, ny = D.ny;
    const long long plane = Dt.plane;
    const gptr<const T> src = to_global<T>(static_cast<const void*>(Dt.buf[a.parity]));
    const gptr<T> dst = to_global<T>(Dt.buf[1 - a.parity]);
    const A shift = A(Dt.shift), c = A(Dt.c);
    const bool record = STATS && (a.flags & kFlagRecord);
    const bool want_ent = STATS && (a.flags & kFlagEntropy);
    const bool median = D.limiter & kLimMedian;
    const long long step = a.counter[a.parity];
    // the index of the next step, read by the next launch (which reads buffer 1 - parity)
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counter[1 - a.parity] = step + 1;

    const int lane = int(threadIdx.x) & (kWave - 1);
    const int xw = t.x0 + (int(threadIdx.x) >> 6) * kFusedCols;   // the wave's first owned column
    const int xw1 = xw + kFusedCols < t.x1 ? xw + kFusedCols : t.x1;
    // per-thread sums over the rows it owns: moments and limiter production
    // in FP64, the rest in the arithmetic type
    AccT<A, double> acc;
    double am = 0.0, ax = 0.0, ay = 0.0;
    if (xw < t.x1) {   // uniform per wave
        // the lane's column; lanes past the right neighbour of the last owned
        // column repeat it (their values are never used)
        const int x = xw - 1 + lane;
        const int xe = x < xw1 ? x : xw1;
        const bool owned = lane >= 1 && x < xw1;
        bool in_x = true;
        int xc = xe;
        if constexpr (BC == kPeriodic) {
            xc = xe < 0 ? xe + nx : (xe >= nx ? xe - nx : xe);
        } else {
            in_x = xe >= 0 && xe < nx;
            xc = xe < 0 ? 0 : (xe >= nx ? nx - 1 : xe);
        }
        const Cols<T, BC> cl(xc, nx);
        // rows y0 - 1 .. y1; off a cavity they are no nodes (clamped loads)
        auto row_of = [&](int y) -> int {
            if constexpr (BC == kPeriodic) return y < 0 ? y + ny : (y >= ny ? y - ny : y);
            else return y < 0 ? 0 : (y >= ny ? ny - 1 : y);
        };
        // Delta S' window of the node's stencil: rows y - 2 (b), y - 1 (m)
        // and y (n) relative to the row being computed; [0] left, [1] own,
        // [2] right column
        A wb[3] = {A(0), A(0), A(0)}, wm[3] = {A(0), A(0), A(0)};
        // the pending row (the one above the row being computed): f* and d
        // in LDS, the rest here
        const int tid = int(threadIdx.x);
        A p_dpost = A(0), p_phi = A(1);
        unsigned p_mask = 0;
        bool p_fluid = false;
        // one row: collision of row y from its gathered populations g, then the
        // decision and store of row y - 1
        auto do_row = [&](int y, const A (&g)[Q]) {
            const int yr = row_of(y);
            const bool in_dom = in_x && (BC == kPeriodic || (y >= 0 && y < ny));
            const int cls = in_dom ? node_class<BC>(xc, yr, nx, ny) : int(kNodeNone);
            const bool own = owned && y >= t.y0 && y < t.y1;
            const long long row = (long long)yr * nx;
            const unsigned node = unsigned(row) + unsigned(xc);
            SiteState<kD2Q9, A> S;
            SiteScalars sc;
            A dcur = A(0);
            unsigned mask = 0;
            A phi = A(1);
            if (cls == kNodeFluid) {
                collide_site<kD2Q9, QE, DS, false>(g, shift, c, S, sc, STATS);
                dcur = S.dpost;
                if (own) {
                    if constexpr (STATS) {
                        am += sc.dr;
                        ax += sc.jx;
                        ay += sc.jy;
                        if (!(isfinite(sc.dr) && isfinite(sc.jx) && isfinite(sc.jy))) ++acc.nonfin;
                        acc.fluid_site(sc, S.dpost);
                    }
                    if (want_ent) {
                        const double e = entropy_site<kD2Q9>(g, shift);
                        if (isfinite(e)) acc.ent += A(e);
                    }
                    if (xc == D.probe_x && yr == D.probe_y) {
                        const gptr<float> pr = to_global<float>(D.probe) + 2 * (step % D.probe_cap);
                        pr[0] = sc.ux;
                        pr[1] = sc.uy;
                    }
                    phi = trim_phi(D, S.dpost, mask);
                    if constexpr (DS == kExactHom) {
                        if (D.homothety && (mask & kMaskTrim) && !D.trim_mode && isfinite(S.dpost))
                            phi = exact_homothety_call(S, shift, A(D.delta_trim));
                    }
                    if (D.limiter & kLimPos) {
                        const A pp = positivity_phi<kD2Q9>(S, shift);
                        if (pp < A(1)) {
                            mask |= kMaskPos;
                            if constexpr (STATS) ++acc.pos;
                            phi = fmin(phi, pp);
                        }
                    }
                    if (sc.nonpos) mask |= kMaskNonpos;
                    if (record) to_global<double>(D.dS)[node] = double(S.dpost);
                }
            } else if (own && cls != kNodeNone) {
                // walls and lid: no collision, no limiter; stored at once
                A out[Q];
                wall_state<QE>(D, cls, xc, yr, nx, ny, g, shift, out);
#pragma unroll
                for (int i = 0; i < Q; ++i) Store<T>::st(at_bytes(dst + (i * plane + row), cl.own), out[i]);
                if constexpr (STATS) {
                    double dr, jx, jy;
                    moments_fp64(g, dr, jx, jy);
                    am += dr;
                    ax += jx;
                    ay += jy;
                    if (!(isfinite(dr) && isfinite(jx) && isfinite(jy))) ++acc.nonfin;
                }
                if (record) {
                    to_global<unsigned char>(D.mask)[node] = (unsigned char)kMaskNotFluid;
                    to_global<double>(D.dS)[node] = 0.0;
                }
            }
            // this row's Delta S' with its neighbours' (every lane takes part)
            A wn[3];
            wn[1] = dcur;
            wn[0] = lane_shift<-1>(dcur);
            wn[2] = lane_shift<+1>(dcur);
            // decide and store the row above (row y - 1)
            const int yd = y - 1;
            if (owned && yd >= t.y0 && yd < t.y1 && p_fluid) {
                const int ydr = row_of(yd);
                const long long drow = (long long)ydr * nx;
                SiteState<kD2Q9, A> P;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    P.gs[i] = pend[i][tid];
                    P.d[i] = pend[Q + i][tid];
                }
                P.dpost = p_dpost;
                P.c = c;
                P.posrule = false;
                A thr;
                if (median && median_hit<BC>(D, xc, ydr, nx, ny, wb, wm, wn, thr)) {
                    p_mask |= kMaskMedian;
                    if constexpr (STATS) ++acc.filt;
                    A pm = A(1);
                    bool done = false;
                    if constexpr (DS == kExactHom) {
                        if (D.homothety && isfinite(p_dpost)) {
                            pm = exact_homothety_call(P, shift, thr);
                            done = true;
                        }
                    }
                    if (!done) pm = sqrt_(thr * rcp(p_dpost));
                    p_phi = fmin(p_phi, pm);
                }
                store_limited<T, false>(dst, plane, drow, cl.own, P, p_phi, c);
                if constexpr (STATS) {
                    if (p_mask & kMaskTrim) ++acc.trim;
                    if (p_phi < A(1) && isfinite(p_dpost))
                        acc.lim += double(p_dpost - delta_s_scaled<kD2Q9, DS>(P, shift, c, p_phi));
                }
                if (record) to_global<unsigned char>(D.mask)[unsigned(drow) + unsigned(xc)] = (unsigned char)p_mask;
            }
            // this row becomes the pending one
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                wb[k] = wm[k];
                wm[k] = wn[k];
            }
            p_fluid = own && cls == kNodeFluid;
            if (p_fluid) {
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    pend[i][tid] = S.gs[i];
                    pend[Q + i][tid] = S.d[i];
                }
                p_dpost = S.dpost;
                p_phi = phi;
                p_mask = mask;
            }
        };
        // rows y0 - 1 .. y1, the gathers of the next two rows in flight while a
        // row is computed (a wave walks its rows alone, so its own loads are
        // what hides the memory latency); three buffers used in turn, so no
        // register copy waits for a load.  The gathers are unconditional
        // (past the last row they repeat it and go unused): a load skipped on
        // one path would make every use wait for all loads in flight.
        auto fetch = [&](int y, A (&g)[Q]) { gather2d<BC>(src, plane, nx, ny, cl, row_of(y <= t.y1 ? y : t.y1), g); };
        A ga[Q], gb[Q], gc[Q];
        fetch(t.y0 - 1, ga);
        fetch(t.y0, gb);
        for (int y = t.y0 - 1;; y += 3) {
            fetch(y + 2, gc);
            do_row(y, ga);
            if (y + 1 > t.y1) break;
            fetch(y + 3, ga);
            do_row(y + 1, gb);
            if (y + 2 > t.y1) break;
            fetch(y + 4, gb);
            do_row(y + 2, gc);
            if (y + 3 > t.y1) break;
        }
    }
    if constexpr (!STATS) return;
    AccT<double> tot;
    tot.mass = am;
    tot.jx = ax;
    tot.jy = ay;
    tot.dpre = double(acc.dpre);
    tot.dpost = double(acc.dpost);
    tot.maxd = double(acc.maxd);
    tot.lim = acc.lim;
    tot.ent = double(acc.ent);
    tot.trim = acc.trim;
    tot.filt = acc.filt;
    tot.nonpos = acc.nonpos;
    tot.nonfin = acc.nonfin;
    tot.fluid = acc.fluid;
    tot.pos = acc.pos;
    store_partial(tot, partial_slot(a, 1, tidx), red);
}

// Small D2Q9 domains (LBGK, no ensemble limiter): whole steps of a tile in one
// workgroup, one node per thread, a.steps of them.  A step needs the
// populations of the nodes around and, for the median, their Delta S', so the
// threads cover the tile and a halo of 2 a.steps - 1 nodes; populations go from
// step to step in LDS (rounded to storage, as a store would), Delta S' within a
// step.  What bounds a small domain is latency: the collision kernel and the
// second pass each take a launch and a chain of memory accesses of
// microseconds (7 + 8 us for a 100 x 100 FP64 cavity), here a step is its
// arithmetic and two barriers.  Decisions and states are those of the other
// forms; the sums belong to the last step, one partial per tile in set 1.
// MULTI: several steps (then without sums); the single step, with or without
// them, needs no loop, whose hoisted constants cost it a wave per SIMD.
constexpr int kBlockMax = 512;      // threads of a workgroup
template <class T, int QE, int DS, int BC, bool STATS, bool MULTI>
__global__ void __launch_bounds__(kBlockMax) k_block2d(StepArgs a)
{
    using A = typename Store<T>::A;
    using L = Lat<kD2Q9>;
    constexpr int Q = 9;
    __shared__ T leaving[MULTI ? Q : 1][MULTI ? kBlockMax : 1];
    __shared__ A ds[kBlockMax];
    __shared__ double red[STATS ? kBlockMax / kWave * kNStat : 1];
    const int tidx = tile_of_block(a, 0);
    const Tile t = a.tiles[tidx];
    const DomainDev& D = a.dom[t.domain];
    const int nx = D.nx, ny = D.ny;
    const long long plane = D.plane;
    const gptr<const T> src = to_global<T>(static_cast<const void*>(D.buf[a.parity]));
    const gptr<T> dst = to_global<T>(D.buf[1 - a.parity]);
    const A shift = A(D.shift), c = A(D.c);
    const bool record = STATS && (a.flags & kFlagRecord);
    const bool want_ent = STATS && (a.flags & kFlagEntropy);
    const bool median = D.limiter & kLimMedian;
    const long long step = a.counter[a.parity];
    const int steps = MULTI ? a.steps : 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counter[1 - a.parity] = step + steps;

    const int halo = 2 * steps - 1, bw = a.block_w + 2 * halo, bh = a.block_h + 2 * halo;
    // the first threads take the tile's own nodes in row-major order, the others
    // the frame of the halo (so that the sums do not depend on a.steps): the
    // rows below the tile, the rows above it, the columns left and right
    const int tid = int(threadIdx.x), w = a.block_w, own_nodes = w * a.block_h;
    int lx, ly;
    if (tid < own_nodes) {
        ly = tid / w;
        lx = tid - ly * w + halo;
        ly += halo;
    } else if (tid < own_nodes + 2 * halo * bw) {
        const int r = tid - own_nodes;
        ly = r / bw;
        lx = r - ly * bw;
        ly += ly < halo ? 0 : a.block_h;
    } else {
        const int r = tid - own_nodes - 2 * halo * bw;
        ly = r / (2 * halo);
        lx = r - ly * 2 * halo;
        lx += lx < halo ? 0 : w;
        ly = tid < bw * bh ? ly + halo : bh;        // past the frame: no node
    }
    const int pos = ly * bw + lx;          // place in LDS
    // the thread's node; off a cavity, and past the halo of a short last tile,
    // there is none
    const int X = t.x0 - halo + lx, Y = t.y0 - halo + ly;
    bool inside = ly < bh && X < t.x1 + halo && Y < t.y1 + halo;
    int x = X, y = Y;
    if constexpr (BC == kPeriodic) {
        x = wrapi(X, nx);
        y = wrapi(Y, ny);
    } else {
        inside = inside && X >= 0 && X < nx && Y >= 0 && Y < ny;
    }
    const bool owned = inside && X >= t.x0 && X < t.x1 && Y >= t.y0 && Y < t.y1;
    const int cls = inside ? node_class<BC>(x, y, nx, ny) : int(kNodeNone);
    const unsigned node = unsigned(y) * unsigned(nx) + unsigned(x);
    // neighbours in the workgroup (at the ends of its nodes a node stands in for
    // the missing one: nothing that is stored depends on it.  What lies past a
    // short tile in LDS does not: nobody writes it, and the logarithms and roots
    // of what was left there held whole workgroups up, 40 x 40 periodic nodes
    // with the exact homothety in FP64 20 us a step against 4)
    const int lx1 = t.x1 - t.x0 + 2 * halo - 1, ly1 = t.y1 - t.y0 + 2 * halo - 1;
    const int dl = lx > 0 ? -1 : 0, dr = lx < lx1 ? 1 : 0;
    const int db = ly > 0 ? -bw : 0, dt = ly < ly1 ? bw : 0;
    const int at = ly < bh ? pos : 0;

    AccT<A, double> acc;      // (the second pass, whose terms these are too, adds them in FP64)
    A g[Q];
    if (inside) gather_at<BC>(src, plane, nx, ny, Node{node, x, y, true, false}, g);
    for (int n = 0; n < steps; ++n) {
        const bool last = !MULTI || n == steps - 1;
        SiteState<kD2Q9, A> S;
        SiteScalars sc;
        A out[Q];
        A phi = A(1);
        unsigned mask = 0;
        A dsv = A(0);
        if (cls == kNodeFluid) {
            collide_site<kD2Q9, QE, DS, false>(g, shift, c, S, sc, STATS && last);
            dsv = S.dpost;
            if constexpr (STATS) {
                if (owned) {
                    acc.moments(sc);
                    acc.fluid_site(sc, S.dpost);
                    if (want_ent) {
                        const double e = entropy_site<kD2Q9>(g, shift);
                        if (isfinite(e)) acc.ent += A(e);
                    }
                }
            }
            if (owned && x == D.probe_x && y == D.probe_y) {
                const gptr<float> p = to_global<float>(D.probe) + 2 * ((step + n) % D.probe_cap);
                p[0] = sc.ux;
                p[1] = sc.uy;
            }
        } else if (cls != kNodeNone) {
            wall_state<QE>(D, cls, x, y, nx, ny, g, shift, out);
            if constexpr (STATS) {
                if (owned) {
                    moments_fp64(g, sc.dr, sc.jx, sc.jy);
                    acc.moments(sc);
                    if (record) {
                        to_global<unsigned char>(D.mask)[node] = (unsigned char)kMaskNotFluid;
                        to_global<double>(D.dS)[node] = 0.0;
                    }
                }
            }
        }
        if (median) {
            if (ly < bh) ds[pos] = dsv;
            __syncthreads();
        }
        if (cls == kNodeFluid) {
            phi = trim_phi(D, S.dpost, mask);
            if constexpr (DS == kExactHom) {
                if (D.homothety && (mask & kMaskTrim) && !D.trim_mode && isfinite(S.dpost))
                    phi = exact_homothety_call(S, shift, A(D.delta_trim));
            }
            if (D.limiter & kLimPos) {
                const A pp = positivity_phi<kD2Q9>(S, shift);
                if (pp < A(1)) {
                    mask |= kMaskPos;
                    if (STATS && owned) ++acc.pos;
                    phi = fmin(phi, pp);
                }
            }
            if (median) {
                const A* r = ds + at;
                const A b[3] = {r[db + dl], r[db], r[db + dr]}, m[3] = {r[dl], dsv, r[dr]},
                        u[3] = {r[dt + dl], r[dt], r[dt + dr]};
                A thr;
                if (median_hit<BC>(D, x, y, nx, ny, b, m, u, thr)) {
                    mask |= kMaskMedian;
                    if (STATS && owned) ++acc.filt;
                    A pm = A(1);
                    bool done = false;
                    if constexpr (DS == kExactHom) {
                        if (D.homothety && isfinite(dsv)) {
                            pm = exact_homothety_call(S, shift, thr);
                            done = true;
                        }
                    }
                    if (!done) pm = sqrt_(thr * rcp(dsv));
                    phi = fmin(phi, pm);
                }
            }
            const A k = phi * c;
#pragma unroll
            for (int i = 0; i < Q; ++i) out[i] = S.gs[i] - k * S.d[i];
            if constexpr (STATS) {
                if (owned) {
                    if (mask & kMaskTrim) ++acc.trim;
                    if (phi < A(1) && isfinite(dsv)) acc.lim += dsv - delta_s_scaled<kD2Q9, DS>(S, shift, c, phi);
                    if (record) {
                        if (sc.nonpos) mask |= kMaskNonpos;
                        to_global<unsigned char>(D.mask)[node] = (unsigned char)mask;
                        to_global<double>(D.dS)[node] = double(dsv);
                    }
                }
            }
        }
        if (last) {
            if (owned) {
#pragma unroll
                for (int i = 0; i < Q; ++i) Store<T>::st(at_bytes(dst + i * plane, unsigned(sizeof(T)) * node), out[i]);
            }
            break;
        }
        if constexpr (MULTI) {
            if (inside) {
#pragma unroll
                for (int i = 0; i < Q; ++i) st_shared<T>(&leaving[i][pos], out[i]);
            }
            __syncthreads();
            if (inside) {
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const int from = at + (L::vx(i) > 0 ? dl : (L::vx(i) < 0 ? dr : 0)) + (L::vy(i) > 0 ? db : (L::vy(i) < 0 ? dt : 0));
                    bool off = false;
                    if constexpr (BC != kPeriodic)
                        off = (L::vx(i) > 0 && x == 0) || (L::vx(i) < 0 && x == nx - 1) || (L::vy(i) > 0 && y == 0) ||
                              (L::vy(i) < 0 && y == ny - 1);
                    g[i] = ld_shared<T>(off ? &leaving[L::opp(i)][pos] : &leaving[i][from]);
                }
            }
            // without the median filter there is no other barrier before the next store
            if (!median) __syncthreads();
        }
    }
    if constexpr (STATS) node_partial(acc, partial_slot(a, 1, tidx), red);
}

template <int BC, class T>
__device__ inline void gather1d(gptr<const T> src, long long plane, int nx, int x,
                                typename Store<T>::A (&g)[3])
{
    using L = Lat<kD1Q3>;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int xs = x - L::vx(i);
        long long off;
        if constexpr (BC == kPeriodic) {
            off = i * plane + wrapi(xs, nx);
        } else {
            off = (xs >= 0 && xs < nx) ? i * plane + xs : L::opp(i) * plane + x;
        }
        g[i] = Store<T>::ld(src + off);
    }
}

// D1Q3: a.steps steps in one launch.  One site per thread; the populations that
// leave the sites stay in LDS from one step to the next (rounded to storage,
// as a store would), the outer sites of the workgroup go out of date by
// a.reach per step and are not written.  A small tube is bound by latency: one
// step per launch cost 6.5 us, of which a launch, the first load and the
// reduction are 5; kept in LDS a step costs its arithmetic and one or two
// barriers.  The sums, the mask and Delta S' belong to the last step alone.
template <class T, int QE, int DS, int BC, bool ELBM>
__global__ void __launch_bounds__(k1DMaxThreads) k_step1d(StepArgs a)
{
    using A = typename Store<T>::A;
    constexpr int LAT = kD1Q3;
    using L = Lat<LAT>;
    constexpr int Q = L::Q;
    __shared__ T leaving[2][Q][k1DMaxThreads];
    __shared__ A ds[k1DMaxThreads];
    __shared__ double red[k1DMaxThreads / kWave * kNStat];

    const int tidx = tile_of_block(a, 0);
    const Tile t = a.tiles[tidx];
    const DomainDev& D = a.dom[t.domain];
    const int tid = threadIdx.x;
    const int nx = D.nx;
    const long long plane = D.plane;
    const gptr<const T> src = to_global<T>(static_cast<const void*>(D.buf[a.parity]));
    const gptr<T> dst = to_global<T>(D.buf[1 - a.parity]);
    const A shift = A(D.shift), c = A(D.c);
    const long long step = a.counter[a.parity];
    // the index of the step after this launch, read by the next one (which reads buffer 1 - parity)
    if (blockIdx.x == 0 && tid == 0) a.counter[1 - a.parity] = step + a.steps;

    // the first threads take the tile's own sites, the others the halo (so that
    // the sums do not depend on a.steps)
    const int halo = a.reach * a.steps;
    const int pos = tid < k1DWidth ? tid + halo : (tid < k1DWidth + halo ? tid - k1DWidth : tid);
    const int xr = t.x0 - halo + pos;
    const int last_pos = t.x1 - t.x0 + 2 * halo - 1;
    const bool used = pos <= last_pos;
    const bool inside = used && (BC == kPeriodic || (xr >= 0 && xr < nx));
    const int x = BC == kPeriodic ? wrapi(xr, nx) : xr;
    const bool owned = inside && xr >= t.x0 && xr < t.x1;
    // neighbours in the workgroup (at the ends of its sites a site stands in for
    // the missing one: nothing that is written depends on it.  Not the LDS past a
    // short tile, see k_block2d: 64 steps of 800 FP64 ELBM sites took 250 to 720 us)
    const int tl = pos > 0 ? pos - 1 : 0, tr = pos < last_pos ? pos + 1 : last_pos;

    Acc acc;
    A g[Q];
    SiteState<LAT, A> S;
    SiteScalars sc;
    if (inside) gather1d<BC>(src, plane, nx, x, g);
    for (int n = 0; n < a.steps; ++n) {
        const bool last = n == a.steps - 1;
        A dsv = A(0);
        if (inside) {
            collide_site<LAT, QE, DS, ELBM>(g, shift, c, S, sc, owned && last);
            dsv = S.dpost;
            if (owned) {
                if (last) {
                    acc.moments(sc);
                    acc.fluid_site(sc, S.dpost);
                    if (a.flags & kFlagEntropy) {
                        const double e = entropy_site<LAT>(g, shift);
                        if (isfinite(e)) acc.ent += e;
                    }
                }
                if (x == D.probe_x) {
                    const gptr<float> p = to_global<float>(D.probe) + 2 * ((step + n) % D.probe_cap);
                    p[0] = sc.ux;
                    p[1] = 0.0f;
                }
            }
        }
        const bool median = D.limiter & kLimMedian;
        if (median) {
            ds[pos] = dsv;
            __syncthreads();
        }
        if (inside) {
            unsigned mask = 0;
            const bool has_med = median && (BC == kPeriodic || (x >= 1 && x <= nx - 2));
            const A med = has_med ? med3(ds[tl], ds[pos], ds[tr]) : A(0);
            A tgt;
            A phi = limiter_phi(S.dpost, has_med, med, D, mask, tgt);
            if constexpr (DS == kExactHom) {
                if (D.homothety && phi > A(0) && tgt < A(__builtin_huge_val()) && isfinite(S.dpost))
                    phi = exact_homothety<LAT>(S, shift, tgt, S.dpost);
            }
            bool posrule = S.posrule;
            if (D.limiter & kLimPos) {
                const A pp = positivity_phi<LAT>(S, shift);
                if (pp < A(1)) {
                    posrule = true;
                    if (last && owned) ++acc.pos;
                    phi = fmin(phi, pp);
                }
            }
            if (posrule) mask |= kMaskPos;
            const A k = phi * S.c;
            if (!last) {
#pragma unroll
                for (int i = 0; i < Q; ++i) st_shared<T>(&leaving[n & 1][i][pos], S.gs[i] - k * S.d[i]);
            } else if (owned) {
                if (S.posrule) ++acc.pos;
#pragma unroll
                for (int i = 0; i < Q; ++i) Store<T>::st(dst + i * plane + x, S.gs[i] - k * S.d[i]);
                if (mask & kMaskTrim) ++acc.trim;
                if (mask & kMaskMedian) ++acc.filt;
                if (phi < A(1) && isfinite(S.dpost))
                    acc.lim += double(S.dpost - delta_s_scaled<LAT, DS>(S, shift, S.c, phi));
                if (sc.nonpos) mask |= kMaskNonpos;
                if (a.flags & kFlagRecord) {
                    to_global<unsigned char>(D.mask)[x] = (unsigned char)mask;
                    to_global<double>(D.dS)[x] = double(S.dpost);
                }
                if (D.limiter & kLimEns) {
                    // for the ensemble pass: Delta S' and the factor applied here
                    Store<A>::st(to_global<A>(D.dsbuf) + x, S.dpost);
                    Store<A>::st(to_global<A>(D.phibuf) + x, phi);
                }
            }
        }
        if (last) break;
        // two buffers in turn: one barrier per step
        __syncthreads();
        if (inside) {
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const bool off = BC != kPeriodic && L::vx(i) != 0 && x == (L::vx(i) > 0 ? 0 : nx - 1);
                const int from = L::vx(i) == 0 ? pos : (L::vx(i) > 0 ? tl : tr);
                g[i] = off ? ld_shared<T>(&leaving[n & 1][L::opp(i)][pos]) : ld_shared<T>(&leaving[n & 1][i][from]);
            }
        }
    }
    store_partial(acc, partial_slot(a, 0, tidx), red);
}

// D1Q3 ensemble pass (after the step kernel and the E(Delta S') reduction):
// a site whose ensemble factor is below the factor the step kernel applied is
// moved further toward its f*, rebuilt from the stored state's moments:
// f* + (phi_ens / phi_applied)(f_stored - f*).
template <class T, int QE, int DS, int BC>
__global__ void __launch_bounds__(kThreads) k_ens1d(StepArgs a)
{
    using A = typename Store<T>::A;
    constexpr int LAT = kD1Q3;
    constexpr int Q = Lat<LAT>::Q;
    __shared__ double red[4 * kNStat];
    const int tidx = int(blockIdx.x);
    const Tile t = a.tiles[tidx];
    const DomainDev& D = a.dom[t.domain];
    const int x = t.x0 + int(threadIdx.x);
    AccT<A> acc;
    if ((D.limiter & kLimEns) && x < t.x1) {
        double ensv[kNEns];
#pragma unroll
        for (int k = 0; k < kNEns; ++k) ensv[k] = D.ens[k];
        const A d = Store<A>::ld(to_global<A>(static_cast<const void*>(D.dsbuf)) + x);
        const A pa = Store<A>::ld(to_global<A>(static_cast<const void*>(D.phibuf)) + x);
        A tgt = A(__builtin_huge_val()), fac = A(1);
        SecondHit h;
        ens_terms(D, ensv, d, tgt, fac, h);
        if (h.bits) {
            acc.ens += h.ens;
            acc.trim += h.trim;
            if (a.flags & kFlagRecord) to_global<unsigned char>(D.mask)[x] |= (unsigned char)h.bits;
            const A pq = fmin(fac, tgt < A(__builtin_huge_val()) ? sqrt_(tgt * rcp(d)) : A(1));
            bool exact = false;
            if constexpr (DS == kExactHom) exact = D.homothety && isfinite(d) && pa > A(0);
            if (exact || pq < pa) {
                const long long plane = D.plane;
                const A shift = A(D.shift);
                const gptr<const T> lsrc = to_global<T>(static_cast<const void*>(D.buf[1 - a.parity]));
                const gptr<T> dst = to_global<T>(D.buf[1 - a.parity]);
                A gl[Q], gs[Q];
#pragma unroll
                for (int i = 0; i < Q; ++i) gl[i] = Store<T>::ld(lsrc + (i * plane + x));
                A dr, jx, jy, rho, ux, uy;
                moments_equilibrium<LAT, QE>(gl, shift, dr, jx, jy, rho, ux, uy, gs);
                A fs[Q], e[Q];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    fs[i] = A(Lat<LAT>::w(i)) * shift + gs[i];
                    e[i] = (gl[i] - gs[i]) * rcp(fs[i]);
                }
                A r = pq * rcp(pa);
                if constexpr (DS == kExactHom) {
                    if (exact) {
                        // exact homothety from f' = f* + e / pa (Sec. 3.6)
                        A xp[Q];
#pragma unroll
                        for (int i = 0; i < Q; ++i) xp[i] = e[i] / pa;
                        A ph = fac;
                        if (tgt < d) ph = fmin(ph, kullback_scale<Q>(fs, xp, tgt, sqrt_(tgt * rcp(d)), A(0), A(1)));
                        r = ph / pa;
                    }
                }
                if (r < A(1)) {
#pragma unroll
                    for (int i = 0; i < Q; ++i) Store<T>::st(dst + (i * plane + x), gs[i] + r * (gl[i] - gs[i]));
                    if (isfinite(d)) {
                        A ds_old, ds_new;
                        if constexpr (DS == kQuad) {
                            ds_old = pa * pa * d;
                            ds_new = r * r * pa * pa * d;
                        } else {
                            ds_old = kull_sum<false>(fs, e, A(1));
                            ds_new = kull_sum<false>(fs, e, r);
                        }
                        // the step kernel counted d - Delta S(stored)
                        acc.lim += ds_old - ds_new;
                    }
                }
            }
        }
    }
    store_partial(acc, partial_slot(a, 1, tidx), red);
}

// one instantiation per (quasiequilibrium, Delta S form, boundary) in use: the
// 2-D kernels serve periodic and cavity grids, the 1-D ones periodic and tube,
// ELBM the entropic f* only.  `f` launches for the three as constants.
template <int B0, int B1, bool ELBM = false, class F>
static hipError_t dispatch(int qe, int ds, int bc, F f)
{
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    auto with_bc = [&](auto q, auto d) {
        if (bc == B0) f(q, d, std::integral_constant<int, B0>());
        else if (bc == B1) f(q, d, std::integral_constant<int, B1>());
        else return hipErrorInvalidValue;
        return hipSuccess;
    };
    auto with_ds = [&](auto q) {
        if (ds == kExact) return with_bc(q, std::integral_constant<int, kExact>());
        if (ds == kQuad) return with_bc(q, std::integral_constant<int, kQuad>());
        return ds == kExactHom ? with_bc(q, std::integral_constant<int, kExactHom>()) : hipErrorInvalidValue;
    };
    hipError_t e = hipErrorInvalidValue;
    if (qe == 1) e = with_ds(I1());
    if constexpr (!ELBM) {
        if (qe == 0) e = with_ds(I0());
    }
    return e == hipSuccess ? hipGetLastError() : e;
}
// a launch of KER<storage, f*, Delta S form, boundary, ...>
#define LBM_LAUNCH_LDS(GRID, BLOCK, LDS, KER, ...)                                                       \
    [&](auto q, auto d, auto b) {                                                                        \
        constexpr int QE = decltype(q)::value, DS = decltype(d)::value, BC = decltype(b)::value;         \
        hipLaunchKernelGGL((KER<StT, QE, DS, BC, ##__VA_ARGS__>), dim3(GRID), dim3(BLOCK), LDS, s, a);    \
    }
#define LBM_LAUNCH(GRID, BLOCK, KER, ...) LBM_LAUNCH_LDS(GRID, BLOCK, 0, KER, ##__VA_ARGS__)

hipError_t LBM_CAT(launch_step2d, LBM_SUFFIX)(int qe, int ds, int bc, const StepArgs& a, int kernel,
                                             hipStream_t s)
{
    const bool stats = a.flags & kFlagStats;
    if (kernel == 0)
        return stats ? dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.nblocks, kThreads, k_collide2d, false, true))
                     : dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH_LDS(a.nblocks, kThreads, a.collide_lds, k_collide2d, false, false));
    if (kernel == 2)
        return stats ? dispatch<0, 1, true>(qe, ds, bc, LBM_LAUNCH(a.nblocks, kThreads, k_collide2d, true, true))
                     : dispatch<0, 1, true>(qe, ds, bc, LBM_LAUNCH(a.nblocks, kThreads, k_collide2d, true, false));
    if (kernel == 3)
        return stats ? dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.ntiles, kThreads, k_fused2d, true))
                     : dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH_LDS(a.ntiles, kThreads, a.fused_lds, k_fused2d, false));
    if (kernel == 5) {
        const int halo = 2 * a.steps - 1;
        const int threads = ((a.block_w + 2 * halo) * (a.block_h + 2 * halo) + kWave - 1) / kWave * kWave;
        if (a.steps > 1) return dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.ntiles, threads, k_block2d, false, true));
        return stats ? dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.ntiles, threads, k_block2d, true, false))
                     : dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.ntiles, threads, k_block2d, false, false));
    }
    if (kernel == 4) return dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.nblocks, kThreads, k_form2d));
    if (a.elbm)
        return a.ens_pass ? dispatch<0, 1, true>(qe, ds, bc, LBM_LAUNCH(a.ntiles, kThreads, k_median_ens2d, true))
                          : dispatch<0, 1, true>(qe, ds, bc, LBM_LAUNCH(a.ntiles, kThreads, k_median2d, true));
    if constexpr (sizeof(StT) >= 4) {
        if (a.in_place)
            return a.ens_pass ? dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.ntiles, kThreads, k_median_ens2d, true))
                              : dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.ntiles, kThreads, k_median2d, true));
    }
    return a.ens_pass ? dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.ntiles, kThreads, k_median_ens2d, false))
                      : dispatch<0, 1>(qe, ds, bc, LBM_LAUNCH(a.ntiles, kThreads, k_median2d, false));
}

hipError_t LBM_CAT(launch_step1d, LBM_SUFFIX)(int qe, int ds, int bc, const StepArgs& a, int kernel,
                                             hipStream_t s)
{
    const int threads = threads1d(a.reach, a.steps);
    if (kernel == 0) return dispatch<0, 2>(qe, ds, bc, LBM_LAUNCH(a.ntiles, threads, k_step1d, false));
    if (kernel == 2) return dispatch<0, 2, true>(qe, ds, bc, LBM_LAUNCH(a.ntiles, threads, k_step1d, true));
    return dispatch<0, 2>(qe, ds, bc, LBM_LAUNCH(a.ntiles, threads1d(0, 0), k_ens1d));
}

}  // namespace lbm

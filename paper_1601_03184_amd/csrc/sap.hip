// sap.hip -- the Schwarz alternating procedure on all right-hand sides at once.
//
// One launch per colour half-sweep, for one operator or a batch of several (lattices of
// uneven size, each with its own right-hand sides).  Workgroup = one SAP block of that
// colour x a tile of T right-hand sides; thread (off, t) owns one site of the block and
// one right-hand side.  The workgroup
//   1. forms the residual r = b - D x on its block: the full stencil on a first visit from a
//      guess, afterwards the block's kept residual (even-odd: formed again from b and the stored
//      x) minus the hops across its faces, which the neighbours left, spin-projected and multiplied by
//      the link, in face buffers (read once and in order, a quarter of the loads of reading the
//      neighbours' spinors across the faces; all of them in flight at once),
//   2. runs n_mr minimal-residual steps on the block operator D_j = I_j^T D I_j with the
//      block residual rho kept in LDS ([24][Vb][T], conflict-free for the thread order),
//      the two inner products per step reduced across the block with lane exchanges
//      and one LDS exchange, and the correction e kept in registers,
//   3. writes x|_j (+)= e, its residual and its own faces.
// Bound by the vector units: an MR step issues 8 us of instructions per workgroup (of 9), and at tile
// 4 the one workgroup of a CU has nothing to run beside its loads and stores (of about 55 us 9 for the
// residual, 3-10 for the end).  32^3 x 64, 32 right-hand sides in FP32, 3 x 4, tile 4: 49.5 -> 46.5 ms per call
// with the face buffers (the 15 vector sets that a call must move take 22 ms at 4.4 TB/s), 42.2 with the reductions
// by lane exchanges, 16-byte LDS vectors and the end of a visit without spills; the even-odd solver, which
// formed the full residual at every visit from global memory, 3.34 -> 2.70 ms at 16^3 x 32 with 24, 3 x 3 (2.60
// with a kept Schur residual, which the roundings of x left: see sap_block_eo).
// The links and clover of a site are loaded once per stencil for all T lanes of the site.
// With the even-odd block solver (k_sap_batched_eo) step 2 runs on the block's Schur
// complement over its even sites instead (sap_block_eo).
#include <algorithm>

#include "launch.h"
#include "stencil.h"

#include <type_traits>

namespace {

// Faces of a block: for every direction mu with more than one block, the +mu face and then the
// -mu face, each [12 / n][face sites][S] component vectors of n numbers (16 bytes).
struct FaceGeo {
    int base[4];   // first vector of direction mu's faces, in units of S
    int vf[4];     // face sites
    int fs[4][4];  // strides of the other coordinates in the face-site index
    int per_blk;   // vectors of one block, in units of S
};

// 16-byte component vectors: type in LDS, mem in the caller's workspace, which is aligned to the
// arithmetic type and to no more (a 16-byte load takes any multiple of 4 bytes)
template <typename Tc> struct V16 {
    static constexpr int n = 16 / sizeof(Tc);
    typedef Tc type __attribute__((ext_vector_type(16 / sizeof(Tc))));
    typedef Tc mem __attribute__((ext_vector_type(16 / sizeof(Tc)), aligned(alignof(Tc))));
};
static_assert(alignof(V16<float>::mem) == alignof(float) && alignof(V16<double>::mem) == alignof(double),
              "the workspace needs no more than the arithmetic type's alignment");

template <typename Tc> FaceGeo face_geo(const KGeo &g)
{
    FaceGeo f{};
    int base = 0;
    for (int mu = 0; mu < 4; ++mu) {
        f.vf[mu] = g.Vb / g.b[mu];
        f.base[mu] = base;
        if (g.nb[mu] > 1) base += 2 * (12 / V16<Tc>::n) * f.vf[mu];
        for (int nu = 0; nu < 4; ++nu)
            f.fs[mu][nu] = nu < mu ? g.ostr[nu] : nu > mu ? g.ostr[nu] / g.b[mu] : 0;
    }
    f.per_blk = base;
    return f;
}

// numbers of the face buffer for n_rhs right-hand sides
template <typename Tc> size_t face_elems(const mrhs_op *op, int n_rhs)
{
    const size_t ngrp = (n_rhs + op->k.S - 1) / op->k.S;
    return ngrp * op->k.nblk * face_geo<Tc>(op->k).per_blk * op->k.S * V16<Tc>::n;
}

template <typename Ts, typename Tc> struct SapArgs {
    KGeo g;
    const Tc *links, *clover;
    const uint32_t *blk_coords, *loc_coords;
    const int32_t *blocks;  // block ids of this colour
    int nblocks;            // number of blocks of this colour
    int ntiles;             // right-hand-side tiles per block
    int mode;               // 0: x = 0 everywhere; 1: x = 0 on this colour's blocks; 2: general
    int n_mr;
    const Ts *b;
    const Ts *xr;           // where neighbours' x is read (x itself, or a snapshot)
    Ts *x;
    Ts *xw;                 // where the new x is written (x itself, or a caller's other vectors)
    // plain MR: kept per block between the visits of a colour (arithmetic type, component vectors of 16
    // bytes: sig_ptr).  inc: the block residual rho after the last visit; a later visit's residual is
    // rho minus the face hops of the neighbours' changes of x since.  Every neighbour has changed
    // once since then, the last time it was visited, and left its hops of that change in the
    // face buffer.  Otherwise (FP32 plain MR where a block can neighbour one of its own colour)
    // sigma = b - D_j x_j, a later visit's residual being sigma minus the face hops of x, which
    // then are what the face buffer holds.
    Tc *sig;
    int sig_in;             // a later visit: this colour's rho or sigma is valid, the neighbours' faces are
    int sig_out;            // write it for the next visit of this colour
    int inc;
    // Every block's outgoing hops across its faces: per face site the two spin rows (1 -+ g_mu)
    // U_mu applied to its last change of x (or to x), which the neighbour adds up.  With an odd number
    // of blocks in a direction the blocks at its ends have the same colour and are visited together: the
    // buffers then alternate from sweep to sweep, a visit reading neighbours of the other colour
    // from face_o, those of its own colour from face_s (null: not visited yet, x = 0).
    Tc *face_w;
    const Tc *face_o, *face_s;
    FaceGeo fg;
    int f_out;              // write this visit's faces (a later visit reads them)
    // even-odd block solver: A^-1 per site (clover layout), block offsets in parity order,
    // number of even sites of a block
    const Tc *cloverinv;
    const int32_t *eo_sites;
    int Ve;
};

// The block residual rho lives in LDS in component vectors of n numbers, [24 / n][Vb][T]: lane
// (off, t) reads vector v at (v * Vb + off) * T + t, consecutive lanes consecutive vectors.  Plain
// MR takes 16-byte vectors (half the LDS instructions and addresses of (re, im) pairs: with the lane
// exchanges of mr_alpha 7.8 -> 7.1 ms per half-sweep at 32^3 x 64, 32 right-hand sides, tile 4); the
// even-odd kernel pairs, whose smaller load groups keep it within its registers.
template <typename Tc> using LdsVec = typename V16<Tc>::type;
template <typename Tc> using LdsPair = typename Vec2<Tc>::type;

// complex component k of a vector
template <typename LV, typename Tc> __device__ inline void vec_get(const LV &q, int k, Tc &re, Tc &im)
{
    if constexpr (std::is_same<LV, LdsPair<Tc>>::value) {
        re = q.x;
        im = q.y;
    } else {
        re = q[2 * k];
        im = q[2 * k + 1];
    }
}
template <typename LV, typename Tc> __device__ inline void vec_set(LV &q, int k, Tc re, Tc im)
{
    if constexpr (std::is_same<LV, LdsPair<Tc>>::value) {
        q = {re, im};
    } else {
        q[2 * k] = re;
        q[2 * k + 1] = im;
    }
}

// the components of s in the vectors [V0, V1)
template <int V0, int V1, typename Tc, typename LV>
__device__ inline void lds_load_range(const LV *rho, int str, int idx, Spinor<Tc> &s)
{
    constexpr int n = int(sizeof(LV) / sizeof(Tc)) / 2;  // complex components of a vector
#pragma unroll
    for (int v = V0; v < V1; ++v) {
        const LV q = rho[v * str + idx];
#pragma unroll
        for (int c = 0; c < n; ++c) vec_get(q, c, s.re[v * n + c], s.im[v * n + c]);
    }
}

template <typename Tc, typename LV> __device__ inline void lds_load(const LV *rho, int str, int idx, Spinor<Tc> &s)
{
    lds_load_range<0, 24 / int(sizeof(LV) / sizeof(Tc))>(rho, str, idx, s);
}

// components 6 HF .. 6 HF + 5 (one chiral half) only
template <int HF, typename Tc, typename LV>
__device__ inline void lds_load_half(const LV *rho, int str, int idx, Spinor<Tc> &s)
{
    constexpr int h = 12 / int(sizeof(LV) / sizeof(Tc));
    lds_load_range<HF * h, (HF + 1) * h>(rho, str, idx, s);
}

template <typename Tc, typename LV> __device__ inline void lds_store(LV *rho, int str, int idx, const Spinor<Tc> &s)
{
    constexpr int n = int(sizeof(LV) / sizeof(Tc)) / 2;  // complex components of a vector
#pragma unroll
    for (int v = 0; v < 12 / n; ++v) {
        LV q;
#pragma unroll
        for (int c = 0; c < n; ++c) vec_set(q, c, s.re[v * n + c], s.im[v * n + c]);
        rho[v * str + idx] = q;
    }
}

// one MR update on this lane's slot: e += alpha rho, rho -= alpha q
template <typename Tc, typename LV>
__device__ inline void mr_update(LV *rho, int str, int idx, Tc ar, Tc ai, const Spinor<Tc> &q, Spinor<Tc> &e)
{
    constexpr int n = int(sizeof(LV) / sizeof(Tc)) / 2;  // complex components of a vector
#pragma unroll
    for (int v = 0; v < 12 / n; ++v) {
        const LV o = rho[v * str + idx];
        LV w;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const int c = v * n + k;
            Tc nr, ni;
            vec_get(o, k, nr, ni);
            e.re[c] += ar * nr;
            e.re[c] -= ai * ni;
            e.im[c] += ar * ni;
            e.im[c] += ai * nr;
            nr -= ar * q.re[c];
            nr += ai * q.im[c];
            ni -= ar * q.im[c];
            ni -= ai * q.re[c];
            vec_set(w, k, nr, ni);
        }
        rho[v * str + idx] = w;
    }
}

// this lane's share of <q,q> and <q,rho>
template <typename Tc, typename LV>
__device__ inline void mr_products(const LV *rho, int str, int idx, const Spinor<Tc> &q, Tc &qq, Tc &qrr,
                                            Tc &qri)
{
    constexpr int n = int(sizeof(LV) / sizeof(Tc)) / 2;  // complex components of a vector
#pragma unroll
    for (int v = 0; v < 12 / n; ++v) {
        const LV o = rho[v * str + idx];
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const int c = v * n + k;
            Tc pr, pi;
            vec_get(o, k, pr, pi);
            qq += q.re[c] * q.re[c];
            qq += q.im[c] * q.im[c];
            qrr += q.re[c] * pr;
            qrr += q.im[c] * pi;
            qri += q.re[c] * pi;
            qri -= q.im[c] * pr;
        }
    }
}

// The links a block operator uses, staged in LDS once per workgroup (the "links in LDS"
// variants): U_mu(x) for the block's sites x whose
// +mu neighbour is inside the block (local coordinate l_mu < b_mu - 1; every site when the
// block spans the lattice in mu and keeps its wrap-around hop).  Per direction they form a
// box of extents e_mu,nu = b_nu, except e_mu,mu = b_mu - 1, stored lexicographically after
// the boxes of the lower directions, 18 reals per link.
//
// A tile of T right-hand sides stages the first T directions: what a 4^4 block's workgroups can
// hold in the 160 KiB of a CU beside rho, as many of them as their registers allow (FP32: one at
// tile 4, two at tile 2, four at tile 1; FP64 half as many).  The other directions are read through L1
// in every MR step, 72 bytes per lane and hop in FP32, which bounds the small tiles; us without / with,
// 3 x 4: FP32 16^3 x 32 n 24 tile 1 3645 / 3359, tile 2 2467 / 2278, 16^4 n 20 tile 2 1208 / 1118; FP64
// 12^3 x 24 n 10 tile 1 1170 / 1091, tile 2 880 / 836; 4^4 and 8^4 within 2 %.
constexpr int staged_links(int T) { return T; }
struct LinkBox {
    int base[4];  // first link of direction mu
    int s[4][4];  // lexicographic strides of direction mu's box
    int n;        // links in all four boxes
};

__host__ __device__ inline LinkBox link_box(const KGeo &g)
{
    LinkBox lb;
    int base = 0;
    for (int mu = 0; mu < 4; ++mu) {
        int st = 1;
        for (int nu = 0; nu < 4; ++nu) {
            lb.s[mu][nu] = st;
            st *= (nu == mu && g.nb[mu] > 1) ? g.b[nu] - 1 : g.b[nu];
        }
        lb.base[mu] = base;
        base += st;
    }
    lb.n = base;
    return lb;
}

template <typename Tf, typename T> __device__ inline void lds_link(const Tf *ul, int idx, T (&U)[18])
{
    using V2 = typename Vec2<Tf>::type;
    const V2 *p = reinterpret_cast<const V2 *>(ul + idx * 18);
#pragma unroll
    for (int c = 0; c < 9; ++c) {
        const V2 v = p[c];
        U[2 * c] = (T)v.x;
        U[2 * c + 1] = (T)v.y;
    }
}

// q += hops of D_j rho at site off (lane t), rho from LDS; hops leaving the block dropped.
// ns is the site's native index (opaque to the compiler, so the link loads stay inside
// the MR loop).  With ul (links in LDS) the links come from there: cf is the site's index
// in direction MU's box, sb the box's stride in MU.
template <int MU, typename Tc, bool LL = false, typename LV>
__device__ inline void block_hops(const KGeo &g, const Tc *__restrict__ links, const LV *rho,
                                  int T, int ns, int off, int t, uint32_t lcp, Spinor<Tc> &q,
                                  const Tc *ul = nullptr, int cf = 0, int sb = 0)
{
    const int str = g.Vb * T;
    const int l = unpack_coord(lcp, MU);
    int noff = -1;
    if (l + 1 < g.b[MU]) noff = off + g.ostr[MU];
    else if (g.nb[MU] == 1) noff = off - (g.b[MU] - 1) * g.ostr[MU];
    if (noff >= 0) {
        Spinor<Tc> chi;
        lds_load<Tc>(rho, str, noff * T + t, chi);
        Tc U[18];
        if constexpr (LL) lds_link(ul, cf, U);
        else load_link(links, g.V, MU, ns, U);
        hop_accumulate<MU, -1, false>(U, chi, q);
    }
    hop_fence(q);
    noff = -1;
    int cb = 0;
    if (l > 0) {
        noff = off - g.ostr[MU];
        cb = cf - sb;
    } else if (g.nb[MU] == 1) {
        noff = off + (g.b[MU] - 1) * g.ostr[MU];
        cb = cf + (g.b[MU] - 1) * sb;
    }
    if (noff >= 0) {
        Spinor<Tc> chi;
        lds_load<Tc>(rho, str, noff * T + t, chi);
        Tc U[18];
        if constexpr (LL) lds_link(ul, cb, U);
        else load_link(links, g.V, MU, ns + (noff - off), U);
        hop_accumulate<MU, +1, true>(U, chi, q);
    }
}

// a site's entry of a block set in component vectors of 16 bytes, [group][block][24 / n][Vb][S]:
// what is kept between visits is read and written by this kernel alone, so it takes a layout of
// its own with a quarter of the load and store instructions of the native one
template <typename Tc>
__device__ __forceinline__ typename V16<Tc>::mem *sig_ptr(const KGeo &g, Tc *sig, int grp, int blk, int off, int tt)
{
    using V = typename V16<Tc>::mem;
    V *base = reinterpret_cast<V *>(sig) + ((size_t)grp * g.nblk + blk) * (24 / V16<Tc>::n) * (size_t)(g.Vb * g.S);
    return base + (uint32_t)(off * g.S + tt);
}

template <typename Tc>
__device__ __forceinline__ void sig_load(const KGeo &g, Tc *sig, int grp, int blk, int off, int tt, Spinor<Tc> &s)
{
    constexpr int n = V16<Tc>::n;
    const typename V16<Tc>::mem *p = sig_ptr(g, sig, grp, blk, off, tt);
    const uint32_t str = (uint32_t)(g.Vb * g.S);
#pragma unroll
    for (int v = 0; v < 24 / n; ++v) {
        const typename V16<Tc>::type q = p[v * str];
#pragma unroll
        for (int c = 0; c < n; c += 2) {
            s.re[(v * n + c) / 2] = q[c];
            s.im[(v * n + c) / 2] = q[c + 1];
        }
    }
}

template <typename Tc>
__device__ __forceinline__ void sig_store(const KGeo &g, Tc *sig, int grp, int blk, int off, int tt,
                                          const Spinor<Tc> &s)
{
    constexpr int n = V16<Tc>::n;
    typename V16<Tc>::mem *p = sig_ptr(g, sig, grp, blk, off, tt);
    const uint32_t str = (uint32_t)(g.Vb * g.S);
#pragma unroll
    for (int v = 0; v < 24 / n; ++v) {
        typename V16<Tc>::type q;
#pragma unroll
        for (int c = 0; c < n; c += 2) {
            q[c] = s.re[(v * n + c) / 2];
            q[c + 1] = s.im[(v * n + c) / 2];
        }
        p[v * str] = q;
    }
}

// two spin rows of three colours, complex
template <typename Tc> struct HalfSpinor {
    Tc re[2][3], im[2][3];
};

// first component vector of a site's entry on face `minus` of direction MU of block blk
template <int MU, typename Ts, typename Tc, typename Tp>
__device__ __forceinline__ auto face_ptr(const SapArgs<Ts, Tc> &a, Tp *face, int grp, int blk, bool minus, int f,
                                         int tt)
{
    using V = std::conditional_t<std::is_const<Tp>::value, const typename V16<Tc>::mem, typename V16<Tc>::mem>;
    const KGeo &g = a.g;
    V *base = reinterpret_cast<V *>(face) + ((size_t)grp * g.nblk + blk) * (size_t)(a.fg.per_blk * g.S);
    return base + (uint32_t)((a.fg.base[MU] + (minus ? (12 / V16<Tc>::n) * a.fg.vf[MU] : 0) + f) * g.S + tt);
}

template <int MU, typename Ts, typename Tc>
__device__ __forceinline__ int face_index(const SapArgs<Ts, Tc> &a, uint32_t lcp)
{
    int f = 0;
#pragma unroll
    for (int nu = 0; nu < 4; ++nu)
        if (nu != MU) f += unpack_coord(lcp, nu) * a.fg.fs[MU][nu];
    return f;
}

// block across the +MU (minus: -MU) face of a block with block coordinate bc in direction MU
template <int MU> __device__ __forceinline__ int face_nbr(const KGeo &g, int blk, int bc, bool minus)
{
    const int wrap = (g.nb[MU] - 1) * g.bstr[MU];
    return minus ? blk + (bc > 0 ? -g.bstr[MU] : wrap) : blk + (bc + 1 < g.nb[MU] ? g.bstr[MU] : -wrap);
}

// the block across the +MU face (fwd) or the -MU face has the block's own colour
template <int MU> __device__ __forceinline__ bool own_colour(const KGeo &g, int bc, bool fwd)
{
    return (g.nb[MU] & 1) && bc == (fwd ? g.nb[MU] - 1 : 0);
}

// What the neighbour across the +MU face (fwd) or the -MU face left for this site
template <int MU, typename Ts, typename Tc>
__device__ __forceinline__ void face_load(const SapArgs<Ts, Tc> &a, int grp, int blk, uint32_t bcp, uint32_t lcp,
                                          int tt, bool fwd, HalfSpinor<Tc> &w)
{
    constexpr int n = V16<Tc>::n;
    const int bc = unpack_coord(bcp, MU);
    // both neighbours are uniform over the workgroup, the choice is the lane's
    const int nf = face_nbr<MU>(a.g, blk, bc, false), nb = face_nbr<MU>(a.g, blk, bc, true);
    const Tc *bf = own_colour<MU>(a.g, bc, true) ? a.face_s : a.face_o;
    const Tc *bb = own_colour<MU>(a.g, bc, false) ? a.face_s : a.face_o;
    const auto *p = face_ptr<MU>(a, fwd ? bf : bb, grp, fwd ? nf : nb, fwd, face_index<MU>(a, lcp), tt);
    const uint32_t str = (uint32_t)(a.fg.vf[MU] * a.g.S);
#pragma unroll
    for (int v = 0; v < 12 / n; ++v) {
        const typename V16<Tc>::type q = p[v * str];
#pragma unroll
        for (int c = 0; c < n; c += 2) {
            const int k = (v * n + c) / 2;
            w.re[k / 3][k % 3] = q[c];
            w.im[k / 3][k % 3] = q[c + 1];
        }
    }
}

// r += the hop whose two upper spin rows are w: rows 2, 3 are sg g_MU's rows of it, sg = -1 for
// the forward hop (1 - g_MU), +1 for the backward one
template <int MU, typename Tc> __device__ __forceinline__ void face_add(const HalfSpinor<Tc> &w, Tc sg, Spinor<Tc> &r)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        Tc t2r, t2i, t3r, t3i;
        mul_ipow<gphase(MU, 2)>(w.re[gperm(MU, 2)][c], w.im[gperm(MU, 2)][c], t2r, t2i);
        mul_ipow<gphase(MU, 3)>(w.re[gperm(MU, 3)][c], w.im[gperm(MU, 3)][c], t3r, t3i);
        r.re[c] += w.re[0][c];
        r.im[c] += w.im[0][c];
        r.re[3 + c] += w.re[1][c];
        r.im[3 + c] += w.im[1][c];
        r.re[6 + c] += sg * t2r;
        r.im[6 + c] += sg * t2i;
        r.re[9 + c] += sg * t3r;
        r.im[9 + c] += sg * t3i;
    }
}

// r += the hops across the block's faces, from the neighbours' face entries.  A site lies on at
// most one of the two faces of a direction unless its block is one site thick there (then the
// backward face follows); the loads of ND directions are issued before their arithmetic.
template <int MU0, int ND, typename Ts, typename Tc>
__device__ __forceinline__ void face_round(const SapArgs<Ts, Tc> &a, int grp, int blk, uint32_t bcp, uint32_t lcp,
                                           int tt, Spinor<Tc> &r)
{
    const KGeo &g = a.g;
    HalfSpinor<Tc> w[ND];
    // the lane is on the face (and the neighbour there has been visited)
    auto fwd = [&](auto m) __attribute__((always_inline)) {
        constexpr int MU = decltype(m)::value;
        return unpack_coord(lcp, MU) + 1 == g.b[MU] && g.nb[MU] > 1 &&
               (a.face_s || !own_colour<MU>(g, unpack_coord(bcp, MU), true));
    };
    auto bwd = [&](auto m) __attribute__((always_inline)) {
        constexpr int MU = decltype(m)::value;
        return unpack_coord(lcp, MU) == 0 && g.nb[MU] > 1 &&
               (a.face_s || !own_colour<MU>(g, unpack_coord(bcp, MU), false));
    };
    auto load = [&](auto m) __attribute__((always_inline)) {
        constexpr int MU = MU0 + decltype(m)::value;
        std::integral_constant<int, MU> mu;
        const bool ff = fwd(mu);
        if (ff || bwd(mu)) face_load<MU>(a, grp, blk, bcp, lcp, tt, ff, w[MU - MU0]);
    };
    auto add = [&](auto m) __attribute__((always_inline)) {
        constexpr int MU = MU0 + decltype(m)::value;
        std::integral_constant<int, MU> mu;
        const bool ff = fwd(mu);
        if (ff || bwd(mu)) face_add<MU>(w[MU - MU0], ff ? Tc(-1) : Tc(1), r);
        if (g.b[MU] == 1 && ff && bwd(mu)) {  // uniform: the site is on the backward face as well
            HalfSpinor<Tc> v;
            face_load<MU>(a, grp, blk, bcp, lcp, tt, false, v);
            face_add<MU>(v, Tc(1), r);
        }
    };
    load(std::integral_constant<int, 0>{});
    load(std::integral_constant<int, 1>{});
    if constexpr (ND == 4) {
        load(std::integral_constant<int, 2>{});
        load(std::integral_constant<int, 3>{});
    }
    sched_fence();
    add(std::integral_constant<int, 0>{});
    add(std::integral_constant<int, 1>{});
    if constexpr (ND == 4) {
        add(std::integral_constant<int, 2>{});
        add(std::integral_constant<int, 3>{});
    }
}

// f = the hops across the block's faces, summed in the order of the full stencil
template <typename Ts, typename Tc>
__device__ __forceinline__ void face_sum(const SapArgs<Ts, Tc> &a, int grp, int blk, uint32_t bcp, uint32_t lcp, int tt,
                                         Spinor<Tc> &f)
{
    spinor_zero(f);
    if constexpr (sizeof(Tc) == 4) {
        face_round<0, 4>(a, grp, blk, bcp, lcp, tt, f);
    } else {
        face_round<0, 2>(a, grp, blk, bcp, lcp, tt, f);
        face_round<2, 2>(a, grp, blk, bcp, lcp, tt, f);
    }
}

// A site's outgoing hops across its faces, for the neighbours' next visits: on the +MU face the
// neighbour's backward hop U^dag (1 + g_MU) e with the site's own link, on the -MU face the
// neighbour's forward hop U (1 - g_MU) e with the neighbour's link.  The lane's face (fwd) selects
// the element order and the sign of the link's imaginary part, so that lanes of both faces share
// one pass.
template <typename Tc> struct FaceLink {
    typename Vec2<Tc>::type u[9];
};

template <int MU, typename Ts, typename Tc>
__device__ __forceinline__ void face_link(const SapArgs<Ts, Tc> &a, int blk, int off, uint32_t bcp, bool fwd,
                                          FaceLink<Tc> &l)
{
    using V2 = typename Vec2<Tc>::type;
    const KGeo &g = a.g;
    const int nb = face_nbr<MU>(g, blk, unpack_coord(bcp, MU), true);
    const int ls = fwd ? blk * g.Vb + off : nb * g.Vb + off + (g.b[MU] - 1) * g.ostr[MU];
    const V2 *U = reinterpret_cast<const V2 *>(a.links + ((size_t)(uint32_t)ls * 4 + MU) * 18);
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) l.u[3 * r + c] = U[r == c ? 4 * r : fwd ? 3 * c + r : 3 * r + c];
}

template <int MU, typename Tc>
__device__ __forceinline__ void face_hop(const FaceLink<Tc> &l, bool fwd, const Spinor<Tc> &e, HalfSpinor<Tc> &w)
{
    const Tc sg = fwd ? Tc(1) : Tc(-1);
    Tc hr[2][3], hi[2][3];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            Tc tr, ti;
            if (r == 0) mul_ipow<gphase(MU, 0)>(e.re[3 * gperm(MU, 0) + c], e.im[3 * gperm(MU, 0) + c], tr, ti);
            else mul_ipow<gphase(MU, 1)>(e.re[3 * gperm(MU, 1) + c], e.im[3 * gperm(MU, 1) + c], tr, ti);
            hr[r][c] = e.re[3 * r + c] + sg * tr;
            hi[r][c] = e.im[3 * r + c] + sg * ti;
        }
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            Tc sr = 0, si = 0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const Tc ur = l.u[3 * x + c].x, ui = -sg * l.u[3 * x + c].y;
                sr += ur * hr[r][c];
                sr -= ui * hi[r][c];
                si += ur * hi[r][c];
                si += ui * hr[r][c];
            }
            w.re[r][x] = sr;
            w.im[r][x] = si;
        }
}

template <int MU, typename Ts, typename Tc>
__device__ __forceinline__ void face_store(const SapArgs<Ts, Tc> &a, int grp, int blk, uint32_t lcp, int tt, bool fwd,
                                           const HalfSpinor<Tc> &w)
{
    constexpr int n = V16<Tc>::n;
    typename V16<Tc>::mem *p = face_ptr<MU>(a, a.face_w, grp, blk, !fwd, face_index<MU>(a, lcp), tt);
    const uint32_t str = (uint32_t)(a.fg.vf[MU] * a.g.S);
#pragma unroll
    for (int v = 0; v < 12 / n; ++v) {
        typename V16<Tc>::type q;
#pragma unroll
        for (int c = 0; c < n; c += 2) {
            const int k = (v * n + c) / 2;
            q[c] = w.re[k / 3][k % 3];
            q[c + 1] = w.im[k / 3][k % 3];
        }
        p[v * str] = q;
    }
}

// The end of a visit on one site: x = e or with add x + e, the faces of the change of the stored x (the correction
// as rounded to the storage type; without inc of x) and, with inc, rho for later visits (keep():
// stores it).  The links of two directions are loaded ahead.
template <typename Ts, typename Tc, typename Keep>
__device__ __forceinline__ void finish_site(const SapArgs<Ts, Tc> &a, int grp, int blk, int off, uint32_t bcp,
                                            uint32_t lcp, int tt, Spinor<Tc> &e, bool add, Keep keep)
{
    const KGeo &g = a.g;
    sched_fence();
    bool ff[4], on[4];
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        const int l = unpack_coord(lcp, mu);
        ff[mu] = l + 1 == g.b[mu];
        on[mu] = a.f_out && g.nb[mu] > 1 && (ff[mu] || l == 0);
    }
    FaceLink<Tc> l0, l1;
    HalfSpinor<Tc> w;
    if (on[0]) face_link<0>(a, blk, off, bcp, ff[0], l0);
    if (on[1]) face_link<1>(a, blk, off, bcp, ff[1], l1);
    Spinor<Tc> xn;
    if (add) {
        Spinor<Tc> xo;
        load_spinor<Tc>(g, a.x, grp, blk, off, tt, xo);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            xn.re[c] = xo.re[c] + e.re[c];
            xn.im[c] = xo.im[c] + e.im[c];
            Ts sr = store_as<Ts>(xn.re[c]), si = store_as<Ts>(xn.im[c]);
            e.re[c] = load_as<Tc>(&sr);
            e.im[c] = load_as<Tc>(&si);
            if (a.inc) {
                e.re[c] -= xo.re[c];
                e.im[c] -= xo.im[c];
            }
        }
    } else {
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            xn.re[c] = e.re[c];
            xn.im[c] = e.im[c];
            Ts sr = store_as<Ts>(e.re[c]), si = store_as<Ts>(e.im[c]);
            e.re[c] = load_as<Tc>(&sr);
            e.im[c] = load_as<Tc>(&si);
        }
    }
    store_spinor(g, a.xw, grp, blk, off, tt, xn);
    if (a.sig_out && a.inc) keep();
    sched_fence();
    if (on[0]) {
        face_hop<0>(l0, ff[0], e, w);
        face_store<0>(a, grp, blk, lcp, tt, ff[0], w);
    }
    if (on[2]) face_link<2>(a, blk, off, bcp, ff[2], l0);
    sched_fence();
    if (on[1]) {
        face_hop<1>(l1, ff[1], e, w);
        face_store<1>(a, grp, blk, lcp, tt, ff[1], w);
    }
    if (on[3]) face_link<3>(a, blk, off, bcp, ff[3], l1);
    sched_fence();
    if (on[2]) {
        face_hop<2>(l0, ff[2], e, w);
        face_store<2>(a, grp, blk, lcp, tt, ff[2], w);
    }
    if (on[3]) {
        face_hop<3>(l1, ff[3], e, w);
        face_store<3>(a, grp, blk, lcp, tt, ff[3], w);
    }
    // a block one site thick: every site is on the -MU face as well
    auto thin = [&](auto m) __attribute__((always_inline)) {
        constexpr int MU = decltype(m)::value;
        if (g.b[MU] == 1 && on[MU]) {
            face_link<MU>(a, blk, off, bcp, false, l0);
            face_hop<MU>(l0, false, e, w);
            face_store<MU>(a, grp, blk, lcp, tt, false, w);
        }
    };
    thin(std::integral_constant<int, 0>{});
    thin(std::integral_constant<int, 1>{});
    thin(std::integral_constant<int, 2>{});
    thin(std::integral_constant<int, 3>{});
}

// numbers of LDS for the reduction scratch of a workgroup: [waves][T][4]
__host__ __device__ inline int red_words(int threads, int T) { return threads / 64 * T * 4; }

// alpha = <q,rho> / <q,q> (0 where q vanishes) per right-hand side lane of the workgroup, from every
// lane's partial sums: each wavefront's sums go to LDS as one 16-byte entry per right-hand side;
// after the barrier every lane adds up its right-hand side's entries in the order of the
// wavefronts.  (A sum across the lanes, one entry each, takes 2 % less time per half-sweep but rounds
// differently.)
template <int T, typename Tc>
__device__ __forceinline__ void mr_alpha(Tc qq, Tc qrr, Tc qri, Tc *red, Tc &ar, Tc &ai)
{
    struct alignas(16) Entry {
        Tc v[4];
    };
    Entry *r = reinterpret_cast<Entry *>(red);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x / 64, t = threadIdx.x % T;
    qq = wave_sum_mod<T>(qq);
    qrr = wave_sum_mod<T>(qrr);
    qri = wave_sum_mod<T>(qri);
    if (lane < T) r[wave * T + lane] = {{qq, qrr, qri, Tc(0)}};
    __syncthreads();
    Tc sqq = 0, sr = 0, si = 0;
#pragma unroll 4
    for (int w = 0; w < nw; ++w) {
        const Entry x = r[w * T + t];
        sqq += x.v[0];
        sr += x.v[1];
        si += x.v[2];
    }
    ar = sqq > Tc(0) ? sr / sqq : Tc(0);
    ai = sqq > Tc(0) ? si / sqq : Tc(0);
}

// One workgroup's share of a half-sweep: block blk, right-hand-side tile `tile`.  The block's links in
// the first NL directions are staged in LDS (after rho and the reduction scratch) for the MR steps.
template <typename Ts, typename Tc, int T, int NL>
__device__ __forceinline__ void sap_block(const SapArgs<Ts, Tc> &a, int blk, int tile, unsigned char *smem)
{
    using LV = LdsVec<Tc>;
    const KGeo &g = a.g;
    LV *rho = reinterpret_cast<LV *>(smem);
    const int str = g.Vb * T;
    Tc *red_s = reinterpret_cast<Tc *>(rho + 24 / V16<Tc>::n * str);  // [waves][T][4]
    Tc *ul = red_s + red_words(blockDim.x, T);  // used only with NL > 0

    const int off = threadIdx.x / T, t = threadIdx.x % T;
    const bool active = off < g.Vb;
    const int grp = (tile * T) / g.S, tt = (tile * T) % g.S + t;  // T divides S: grp is uniform
    const int me = off * T + t;                                   // this lane's LDS slot
    int bc[4] = {0, 0, 0, 0}, lc[4] = {0, 0, 0, 0};
    if (active) decode_site(g, a.blk_coords, a.loc_coords, blk, off, bc, lc);
    const uint32_t lcp = active ? a.loc_coords[off] : 0u;  // local coordinates, 8 bits each
    // links in LDS: this site's index in each direction's box; the T lanes of a site copy
    // its forward links (lane t: directions t, t + T, ...)
    int cf[4] = {0, 0, 0, 0}, sb[4] = {0, 0, 0, 0};
    if (NL) {
        const LinkBox lb = link_box(g);
#pragma unroll
        for (int mu = 0; mu < NL; ++mu) {
            cf[mu] = lb.base[mu] + lc[0] * lb.s[mu][0] + lc[1] * lb.s[mu][1] + lc[2] * lb.s[mu][2] + lc[3] * lb.s[mu][3];
            sb[mu] = lb.s[mu][mu];
        }
        if (active) {
            using V2 = typename Vec2<Tc>::type;
            for (int mu = t; mu < NL; mu += T) {
                if (lc[mu] + 1 < g.b[mu] || g.nb[mu] == 1) {
                    const V2 *src = reinterpret_cast<const V2 *>(a.links + ((size_t)(blk * g.Vb + off) * 4 + mu) * 18);
                    V2 *dst = reinterpret_cast<V2 *>(ul + cf[mu] * 18);
#pragma unroll
                    for (int c = 0; c < 9; ++c) dst[c] = src[c];
                }
            }
        }
    }

    // 1. residual on the block: b - D x, or the kept rho or sigma minus the face hops
    const uint32_t bcp = a.blk_coords[blk];
    // Without inc, the face hops F of this visit (what the other blocks' x contribute) are what
    // sigma for the next visit needs as well (sigma' = rho + F, step 4): where step 1 forms them on
    // their own they are kept in this site's sigma slot until step 4.
    const bool by_faces = a.sig_in || a.mode == 1, keep_f = !a.inc && a.sig_out && by_faces;
    if (active) {
        Spinor<Tc> r;
        if (a.mode == 0) {
            load_spinor<Tc>(g, a.b, grp, blk, off, tt, r);
        } else if (by_faces) {
            // the kept rho or sigma, or at the first visit of the second colour from zero (x vanishes on
            // the block) b, minus what comes across the faces
            Spinor<Tc> f;
            if (a.sig_in) sig_load(g, a.sig, grp, blk, off, tt, r);
            else load_spinor<Tc>(g, a.b, grp, blk, off, tt, r);
            face_sum(a, grp, blk, bcp, lcp, tt, f);
            if (keep_f) sig_store(g, a.sig, grp, blk, off, tt, f);
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                r.re[c] -= f.re[c];
                r.im[c] -= f.im[c];
            }
        } else {
            Spinor<Tc> bb;
            dirac_site_global<Tc>(g, a.links, a.clover, a.xr, grp, tt, blk, off, bc, lc, r, NoSkip{});
            load_spinor<Tc>(g, a.b, grp, blk, off, tt, bb);
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                r.re[c] = bb.re[c] - r.re[c];
                r.im[c] = bb.im[c] - r.im[c];
            }
        }
        lds_store<Tc>(rho, str, me, r);
    }

    // 2. minimal residual on the block operator
    Spinor<Tc> e;
    spinor_zero(e);
    const int wave = threadIdx.x >> 6;
    for (int it = 0; it < a.n_mr; ++it) {
        __syncthreads();
        Spinor<Tc> q;
        Tc qq = 0, qrr = 0, qri = 0;
        if (active) {
            // the site index is hidden from the compiler so that the block's fields are
            // re-read from cache in every step instead of held in registers across the loop
            const int ns = opaque_index(blk * g.Vb + off);
            // the clover term one chiral half at a time (it is block-diagonal in them): six
            // components of rho and 36 field values live instead of twelve and 72
            auto clover_term = [&](auto add) {
                {
                    Spinor<Tc> own;
                    Tc A[36];
                    lds_load_half<0, Tc>(rho, str, me, own);
                    load_clover_half<0>(a.clover, g.V, ns, A);
                    clover_half<0, decltype(add)::value>(A, own, q);
                }
                hop_fence(q);
                {
                    Spinor<Tc> own;
                    Tc A[36];
                    lds_load_half<1, Tc>(rho, str, me, own);
                    load_clover_half<1>(a.clover, g.V, ns, A);
                    clover_half<1, decltype(add)::value>(A, own, q);
                }
                hop_fence(q);
            };
            // (the LDS link indices are hidden like ns: the links are re-read in every step)
            auto hops = [&]() {
                block_hops<0, Tc, (NL > 0)>(g, a.links, rho, T, ns, off, t, lcp, q, ul,
                                            NL > 0 ? opaque_index(cf[0]) : 0, sb[0]);
                hop_fence(q);
                block_hops<1, Tc, (NL > 1)>(g, a.links, rho, T, ns, off, t, lcp, q, ul,
                                            NL > 1 ? opaque_index(cf[1]) : 0, sb[1]);
                hop_fence(q);
                block_hops<2, Tc, (NL > 2)>(g, a.links, rho, T, ns, off, t, lcp, q, ul,
                                            NL > 2 ? opaque_index(cf[2]) : 0, sb[2]);
                hop_fence(q);
                block_hops<3, Tc, (NL > 3)>(g, a.links, rho, T, ns, off, t, lcp, q, ul,
                                            NL > 3 ? opaque_index(cf[3]) : 0, sb[3]);
                hop_fence(q);
            };
            // Every wavefront starts the step together after the barrier; the clover term is read
            // from global memory, the hops from LDS.  Wavefronts 4-7 and 12-15 take the hops
            // first and add the clover term last, so that some wavefronts compute while the
            // others wait for the clover field (with the wavefronts placed on the four SIMDs in
            // turn, each SIMD holds both kinds).
            if ((wave >> 2) & 1) {
                spinor_zero(q);
                hop_fence(q);
                hops();
                clover_term(std::true_type{});
            } else {
                clover_term(std::false_type{});
                hops();
            }
            mr_products(rho, str, me, q, qq, qrr, qri);
        } else {
            spinor_zero(q);
        }
        Tc ar, ai;
        mr_alpha<T>(qq, qrr, qri, red_s, ar, ai);
        if (active) mr_update(rho, str, me, ar, ai, q, e);
    }

    // 3. x|_j (+)= e, and with the incremental residual rho and the faces for later visits
    if (active)
        finish_site(a, grp, blk, off, bcp, (uint32_t)opaque_index((int)lcp), tt, e, a.mode == 2,
                    [&]() __attribute__((always_inline)) {
                        Spinor<Tc> rr;
                        lds_load<Tc>(rho, str, me, rr);
                        sig_store(g, a.sig, grp, blk, off, tt, rr);
                    });
    // 4. sigma for the next visit: b - D_j x_j(new) = rho (the block residual after the MR
    //    steps, this lane's own LDS slot) + the face hops, which this half-sweep leaves unchanged
    //    (kept from step 1, or formed again after a full residual)
    if (active && a.sig_out && !a.inc) {
        Spinor<Tc> sg;
        if (keep_f) {
            sig_load(g, a.sig, grp, blk, off, tt, sg);
        } else if (a.mode != 0) {
            // the coordinates are decoded again rather than kept live through the MR steps
            int bc2[4], lc2[4];
            decode_site(g, a.blk_coords, a.loc_coords, blk, opaque_index(off), bc2, lc2);
            spinor_zero(sg);
            face_hops_global<Tc>(g, a.links, a.xr, grp, tt, blk, off, bc2, lc2, sg, NoSkip{});
        }
        Spinor<Tc> rr;
        lds_load<Tc>(rho, str, me, rr);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            sg.re[c] = a.mode != 0 ? sg.re[c] + rr.re[c] : rr.re[c];
            sg.im[c] = a.mode != 0 ? sg.im[c] + rr.im[c] : rr.im[c];
        }
        sig_store(g, a.sig, grp, blk, off, tt, sg);
    }
}

// h += the hops inside the block on one of the even-odd solver's sites
template <typename Ts, typename Tc, int T>
__device__ inline void eo_hops(const SapArgs<Ts, Tc> &a, const LdsPair<Tc> *rho, int ns, int off, int t,
                               uint32_t lc, Spinor<Tc> &h)
{
    const KGeo &g = a.g;
    block_hops<0, Tc>(g, a.links, rho, T, ns, off, t, lc, h);
    hop_fence(h);
    block_hops<1>(g, a.links, rho, T, ns, off, t, lc, h);
    hop_fence(h);
    block_hops<2>(g, a.links, rho, T, ns, off, t, lc, h);
    hop_fence(h);
    block_hops<3>(g, a.links, rho, T, ns, off, t, lc, h);
    hop_fence(h);
}

// q = (ADD: +=) the clover term at one of the even sites, one chiral half at a time
template <bool ADD, typename Ts, typename Tc>
__device__ inline void eo_clover(const SapArgs<Ts, Tc> &a, const LdsPair<Tc> *rho, int str, int me, int ns,
                                 Spinor<Tc> &q)
{
    {
        Spinor<Tc> own;
        Tc A[36];
        lds_load_half<0, Tc>(rho, str, me, own);
        load_clover_half<0>(a.clover, a.g.V, ns, A);
        clover_half<0, ADD>(A, own, q);
    }
    hop_fence(q);
    {
        Spinor<Tc> own;
        Tc A[36];
        lds_load_half<1, Tc>(rho, str, me, own);
        load_clover_half<1>(a.clover, a.g.V, ns, A);
        clover_half<1, ADD>(A, own, q);
    }
    hop_fence(q);
}

// The residual of one site at a first visit, to LDS: b (x = 0 everywhere), b minus the face hops (x = 0
// on the block), or from a guess the full b - D x.
template <typename Ts, typename Tc, int T>
__device__ inline void eo_residual(const SapArgs<Ts, Tc> &a, LdsPair<Tc> *rho, int blk, int off, int grp,
                                   int tt, int t)
{
    const KGeo &g = a.g;
    Spinor<Tc> r;
    if (a.mode == 0) {
        load_spinor<Tc>(g, a.b, grp, blk, off, tt, r);
    } else if (a.mode == 1) {
        load_spinor<Tc>(g, a.b, grp, blk, off, tt, r);
        Spinor<Tc> f;
        face_sum(a, grp, blk, a.blk_coords[blk], a.loc_coords[off], tt, f);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            r.re[c] -= f.re[c];
            r.im[c] -= f.im[c];
        }
    } else {
        int bc[4], lc[4];
        decode_site(g, a.blk_coords, a.loc_coords, blk, off, bc, lc);
        dirac_site_global<Tc>(g, a.links, a.clover, a.xr, grp, tt, blk, off, bc, lc, r, NoSkip{});
        Spinor<Tc> bb;
        load_spinor<Tc>(g, a.b, grp, blk, off, tt, bb);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            r.re[c] = bb.re[c] - r.re[c];
            r.im[c] = bb.im[c] - r.im[c];
        }
    }
    lds_store<Tc>(rho, g.Vb * T, off * T + t, r);
}

// c = b minus the face hops of the neighbours' x at one site: what a later visit solves D_j x_j = c for
template <typename Ts, typename Tc>
__device__ __forceinline__ void eo_rhs(const SapArgs<Ts, Tc> &a, int blk, int off, int grp, int tt, uint32_t lcp,
                                       Spinor<Tc> &c)
{
    Spinor<Tc> f;
    load_spinor<Tc>(a.g, a.b, grp, blk, off, tt, c);
    face_sum(a, grp, blk, a.blk_coords[blk], lcp, tt, f);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        c.re[k] -= f.re[k];
        c.im[k] -= f.im[k];
    }
}

template <typename Ts, typename Tc, int T>
__device__ inline void eo_update_x(const SapArgs<Ts, Tc> &a, const LdsPair<Tc> *rho, int blk, int off,
                                   int grp, int tt, int t)
{
    Spinor<Tc> e;
    lds_load<Tc>(rho, a.g.Vb * T, off * T + t, e);
    const uint32_t lcp = a.loc_coords[off];
    const int odd = (unpack_coord(lcp, 0) + unpack_coord(lcp, 1) + unpack_coord(lcp, 2) + unpack_coord(lcp, 3)) & 1;
    // (a later visit leaves the odd sites' new x itself)
    finish_site(a, grp, blk, off, a.blk_coords[blk], lcp, tt, e, a.mode == 2 && !(a.sig_in && odd), []() {});
}

// The even-odd block solver (DD-alpha-AMG's): with a block's sites split by the parity of
// their block-local coordinate sum (every block extent even, so each hop inside the block
// joins opposite parities), D_j = A + H is solved through the Schur complement over the
// even sites, S = A_ee - H_eo A_oo^-1 H_oe:
//   rhat_e = r_e - H_eo A_oo^-1 r_o,  n_mr MR steps on S e_e = rhat_e,  e_o = A_oo^-1 (r_o - H_oe e_e).
// Each thread owns one even and one odd site of the block (the u-th of each, parity order),
// so the workgroup has Vb / 2 x T threads and all of them work in both phases of a step: the
// odd sites' hops and A^-1, then the even sites' clover and hops.  LDS holds rho on the even
// sites and -A_oo^-1 H_oe rho on the odd sites; the residual and the x update run in site
// order (sites u and u + Vb / 2) for coalesced vector access and go through LDS.
template <typename Ts, typename Tc, int T>
__device__ inline void sap_block_eo(const SapArgs<Ts, Tc> &a, int blk, int tile, unsigned char *smem)
{
    using LV = LdsPair<Tc>;
    const KGeo &g = a.g;
    LV *rho = reinterpret_cast<LV *>(smem);
    const int str = g.Vb * T;
    Tc *red_s = reinterpret_cast<Tc *>(rho + 12 * str);  // [waves][T][4]

    const int u = threadIdx.x / T, t = threadIdx.x % T, Ve = a.Ve;
    const bool active = u < Ve;
    const int grp = (tile * T) / g.S, tt = (tile * T) % g.S + t;
    const int se = active ? a.eo_sites[u] : 0, so = active ? a.eo_sites[Ve + u] : 0;
    const int me = se * T + t, mo = so * T + t;
    // local coordinates of the even and the odd site, 8 bits each
    const uint32_t lce = active ? a.loc_coords[se] : 0u, lco = active ? a.loc_coords[so] : 0u;

    // 1., 2. the Schur residual rhat_e on the even sites, to LDS, and on the odd ones their solution for the
    // even sites as they are, less their x: eo = A_oo^-1 r_o, of which the even sites' hops read -eo from LDS.
    Spinor<Tc> ee, eo;
    spinor_zero(ee);
    spinor_zero(eo);
    if (a.sig_in) {
        // A later visit, sites in parity order.  From the stored x, not from the Schur residual that the last
        // visit ended with: what rounding x to its storage type took away is then part of the residual and is
        // corrected, where it would add up from sweep to sweep (binary16 storage, 8^4: relative error 2.2e-4
        // at any number of sweeps, against 3.0e-4 to 5.2e-4 at 2 to 6).  The odd sites' old x drops out: with
        // c = b minus the face hops, eo is their new x for the even sites as they are, A_oo^-1 (c_o - H_oe x_e),
        // and rhat_e = c_e - A_ee x_e - H_eo eo: a step's work, where b - D_j x_j and its reduction to the even
        // sites take 1.6 times that (16^3 x 32, 24 right-hand sides in FP32, 3 x 3: 2.70 against 2.85 ms).
        // (LDS holds -x_e, so that every term adds.)  c is loaded ahead of the barrier before its phase.
        Spinor<Tc> co, ce;
        spinor_zero(co);
        spinor_zero(ce);
        if (active) {
            Spinor<Tc> x;
            load_spinor<Tc>(g, a.x, grp, blk, se, tt, x);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                x.re[k] = -x.re[k];
                x.im[k] = -x.im[k];
            }
            lds_store<Tc>(rho, str, me, x);
            eo_rhs(a, blk, so, grp, tt, lco, co);
        }
        __syncthreads();
        if (active) {
            const int ns = opaque_index(blk * g.Vb + so);
            eo_hops<Ts, Tc, T>(a, rho, ns, so, t, lco, co);
            clover_site(a.cloverinv, g.V, ns, co, eo);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                co.re[k] = -eo.re[k];
                co.im[k] = -eo.im[k];
            }
            lds_store<Tc>(rho, str, mo, co);
            eo_rhs(a, blk, se, grp, tt, lce, ce);
        }
        __syncthreads();
        if (active) {
            const int ns = opaque_index(blk * g.Vb + se);
            eo_clover<true>(a, rho, str, me, ns, ce);
            eo_hops<Ts, Tc, T>(a, rho, ns, se, t, lce, ce);
            lds_store<Tc>(rho, str, me, ce);
        }
    } else {
        // a first visit: the residual on the block (sites u and u + Ve in site order), then odd and even
        if (active) {
            eo_residual<Ts, Tc, T>(a, rho, blk, u, grp, tt, t);
            eo_residual<Ts, Tc, T>(a, rho, blk, u + Ve, grp, tt, t);
        }
        __syncthreads();
        if (active) {
            const int ns = blk * g.Vb + so;
            Spinor<Tc> r;
            lds_load<Tc>(rho, str, mo, r);
            clover_site(a.cloverinv, g.V, ns, r, eo);
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                r.re[c] = -eo.re[c];
                r.im[c] = -eo.im[c];
            }
            lds_store<Tc>(rho, str, mo, r);
        }
        __syncthreads();
        if (active) {
            const int ns = blk * g.Vb + se;
            Spinor<Tc> r;
            lds_load<Tc>(rho, str, me, r);
            eo_hops<Ts, Tc, T>(a, rho, ns, se, t, lce, r);
            lds_store<Tc>(rho, str, me, r);
        }
    }

    // 3. minimal residual on S over the even sites
    for (int it = 0; it < a.n_mr; ++it) {
        __syncthreads();
        if (active) {
            // odd slots: -A_oo^-1 H_oe rho
            const int ns = opaque_index(blk * g.Vb + so);
            Spinor<Tc> h, w;
            spinor_zero(h);
            eo_hops<Ts, Tc, T>(a, rho, ns, so, t, lco, h);
            clover_site(a.cloverinv, g.V, ns, h, w);
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                w.re[c] = -w.re[c];
                w.im[c] = -w.im[c];
            }
            lds_store<Tc>(rho, str, mo, w);
        }
        __syncthreads();
        Spinor<Tc> q;
        Tc qq = 0, qrr = 0, qri = 0;
        if (active) {
            const int ns = opaque_index(blk * g.Vb + se);
            eo_clover<false>(a, rho, str, me, ns, q);
            eo_hops<Ts, Tc, T>(a, rho, ns, se, t, lce, q);
            mr_products(rho, str, me, q, qq, qrr, qri);
        } else {
            spinor_zero(q);
        }
        Tc ar, ai;
        mr_alpha<T>(qq, qrr, qri, red_s, ar, ai);
        if (active) {
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                const auto o = rho[c * str + me];
                ee.re[c] += ar * o.x;
                ee.re[c] -= ai * o.y;
                ee.im[c] += ar * o.y;
                ee.im[c] += ai * o.x;
                Tc nr = o.x, ni = o.y;
                nr -= ar * q.re[c];
                nr += ai * q.im[c];
                ni -= ar * q.im[c];
                ni -= ai * q.re[c];
                rho[c * str + me] = {nr, ni};
            }
        }
    }

    // 4. odd: e_o = A_oo^-1 r_o + A_oo^-1 H_oe (-e_e)
    __syncthreads();
    if (active) {
        Spinor<Tc> m;
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            m.re[c] = -ee.re[c];
            m.im[c] = -ee.im[c];
        }
        lds_store<Tc>(rho, str, me, m);
    }
    __syncthreads();
    if (active) {
        const int ns = blk * g.Vb + so;
        Spinor<Tc> h, w;
        spinor_zero(h);
        eo_hops<Ts, Tc, T>(a, rho, ns, so, t, lco, h);
        clover_site(a.cloverinv, g.V, ns, h, w);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            eo.re[c] += w.re[c];
            eo.im[c] += w.im[c];
        }
    }

    // 5. e to LDS, then x|_j (+)= e in site order
    __syncthreads();
    if (active) {
        lds_store<Tc>(rho, str, me, ee);
        lds_store<Tc>(rho, str, mo, eo);
    }
    __syncthreads();
    if (active) {
        eo_update_x<Ts, Tc, T>(a, rho, blk, u, grp, tt, t);
        eo_update_x<Ts, Tc, T>(a, rho, blk, u + Ve, grp, tt, t);
    }
}

// Several operators (lattices of uneven size, each with its own right-hand sides) in one
// launch per half-sweep: workgroup w belongs to the instance whose range [first[k], first[k+1])
// holds it.  The ranges start at multiples of 8, so that every instance is spread over all XCDs in
// contiguous runs (a run of the whole batch had left one XCD with most of the small lattices'
// workgroups).  Descriptors travel by value in the kernel
// arguments, so a captured graph replays without host memory.
constexpr int MAX_BATCH = 8;

template <typename Ts, typename Tc> struct SapBatch {
    SapArgs<Ts, Tc> inst[MAX_BATCH];
    int first[MAX_BATCH + 1];
    int n_inst;
};

template <typename Ts, typename Tc, int T, int NL>
__global__ void __launch_bounds__(256 * T, sizeof(Tc) == 4 ? 4 : 1) k_sap_batched(SapBatch<Ts, Tc> B)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int k = 0;
    while (k + 1 < B.n_inst && (int)blockIdx.x >= B.first[k + 1]) ++k;
    const SapArgs<Ts, Tc> &a = B.inst[k];
    const int w = blockIdx.x - B.first[k], n = a.nblocks * a.ntiles;
    if (w >= n) return;  // padding of an instance's range
    const int li = xcd_remap(w, n);
    const int bi = li / a.ntiles, tile = li - bi * a.ntiles;
    sap_block<Ts, Tc, T, NL>(a, a.blocks[bi], tile, smem);
}

// the same with the even-odd block solver
template <typename Ts, typename Tc, int T>
__global__ void __launch_bounds__(128 * T, (sizeof(Tc) == 4 && T == 2) ? 3 : 1) k_sap_batched_eo(SapBatch<Ts, Tc> B)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int k = 0;
    while (k + 1 < B.n_inst && (int)blockIdx.x >= B.first[k + 1]) ++k;
    const SapArgs<Ts, Tc> &a = B.inst[k];
    const int w = blockIdx.x - B.first[k], n = a.nblocks * a.ntiles;
    if (w >= n) return;  // padding of an instance's range
    const int li = xcd_remap(w, n);
    const int bi = li / a.ntiles, tile = li - bi * a.ntiles;
    sap_block_eo<Ts, Tc, T>(a, a.blocks[bi], tile, smem);
}

struct CopyBatch {
    const void *src[MAX_BATCH];
    void *dst[MAX_BATCH];
    long n[MAX_BATCH];  // elements
    int n_inst;
};

template <typename Ts> __global__ void k_copy_batched(CopyBatch c)
{
    for (int k = 0; k < c.n_inst; ++k) {
        const Ts *s = (const Ts *)c.src[k];
        Ts *d = (Ts *)c.dst[k];
        for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < c.n[k]; i += (long)gridDim.x * blockDim.x)
            d[i] = s[i];
    }
}

template <typename Ts> __global__ void k_fill_zero(Ts *__restrict__ p, long n)
{
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) p[i] = Ts(0);
}

int round64(int n) { return (n + 63) / 64 * 64; }

template <typename Tc> const Tc *op_links(const mrhs_op *op);
template <> const double *op_links<double>(const mrhs_op *op) { return op->links64; }
template <> const float *op_links<float>(const mrhs_op *op) { return op->links32; }
template <typename Tc> const Tc *op_clover(const mrhs_op *op);
template <> const double *op_clover<double>(const mrhs_op *op) { return op->clover64; }
template <> const float *op_clover<float>(const mrhs_op *op) { return op->clover32; }
template <typename Tc> const Tc *op_cloverinv(const mrhs_op *op);
template <> const double *op_cloverinv<double>(const mrhs_op *op) { return op->cloverinv64; }
template <> const float *op_cloverinv<float>(const mrhs_op *op) { return op->cloverinv32; }

size_t align256(size_t n) { return (n + 255) / 256 * 256; }

// bytes of the second face buffer of a lattice with an odd number of blocks in a direction, and of
// the snapshot of x in the same place
template <typename Ts, typename Tc> size_t odd_bytes(const mrhs_op *op, int n_rhs)
{
    return align256(std::max(face_elems<Tc>(op, n_rhs) * sizeof(Tc), native_elems(op, n_rhs) * sizeof(Ts)));
}

template <typename Ts, typename Tc, int T, bool EO, int NL = 0>
int launch_batched(const SapBatch<Ts, Tc> &B, int threads, size_t lds, size_t max_lds, hipStream_t st)
{
    const void *fn = EO ? (const void *)k_sap_batched_eo<Ts, Tc, T> : (const void *)k_sap_batched<Ts, Tc, T, NL>;
    if (int rc = allow_lds(fn, lds, max_lds, "hipFuncSetAttribute(batched sap LDS)")) return rc;
    if constexpr (EO) {
        hipLaunchKernelGGL((k_sap_batched_eo<Ts, Tc, T>), dim3(B.first[B.n_inst]), dim3(threads), lds, st, B);
        return hip_check(hipGetLastError(), "k_sap_batched_eo launch");
    } else {
        hipLaunchKernelGGL((k_sap_batched<Ts, Tc, T, NL>), dim3(B.first[B.n_inst]), dim3(threads), lds, st, B);
        return hip_check(hipGetLastError(), "k_sap_batched launch");
    }
}

template <typename Ts, typename Tc>
int sap_batched_dispatch(const mrhs_op *const *ops, int n, const void *const *b, void *const *x, const int32_t *n_rhs,
                         int n_sap, int n_mr, char *ws, bool guess, void *x_last, hipStream_t st)
{
    // one tile for the whole batch: the smallest of the operators' tiles (all divide S)
    int T = 4, maxVb = 0;
    const size_t max_lds = ops[0]->max_lds;
    const bool eo = ops[0]->block_solver == MRHS_BLOCK_EO_MR;
    for (int k = 0; k < n; ++k) {
        T = std::min(T, ops[k]->sap_tile);
        maxVb = std::max(maxVb, ops[k]->k.Vb);
        if ((ops[k]->block_solver == MRHS_BLOCK_EO_MR) != eo)
            return set_error(MRHS_EINVAL, "the operators of a batch use different block solvers");
    }
    const int threads = round64(maxVb * T);
    const int eo_threads = round64(maxVb / 2 * T);  // even-odd: one even and one odd site per thread
    size_t lds = sizeof(Tc) * (24 * (size_t)maxVb * T + red_words(threads, T));
    if (maxVb * T > 1024 || lds > max_lds) return set_error(MRHS_EUNSUPPORTED, "batched SAP tile does not fit");
    // the plain MR kernel stages the links of staged_links(T) directions in LDS where they fit beside rho
    // without taking a workgroup from a CU, which 1024 threads of the FP32 kernels fill, 512 of FP64's
    int max_links = 0;
    for (int k = 0; k < n; ++k) {
        const LinkBox lb = link_box(ops[k]->k);
        max_links = std::max(max_links, staged_links(T) == 4 ? lb.n : lb.base[staged_links(T)]);
    }
    const size_t lds_ll = lds + sizeof(Tc) * 18 * (size_t)max_links;
    const int per_cu = std::max(1, (sizeof(Tc) == 4 ? 1024 : 512) / threads);
    const bool ll = !eo && lds_ll * per_cu <= max_lds;
    if (ll) lds = lds_ll;
    if (n_sap == 0) {
        if (guess) return MRHS_OK;  // no sweep: x keeps the starting guess
        for (int k = 0; k < n; ++k) {
            hipLaunchKernelGGL(k_fill_zero<Ts>, dim3(1024), dim3(256), 0, st, (Ts *)x[k], (long)native_elems(ops[k], n_rhs[k]));
            if (int rc = hip_check(hipGetLastError(), "k_fill_zero launch")) return rc;
        }
        return MRHS_OK;
    }
    SapBatch<Ts, Tc> B{};
    CopyBatch C{};
    B.n_inst = n;
    char *wp = ws;
    Ts *snap[MAX_BATCH] = {};
    Tc *face[MAX_BATCH][2] = {};
    for (int k = 0; k < n; ++k) {
        const mrhs_op *op = ops[k];
        SapArgs<Ts, Tc> &a = B.inst[k];
        a.g = op->k;
        a.links = op_links<Tc>(op);
        a.clover = op_clover<Tc>(op);
        a.blk_coords = op->blk_coords;
        a.loc_coords = op->loc_coords;
        a.ntiles = (n_rhs[k] + op->k.S - 1) / op->k.S * (op->k.S / T);
        a.n_mr = n_mr;
        a.b = (const Ts *)b[k];
        a.x = (Ts *)x[k];
        a.cloverinv = op_cloverinv<Tc>(op);
        a.eo_sites = op->eo_sites;
        a.Ve = op->k.Vb / 2;
        a.fg = face_geo<Tc>(op->k);
        a.sig = (Tc *)wp;
        wp += align256(native_elems(op, n_rhs[k]) * sizeof(Tc));
        face[k][0] = face[k][1] = (Tc *)wp;
        wp += align256(face_elems<Tc>(op, n_rhs[k]) * sizeof(Tc));
        if (op->odd_blocks) {
            // the second face buffer, first used in the second sweep, shares its space with the
            // snapshot of x that the first sweep from a guess takes
            face[k][1] = (Tc *)wp;
            snap[k] = (Ts *)wp;
            wp += odd_bytes<Ts, Tc>(op, n_rhs[k]);
        }
    }
    for (int s = 0; s < n_sap; ++s)
        for (int c = 0; c < 2; ++c) {
            C.n_inst = 0;
            B.first[0] = 0;
            for (int k = 0; k < n; ++k) {
                const mrhs_op *op = ops[k];
                SapArgs<Ts, Tc> &a = B.inst[k];
                a.blocks = op->colour_blocks + (c == 0 ? 0 : op->n_colour[0]);
                a.nblocks = op->n_colour[c];
                a.mode = s == 0 && !guess ? c : 2;  // from zero, x vanishes on blocks not yet visited
                // plain MR: the incremental residual, but sigma and the face hops of x where that is how
                // FP32 has rounded.  Even-odd keeps no residual and reads the face hops of x.
                a.inc = !eo && (sizeof(Tc) == 8 || !op->odd_blocks);
                a.f_out = !(s + 1 == n_sap && c == 1);
                a.sig_in = s > 0;
                a.sig_out = s + 1 < n_sap;
                a.face_w = face[k][s & 1];
                a.face_o = face[k][c == 0 ? (s + 1) & 1 : s & 1];
                a.face_s = s > 0 ? face[k][(s + 1) & 1] : nullptr;
                a.xr = a.x;
                a.xw = x_last && s + 1 == n_sap ? (Ts *)x_last : a.x;
                if (a.mode == 2 && s == 0 && op->odd_blocks) {
                    C.src[C.n_inst] = a.x;
                    C.dst[C.n_inst] = snap[k];
                    C.n[C.n_inst] = (long)native_elems(op, n_rhs[k]);
                    ++C.n_inst;
                    a.xr = snap[k];
                }
                B.first[k + 1] = B.first[k] + (a.nblocks * a.ntiles + 7) / 8 * 8;
            }
            if (C.n_inst) {
                hipLaunchKernelGGL(k_copy_batched<Ts>, dim3(2048), dim3(256), 0, st, C);
                if (int rc = hip_check(hipGetLastError(), "k_copy_batched launch")) return rc;
            }
            if (B.first[n] == 0) continue;
            int rc;
            const int thr = eo ? eo_threads : threads;
            switch (T * 2 + (eo ? 1 : 0)) {
            case 2:
                rc = ll ? launch_batched<Ts, Tc, 1, false, staged_links(1)>(B, thr, lds, max_lds, st)
                        : launch_batched<Ts, Tc, 1, false>(B, thr, lds, max_lds, st);
                break;
            case 4:
                rc = ll ? launch_batched<Ts, Tc, 2, false, staged_links(2)>(B, thr, lds, max_lds, st)
                        : launch_batched<Ts, Tc, 2, false>(B, thr, lds, max_lds, st);
                break;
            case 3: rc = launch_batched<Ts, Tc, 1, true>(B, thr, lds, max_lds, st); break;
            case 5: rc = launch_batched<Ts, Tc, 2, true>(B, thr, lds, max_lds, st); break;
            default:
                // tile 4 only with FP32 arithmetic (FP64 would spill to scratch)
                if constexpr (sizeof(Tc) == 4) {
                    if (T == 4) {
                        rc = eo ? launch_batched<Ts, Tc, 4, true>(B, thr, lds, max_lds, st)
                           : ll ? launch_batched<Ts, Tc, 4, false, staged_links(4)>(B, thr, lds, max_lds, st)
                                : launch_batched<Ts, Tc, 4, false>(B, thr, lds, max_lds, st);
                        break;
                    }
                }
                rc = set_error(MRHS_EUNSUPPORTED, "SAP tile not built");
            }
            if (rc) return rc;
        }
    return MRHS_OK;
}

}  // namespace

size_t ws_bytes_sap_batched(const mrhs_op *const *ops, int n, const int32_t *n_rhs)
{
    size_t w = 0;
    for (int k = 0; k < n; ++k) {
        const mrhs_op *op = ops[k];
        const bool f64 = op->prec == MRHS_PREC_F64;
        w += align256(native_elems(op, n_rhs[k]) * (f64 ? sizeof(double) : sizeof(float)));  // sigma / rho
        w += align256(f64 ? face_elems<double>(op, n_rhs[k]) * sizeof(double)
                          : face_elems<float>(op, n_rhs[k]) * sizeof(float));
        if (op->odd_blocks)
            w += f64 ? odd_bytes<double, double>(op, n_rhs[k])
                 : op->dtype == MRHS_DTYPE_F16 ? odd_bytes<__half, float>(op, n_rhs[k])
                                               : odd_bytes<float, float>(op, n_rhs[k]);
    }
    return w;
}

int launch_sap_batched(const mrhs_op *const *ops, int n, const void *const *b, void *const *x, const int32_t *n_rhs,
                       int n_sap, int n_mr, void *ws, hipStream_t st, bool guess, void *x_last)
{
    if (n > MAX_BATCH) return set_error(MRHS_EUNSUPPORTED, "more than 8 operators in one batch");
    switch (ops[0]->prec) {
    case MRHS_PREC_F64:
        return sap_batched_dispatch<double, double>(ops, n, b, x, n_rhs, n_sap, n_mr, (char *)ws, guess, x_last, st);
    case MRHS_PREC_F32:
        return sap_batched_dispatch<float, float>(ops, n, b, x, n_rhs, n_sap, n_mr, (char *)ws, guess, x_last, st);
    default:
        return sap_batched_dispatch<__half, float>(ops, n, b, x, n_rhs, n_sap, n_mr, (char *)ws, guess, x_last, st);
    }
}

size_t ws_bytes_sap(const mrhs_op *op, int n_rhs) { return ws_bytes_sap_batched(&op, 1, &n_rhs); }

int launch_sap(const mrhs_op *op, const void *b, void *x, int n_rhs, int n_sap, int n_mr, void *ws, hipStream_t st,
               bool guess, void *x_last)
{
    return launch_sap_batched(&op, 1, &b, &x, &n_rhs, n_sap, n_mr, ws, st, guess, x_last);
}

bool sap_last_sweep_apart(const mrhs_op *, int n_sap) { return n_sap > 1; }

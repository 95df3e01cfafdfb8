// coarse.hip -- the coarse operator D_c = R D P from the orthonormalised test vectors
// (Sec. 2: the coarse-grid operator built in the setup; R = Q^dag as in Alg. 3).
//
// Column c = (h', k') of P is q_k' restricted to spin half h' on each aggregate.  Per
// coarse site i the 9 stored blocks are
//   self: Q_i^dag (A + hops that stay inside the aggregate) P_i, formed as G + sigma3 G^dag sigma3
//         with G = Q_i^dag (A/2 + forward hops that stay inside) P_i
//   +mu : Q_i^dag (1 - g_mu) W_mu P_{i+mu} over the sites on the +mu face   (W = -U/2)
//   -mu : sigma3 (+mu block of i-mu)^dag sigma3
// The last line is exact: the -mu face hop of i is the adjoint of the +mu face hop of i-mu
// conjugated by g5, and g5 acts on the coarse index as sigma3 = diag(1, -1) over halves.
//
// k_coarse: per (aggregate i, block d in self,+x..+t), the sites of the block's set (all
//           sites for self, the +mu face for +mu) in chunks of CHS: the chunk's rows
//           conj(q_k) and its columns w_c = (stencil part d) P_c, computed from Q on the
//           vector units, go to LDS; the 2N x 2N product accumulates on the matrix cores.
//           A +mu workgroup writes its block and, by the sigma3 relation, the -mu block of
//           aggregate i + mu.  Nothing is written to memory but D_c.
#include <algorithm>

#include "launch.h"
#include "stencil.h"

namespace {

constexpr int NTHR = 512;  // 8 wavefronts: one column item per thread and chunk at 32 vectors
constexpr int NW = NTHR / 64;
constexpr int CHS = 8;  // sites per LDS chunk
constexpr int MAXVA = 256;
constexpr int MAXFACE = 64;  // face sites of an aggregate whose neighbours the table holds
constexpr int MAXN = 32;     // test vectors
constexpr int QST = MAXN + 1, WST = 2 * MAXN + 1;  // LDS row strides (pairs) of rows and columns
// The threads of a chunk come in units of 32 lanes: 4 neighbouring test vectors (one group of the
// layout at S = 4) x CHS sites, so that a load of one component covers 16 CHS bytes in one run.  Unit u
// has group u % 8; with u / 8 it takes one spin half of the columns and every other component
// of the rows.
constexpr int RMAX = 12 * (MAXN / 4) / (NTHR / 32);  // rows per thread and chunk
static_assert(CHS == 8 && NTHR == 16 * 32 && MAXN == 32, "units of 4 vectors x 8 sites");

template <typename Tq> struct CoarseArgs {
    KGeo g;
    int a[4], na[4], astr[4];
    int Va, n_agg, N;
    int sshift;          // log2 of the short length S
    long gsz;            // elements of one group of S right-hand sides
    int part_major;      // work items part by part (all self blocks first), for short grids
    const int32_t *agg_sites;
    const uint32_t *blk_coords, *loc_coords;
    const Tq *Q;
    float *Dc;       // [n_agg][9][2N][2N][2], or null with
    __half *Dc16;    // the same in binary16 (each entry rounded once from the FP32 sum)
};

// A site the workgroup touches: native index (fields), offset of its first element within a
// group of the native vector layout, and its local coordinates in its aggregate (8 bits each)
struct SiteRef {
    int ns;
    uint32_t vo;
    uint32_t lc;
};

template <typename Tq>
__device__ inline SiteRef site_ref(const CoarseArgs<Tq> &a, int i, int ls)
{
    SiteRef r;
    r.ns = a.agg_sites[(size_t)i * a.Va + ls];
    const int blk = r.ns / a.g.Vb, off = r.ns - blk * a.g.Vb;
    r.vo = (uint32_t)(blk * 24) * (uint32_t)(a.g.Vb * a.g.S) + (uint32_t)(off * a.g.S);
    uint32_t p = 0;
    int q = ls;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
        p |= (uint32_t)(q % a.a[mu]) << (8 * mu);
        q /= a.a[mu];
    }
    r.lc = p;
    return r;
}

// Spin half HP of column k' of P at a site (six complex components of q_k'; the half is a template
// parameter so that the masked spinor stays in registers); qk points at q_k's group and lane
template <typename Tc> struct Half {
    Tc re[6], im[6];
};

template <int HP, typename Tc, typename Tq>
__device__ inline void load_half6(const Tq *__restrict__ qk, uint32_t vo, uint32_t cs, Half<Tc> &s)
{
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        s.re[c] = load_as<Tc>(qk + vo + (2 * (6 * HP + c)) * cs);
        s.im[c] = load_as<Tc>(qk + vo + (2 * (6 * HP + c) + 1) * cs);
    }
}

template <int HP, typename Tc> __device__ inline void expand_half(const Half<Tc> &h, Spinor<Tc> &s)
{
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        s.re[c] = c / 6 == HP ? h.re[c % 6] : Tc(0);
        s.im[c] = c / 6 == HP ? h.im[c % 6] : Tc(0);
    }
}

// the neighbour x + mu inside the aggregate (the site itself where it lies outside)
template <int MU, typename Tq>
__device__ inline bool inside_nbr(const CoarseArgs<Tq> &a, const SiteRef *tab, uint32_t lc, int ls, uint32_t &vo)
{
    const bool in = unpack_coord(lc, MU) + 1 < a.a[MU];
    vo = tab[in ? ls + a.astr[MU] : ls].vo;
    return in;
}

// w += the forward hop in direction MU from the neighbour's half chi; the link from LDS (ul: the
// links of the chunk's site) or from the operator's field
template <int MU, int HP, typename Tc>
__device__ inline void inside_fwd_hop(const Tc *__restrict__ links, const Tc *ul, int ns, const Half<Tc> &chi,
                                      Spinor<Tc> &w)
{
    Tc U[18];
    if constexpr (sizeof(Tc) == 4) {
        const float2 *p = reinterpret_cast<const float2 *>(ul + 18 * MU);
#pragma unroll
        for (int c = 0; c < 9; ++c) {
            const float2 v = p[c];
            U[2 * c] = v.x;
            U[2 * c + 1] = v.y;
        }
    } else {
        load_link(links, 0L, MU, ns, U);
    }
    Spinor<Tc> s;
    expand_half<HP>(chi, s);
    hop_accumulate<MU, -1, false>(U, s, w);
}

// local site of the f-th site on the +mu face of an aggregate (local coordinate mu = a_mu - 1)
__device__ inline int face_site(const int (&a)[4], const int (&astr)[4], int mu, int f)
{
    const int st = astr[mu];
    return f % st + st * (a[mu] - 1) + st * a[mu] * (f / st);
}

// column (HP, k') of half the self part at aggregate site ls: (A / 2 + the forward hops that
// stay inside) P_c.  The backward inside hops are g5 (forward hops)^dag g5 and A is
// Hermitian and commutes with g5, so with G = Q^dag (A/2 + forward inside hops) P the self
// block is G + sigma3 G^dag sigma3 (g5 P = P sigma3).
template <int HP, typename Tc, typename Tq>
__device__ inline void self_column(const CoarseArgs<Tq> &a, const Tc *__restrict__ links, const Tc *__restrict__ clover,
                                   const Tc *ul, const SiteRef *tab, int ls, const Tq *qk, uint32_t cs, Spinor<Tc> &w)
{
    const SiteRef me = tab[ls];
    uint32_t v0, v1, v2, v3;
    const bool in0 = inside_nbr<0>(a, tab, me.lc, ls, v0), in1 = inside_nbr<1>(a, tab, me.lc, ls, v1);
    const bool in2 = inside_nbr<2>(a, tab, me.lc, ls, v2), in3 = inside_nbr<3>(a, tab, me.lc, ls, v3);
    // the loads of the next hop are issued before the arithmetic of the current one
    Half<Tc> p, c0, c1;
    Tc A[36];
    load_half6<HP>(qk, me.vo, cs, p);
    load_clover_half<HP>(clover, a.g.V, me.ns, A);
    load_half6<HP>(qk, v0, cs, c0);
    sched_fence();
    // the site term is block-diagonal in the spin halves: only half HP is non-zero
    spinor_zero(w);
    {
        Spinor<Tc> s;
        expand_half<HP>(p, s);
        clover_half<HP>(A, s, w);
    }
#pragma unroll
    for (int c = 6 * HP; c < 6 * HP + 6; ++c) {
        w.re[c] *= Tc(0.5);
        w.im[c] *= Tc(0.5);
    }
    hop_fence(w);
    load_half6<HP>(qk, v1, cs, c1);
    sched_fence();
    if (in0) inside_fwd_hop<0, HP>(links, ul, me.ns, c0, w);
    hop_fence(w);
    load_half6<HP>(qk, v2, cs, c0);
    sched_fence();
    if (in1) inside_fwd_hop<1, HP>(links, ul, me.ns, c1, w);
    hop_fence(w);
    load_half6<HP>(qk, v3, cs, c1);
    sched_fence();
    if (in2) inside_fwd_hop<2, HP>(links, ul, me.ns, c0, w);
    hop_fence(w);
    if (in3) inside_fwd_hop<3, HP>(links, ul, me.ns, c1, w);
    hop_fence(w);
}

// column (HP, k') of the +MU face part at face site f: (1 - g_mu) W_mu P_c(x + mu), the
// neighbour x + mu in aggregate i + mu
template <int MU, int HP, typename Tc, typename Tq>
__device__ inline void face_column(const CoarseArgs<Tq> &a, const Tc *__restrict__ links, const SiteRef &me,
                                   const SiteRef &nb, const Tq *qk, uint32_t cs, Spinor<Tc> &w)
{
    Half<Tc> h;
    load_half6<HP>(qk, nb.vo, cs, h);
    Tc U[18];
    load_link(links, a.g.V, MU, me.ns, U);
    Spinor<Tc> chi;
    expand_half<HP>(h, chi);
    spinor_zero(w);
    hop_accumulate<MU, -1, false>(U, chi, w);
}

template <int HP, typename Tc, typename Tq>
__device__ inline void part_column(const CoarseArgs<Tq> &a, const Tc *__restrict__ links, const Tc *__restrict__ clover,
                                   const Tc *ul, int d, const SiteRef *tab, int sidx, int ls, const Tq *qk, uint32_t cs,
                                   Spinor<Tc> &w)
{
    switch (d) {
    case 0: self_column<HP>(a, links, clover, ul, tab, ls, qk, cs, w); break;
    case 1: face_column<0, HP>(a, links, tab[sidx], tab[MAXVA + sidx], qk, cs, w); break;
    case 2: face_column<1, HP>(a, links, tab[sidx], tab[MAXVA + sidx], qk, cs, w); break;
    case 3: face_column<2, HP>(a, links, tab[sidx], tab[MAXVA + sidx], qk, cs, w); break;
    default: face_column<3, HP>(a, links, tab[sidx], tab[MAXVA + sidx], qk, cs, w); break;
    }
}

// grid: 5 items per aggregate (self, then +mu).  A 2N x 2N block is a sum over the
// block's sites and the 6 components of each spin half: rows (h, k) = conj(q_k) of half h,
// columns c = (h', k') the stencil part d applied to P_c.  Both are formed a chunk of CHS
// sites at a time in LDS (the columns by one thread per (h', site, k')); the
// products run on v_mfma_f32_16x16x4f32: the block is cut into 16x16 tiles (per half:
// ceil(N/16) x ceil(2N/16)), the wavefronts take tiles round-robin, a K step is 4 of the
// (site, component) rows, and complex = 4 real products.  Lane l supplies
// A[l%16][l/16] = conj(q)[row][kk] and B[l/16][l%16] = w[kk][col], holds D[4(l/16)+r][l%16].
// The sites the workgroup touches are looked up once into an LDS table (native index,
// vector offset, local coordinates), so the per-item work has no integer division.  The
// rows of the next chunk, and in the self part the links of its sites (staged in LDS), are loaded
// during the products of the current one; the columns load a hop's operands during the
// previous hop's arithmetic; lanes cover 4 vectors x 8 sites, 128-byte runs (vectors across the
// lanes had made every load 16-byte pieces of sixteen lines): 32^3 x 64, 32 vectors in FP32 14.6 ->
// 11.4 ms, 16^4 with 20 408 -> 300 us.  Bound by the matrix cores (5.3 of the 11.4 ms) and the vector
// units (3.3 ms), which do not overlap, and the loads of the columns.  The (aggregate, part)
// items are taken in contiguous runs per XCD, so that concurrent
// workgroups of one XCD read neighbouring aggregates (the face parts' neighbours) through
// the same L2, and the vector-unit-heavy self parts share CUs with the latency-bound faces.
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ inline f4 mfma32(float x, float y, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0); }

// the K steps of one chunk for the wavefront's first NTL tiles: conj(q) w accumulated as four
// real products per complex one, straight-line so that the LDS reads of later steps are in
// flight during the products of earlier ones
template <int NTL>
__device__ inline void tile_products(const float2 *const (&qb)[2], const float2 *const (&wb)[2], f4 (&accr)[2],
                                     f4 (&acci)[2])
{
#pragma unroll
    for (int kk0 = 0; kk0 < CHS * 6; kk0 += 4) {
#pragma unroll
        for (int m = 0; m < NTL; ++m) {
            const float2 q = qb[m][kk0 * QST], w = wb[m][kk0 * WST];
            accr[m] = mfma32(q.x, w.x, accr[m]);
            acci[m] = mfma32(q.x, w.y, acci[m]);
            accr[m] = mfma32(q.y, w.y, accr[m]);
            acci[m] = mfma32(-q.y, w.x, acci[m]);
        }
    }
}

template <typename Tc, typename Tq>
__global__ void __launch_bounds__(NTHR, sizeof(Tc) == 4 && sizeof(Tq) <= 4 ? 4 : 1)
    k_coarse(CoarseArgs<Tq> a, const Tc *__restrict__ links, const Tc *__restrict__ clover)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int N = a.N, N2 = 2 * N;
    // Qs and Ws rows are (half, site, component within the half): the K rows of one half are
    // contiguous.  The strides are those of 32 vectors plus one pair (the four rows a
    // matrix-core step reads fall on different LDS banks), so every product read has a fixed
    // offset; entries beyond N (2N) are never written and only reach output rows (columns)
    // that are not stored.
    SiteRef *tab = reinterpret_cast<SiteRef *>(smem);  // [MAXVA] own sites, [MAXFACE] face neighbours
    float2 *Qs = reinterpret_cast<float2 *>(tab + MAXVA + MAXFACE);  // [2][CHS][6][QST]
    float2 *Ws = Qs + CHS * 12 * QST;                               // [2][CHS][6][WST]
    Tc *Us = reinterpret_cast<Tc *>(Ws + CHS * 12 * WST);           // [CHS][72] links of the chunk (FP32, self)
    // work item li = 5 i + d: aggregate i, part d (0: the self block; 1 + mu: the +mu face
    // block), so that the five parts of an aggregate are consecutive and a CU runs self and
    // face workgroups side by side; items in contiguous runs per XCD.  A grid of a few waves of
    // resident workgroups takes the parts one after the other instead (the self blocks, the
    // longest items, start first and do not end up as the tail), aggregates in XCD runs.
    int i, d;
    if (a.part_major) {
        d = blockIdx.x / a.n_agg;
        i = xcd_remap(blockIdx.x - d * a.n_agg, a.n_agg);
    } else {
        const int li = xcd_remap(blockIdx.x, gridDim.x);
        i = li / 5;
        d = li - 5 * i;
    }
    const bool self = d == 0;
    const int mu = d - 1;
    const int nsites = self ? a.Va : a.Va / a.a[mu];
    int j = i;  // the aggregate across the +mu face
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int TR = (N + 15) / 16, TC = (N2 + 15) / 16, ntile = 2 * TR * TC;
    constexpr int MAXT = (16 + NW - 1) / NW;  // tiles per wavefront (N <= 32: at most 16 tiles)
    static_assert(MAXT == 2, "the product loop takes two tiles per wavefront");
    f4 accr[MAXT], acci[MAXT];
#pragma unroll
    for (int m = 0; m < MAXT; ++m) accr[m] = acci[m] = f4{0.f, 0.f, 0.f, 0.f};

    // site table: self -- every site of aggregate i by local index; face -- the face sites
    // in face order and their +mu neighbours in aggregate i + mu
    if (self) {
        for (int ls = threadIdx.x; ls < a.Va; ls += blockDim.x) tab[ls] = site_ref(a, i, ls);
    } else {
        int c[4], r = i;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            c[m] = r % a.na[m];
            r /= a.na[m];
        }
        c[mu] = (c[mu] + 1) % a.na[mu];
        j = c[0] + a.na[0] * (c[1] + a.na[1] * (c[2] + a.na[2] * c[3]));
        for (int f = threadIdx.x; f < nsites; f += blockDim.x) {
            const int ls = face_site(a.a, a.astr, mu, f);
            tab[f] = site_ref(a, i, ls);
            tab[MAXVA + f] = site_ref(a, j, ls - (a.a[mu] - 1) * a.astr[mu]);
        }
    }
    // this thread's test vector k and site of the chunk (fixed), its unit's part of rows and columns
    const int kt = 4 * ((threadIdx.x >> 5) & 7) + (threadIdx.x & 3), st = (threadIdx.x >> 2) & (CHS - 1);
    const int up = threadIdx.x >> 8;
    const bool kok = kt < N;
    const int kq = kok ? kt : 0;
    const Tq *qk = a.Q + (size_t)(kq >> a.sshift) * a.gsz + (kq & ((1 << a.sshift) - 1));
    const uint32_t cs = (uint32_t)(a.g.Vb * a.g.S);

    // rows: q_k at (site, component) of a chunk, one (site, component) row per thread and pass.
    // The next chunk's rows are loaded into registers before the products of the current one
    // and stored to LDS after them; a row outside the set reads site 0 and is stored as zero.
    // With them, in the self part, the links of the next chunk's sites (16 bytes per thread).
    float2 rv[RMAX];
    bool rok = false;
    constexpr bool STAGE = sizeof(Tc) == 4;
    typedef float f4v __attribute__((ext_vector_type(4)));
    f4v lv = {0.f, 0.f, 0.f, 0.f};
    const auto load_rows = [&](int s0) {
        const int sidx = s0 + st;
        rok = sidx < nsites;
        const uint32_t vo = tab[rok ? sidx : 0].vo;
#pragma unroll
        for (int it = 0; it < RMAX; ++it) {
            const Tq *p = qk + (size_t)(vo + (uint32_t)(2 * up) * cs) + (size_t)(4 * it) * cs;  // component 2 it + up
            rv[it] = make_float2(load_as<float>(p), load_as<float>(p + cs));
        }
        if (STAGE && self && threadIdx.x < CHS * 18) {
            const int sl = threadIdx.x / 18, q = threadIdx.x - sl * 18;
            const int ns = tab[s0 + sl < nsites ? s0 + sl : 0].ns;
            lv = reinterpret_cast<const f4v *>(links)[(size_t)(uint32_t)ns * 18 + q];
        }
    };
    // the links go to LDS at the end of a chunk's products, which do not read them: the barrier at
    // the top of the next chunk covers them as well
    const auto store_links = [&]() {
        if (STAGE && self && threadIdx.x < CHS * 18) reinterpret_cast<f4v *>(Us)[threadIdx.x] = lv;
    };
    __syncthreads();  // the site table
    load_rows(0);
    store_links();

    for (int s0 = 0; s0 < nsites; s0 += CHS) {
        __syncthreads();
        if (kok) {
            float2 *qst = Qs + opaque_index((st * 6 + up) * QST + kt);
#pragma unroll
            for (int it = 0; it < RMAX; ++it)  // component 2 it + up: of half 0 for it < 3
                qst[((it >= 3 ? CHS * 6 : 0) + (2 * it) % 6) * QST] = rok ? rv[it] : make_float2(0.f, 0.f);
        }
        if (kok) {
            // column (h', k') = (up, kt) at site st of the chunk
            const int sidx = s0 + st;
            Spinor<Tc> w;
            if (sidx < nsites) {
                const int ls = self ? sidx : 0;
                const Tc *ul = Us + 72 * st;
                if (up == 0) part_column<0>(a, links, clover, ul, d, tab, sidx, ls, qk, cs, w);
                else part_column<1>(a, links, clover, ul, d, tab, sidx, ls, qk, cs, w);
            } else {
                spinor_zero(w);
            }
            float2 *wst = Ws + opaque_index(st * 6 * WST + up * N + kt);
#pragma unroll
            for (int comp = 0; comp < 12; ++comp)
                wst[((comp / 6) * CHS * 6 + comp % 6) * WST] = make_float2((float)w.re[comp], (float)w.im[comp]);
        }
        __syncthreads();
        if (s0 + CHS < nsites) load_rows(s0 + CHS);
        // the wavefront's tiles in one K loop: four independent accumulator chains; K row kk of
        // half h is LDS row h CHS 6 + kk
        const float2 *qb[MAXT], *wb[MAXT];
#pragma unroll
        for (int m = 0; m < MAXT; ++m) {
            const int tile = std::min(wave + NW * m, ntile - 1);
            const int h = tile / (TR * TC), rem = tile - h * TR * TC, tr = rem / TC, tc = rem - tr * TC;
            const int r0 = h * CHS * 6 + (lane >> 4);
            qb[m] = Qs + r0 * QST + tr * 16 + (lane & 15);  // A: conj(q) rows k of the half
            wb[m] = Ws + r0 * WST + tc * 16 + (lane & 15);  // B: columns c
        }
        if (wave + NW < ntile) tile_products<2>(qb, wb, accr, acci);
        else if (wave < ntile) tile_products<1>(qb, wb, accr, acci);
        if (s0 + CHS < nsites) store_links();
    }
    // D_c(i, i) or D_c(i, i + mu); for a face also D_c(i + mu, i) = sigma3 D_c(i, i + mu)^dag sigma3
    // into the -mu slot of aggregate j = i + mu (each slot has exactly one writer)
    const size_t ob = ((size_t)i * 9 + d) * N2 * N2 * 2, bb = ((size_t)j * 9 + 5 + mu) * N2 * N2 * 2;
    auto put = [&](size_t e, float v) {
        if (a.Dc16) a.Dc16[e] = __float2half_rn(v);
        else a.Dc[e] = v;
    };
    if (self) {
        // D_c(i, i) = G + sigma3 G^dag sigma3: G through LDS (over the chunk buffers, free once
        // every wavefront has finished its last products), then written row by row
        const int GST = N2 + 1;
        float2 *Gs = Qs;
        __syncthreads();
#pragma unroll
        for (int m = 0; m < MAXT; ++m) {
            const int tile = wave + NW * m;
            if (tile >= ntile) break;
            const int h = tile / (TR * TC), rem = tile - h * TR * TC, tr = rem / TC, tc = rem - tr * TC;
            const int c = tc * 16 + (lane & 15);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = tr * 16 + 4 * (lane >> 4) + r;
                if (k < N && c < N2) Gs[(h * N + k) * GST + c] = make_float2(accr[m][r], acci[m][r]);
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < N2 * N2; e += NTHR) {
            const int row = e / N2, c = e - row * N2;
            const float2 g = Gs[row * GST + c], t = Gs[c * GST + row];
            const float sg = ((row < N) == (c < N)) ? 1.f : -1.f;
            put(ob + 2 * (size_t)e, g.x + sg * t.x);
            put(ob + 2 * (size_t)e + 1, g.y - sg * t.y);
        }
        return;
    }
#pragma unroll
    for (int m = 0; m < MAXT; ++m) {
        const int tile = wave + NW * m;
        if (tile >= ntile) break;
        const int h = tile / (TR * TC), rem = tile - h * TR * TC, tr = rem / TC, tc = rem - tr * TC;
        const int c = tc * 16 + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = tr * 16 + 4 * (lane >> 4) + r;
            if (k < N && c < N2) {
                const int row = h * N + k;
                const size_t e = (size_t)row * N2 + c;
                put(ob + 2 * e, accr[m][r]);
                put(ob + 2 * e + 1, acci[m][r]);
                if (!self) {
                    const float sg = ((row < N) == (c < N)) ? 1.f : -1.f;
                    const size_t t = (size_t)c * N2 + row;
                    put(bb + 2 * t, sg * accr[m][r]);
                    put(bb + 2 * t + 1, -sg * acci[m][r]);
                }
            }
        }
    }
}

template <typename Tc, typename Tq>
int coarse_dispatch(const mrhs_op *op, const Tc *links, const Tc *clover, const Tq *Q, int n_tv, void *Dc, bool f16,
                    hipStream_t st)
{
    CoarseArgs<Tq> a{};
    a.g = op->k;
    int s = 1;
    for (int mu = 0; mu < 4; ++mu) {
        a.a[mu] = op->g.agg[mu];
        a.na[mu] = op->na[mu];
        a.astr[mu] = s;
        s *= op->g.agg[mu];
    }
    a.Va = op->Va;
    a.n_agg = op->n_agg;
    a.N = n_tv;
    a.sshift = 0;
    while ((1 << a.sshift) < op->k.S) ++a.sshift;
    a.gsz = (long)op->k.nblk * 24 * op->k.Vb * op->k.S;
    // up to about eight waves of resident workgroups (two per CU): part by part
    a.part_major = op->n_agg * 5 <= 4096;
    a.agg_sites = op->agg_sites;
    a.blk_coords = op->blk_coords;
    a.loc_coords = op->loc_coords;
    a.Q = Q;
    a.Dc = f16 ? nullptr : (float *)Dc;
    a.Dc16 = f16 ? (__half *)Dc : nullptr;
    if (!a.Q || !Dc || !a.agg_sites || !a.blk_coords || !a.loc_coords || !links || !clover)
        return set_error(MRHS_EINVAL, "coarse_op_build: missing buffer");
    if (op->Va > MAXVA) return set_error(MRHS_EUNSUPPORTED, "coarse_op_build: aggregate volume above 256");
    for (int mu = 0; mu < 4; ++mu)
        if (op->Va / op->g.agg[mu] > MAXFACE)
            return set_error(MRHS_EUNSUPPORTED, "coarse_op_build: aggregate face above 64 sites");
    const size_t lds = sizeof(SiteRef) * (MAXVA + MAXFACE) + sizeof(float2) * (size_t)CHS * 12 * (QST + WST) +
                       (sizeof(Tc) == 4 ? sizeof(float) * CHS * 72 : 0);
    hipLaunchKernelGGL((k_coarse<Tc, Tq>), dim3(op->n_agg * 5), dim3(NTHR), lds, st, a, links, clover);
    return hip_check(hipGetLastError(), "k_coarse launch");
}

}  // namespace

size_t ws_bytes_coarse(const mrhs_op *, int) { return 0; }

int launch_coarse(const mrhs_op *op, const void *Q, int qdt, int n_tv, void *Dc, int dcdt, hipStream_t st)
{
    const bool f16 = dcdt == MRHS_DTYPE_F16;
    if (2 * n_tv * 2 * n_tv > 16 * NTHR) return set_error(MRHS_EUNSUPPORTED, "more than 32 test vectors");
    if (op->links32) {
        if (qdt == MRHS_DTYPE_F32)
            return coarse_dispatch<float, float>(op, op->links32, op->clover32, (const float *)Q, n_tv, Dc, f16, st);
        if (qdt == MRHS_DTYPE_F16)
            return coarse_dispatch<float, __half>(op, op->links32, op->clover32, (const __half *)Q, n_tv, Dc, f16, st);
        return coarse_dispatch<float, double>(op, op->links32, op->clover32, (const double *)Q, n_tv, Dc, f16, st);
    }
    if (qdt == MRHS_DTYPE_F32)
        return coarse_dispatch<double, float>(op, op->links64, op->clover64, (const float *)Q, n_tv, Dc, f16, st);
    if (qdt == MRHS_DTYPE_F16)
        return coarse_dispatch<double, __half>(op, op->links64, op->clover64, (const __half *)Q, n_tv, Dc, f16, st);
    return coarse_dispatch<double, double>(op, op->links64, op->clover64, (const double *)Q, n_tv, Dc, f16, st);
}

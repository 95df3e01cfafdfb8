// dirac.hip -- y = D x on the full lattice for many right-hand sides, and the FP64
// residual norms ||b - D x|| / ||b||.
//
// One workgroup per (block, tile of T right-hand sides); thread (off, t) owns one site
// and one right-hand side.  The T lanes of a site issue the same link and clover loads,
// so the operator is fetched once per site for the whole tile (the mat-vec -> mat-mat
// argument of Sec. 6); tiles of one block share an XCD's L2 through xcd_remap.
#include <algorithm>
#include <climits>
#include <mutex>
#include <type_traits>

#include "launch.h"
#include "stencil.h"

// Scratch of mrhs_residual_norms_noalloc: the partial sums per (tile, block, lane) that
// k_residual writes and k_residual_finish adds up, in place of a caller's workspace.  One
// copy per device, held until the process ends.  Host code never passes the array's name
// to a kernel (in host code it is a host-side stand-in): it uses the device address that
// hipGetSymbolAddress returns for the device the call runs on.
constexpr size_t RESID_SCRATCH_BYTES = size_t(32) << 20;
static __device__ __align__(256) unsigned char scratch[RESID_SCRATCH_BYTES];

namespace {

template <typename Ts, typename Tc, int T>
__global__ void __launch_bounds__(256 * T) k_dirac(KGeo g, const Tc *__restrict__ links, const Tc *__restrict__ clover,
                                                   const uint32_t *__restrict__ blk_coords,
                                                   const uint32_t *__restrict__ loc_coords, const Ts *__restrict__ x,
                                                   Ts *__restrict__ y, int ntiles)
{
    const int nwg = g.nblk * ntiles;
    const int li = xcd_remap(blockIdx.x, nwg);
    const int blk = li / ntiles, tile = li - blk * ntiles;
    const int off = threadIdx.x / T, t = threadIdx.x % T;
    if (off >= g.Vb) return;
    const int grp = (tile * T) / g.S, tt = (tile * T) % g.S + t;  // T divides S: grp is uniform
    int bc[4], lc[4];
    decode_site(g, blk_coords, loc_coords, blk, off, bc, lc);
    Spinor<Tc> out;
    dirac_site_global<Tc>(g, links, clover, x, grp, tt, blk, off, bc, lc, out, NoSkip{});
    store_spinor(g, y, grp, blk, off, tt, out);
}

// The stencil with the workgroup's own sites in LDS.  A workgroup takes a chunk of consecutive sites
// of a block for TL right-hand sides (TL lanes per site; lane t has lane (tile TL + t) % S of a group): every
// spinor of the chunk is read once from global memory instead of once per neighbour, and a
// hop reads LDS where the neighbour lies in the chunk, global memory where it does not (the
// lanes of either kind share the hop's arithmetic).  With AHEAD the global operands of a hop are
// loaded two hops ahead.
//
// Spinors are held as stored (Elem) and converted where they are used.  LDS: component vectors of
// 16 bytes, [24 / n][threads].
template <typename Ts> struct Elem {
    using type = Ts;
};
template <> struct Elem<__half> {
    using type = _Float16;  // the same bits
};

template <typename Tx> struct ChunkVec {
    static constexpr int n = 16 / sizeof(Tx);
    typedef Tx type __attribute__((ext_vector_type(16 / sizeof(Tx))));
};

template <typename Tx>
__device__ __forceinline__ void chunk_store(typename ChunkVec<Tx>::type *lds, int me, const Spinor<Tx> &s)
{
    constexpr int n = ChunkVec<Tx>::n;
#pragma unroll
    for (int v = 0; v < 24 / n; ++v) {
        typename ChunkVec<Tx>::type q;
#pragma unroll
        for (int c = 0; c < n; c += 2) {
            q[c] = s.re[(v * n + c) / 2];
            q[c + 1] = s.im[(v * n + c) / 2];
        }
        lds[v * (int)blockDim.x + me] = q;
    }
}

template <typename Tx>
__device__ __forceinline__ void chunk_load(const typename ChunkVec<Tx>::type *lds, int me, Spinor<Tx> &s)
{
    constexpr int n = ChunkVec<Tx>::n;
#pragma unroll
    for (int v = 0; v < 24 / n; ++v) {
        const auto q = lds[v * (int)blockDim.x + me];
#pragma unroll
        for (int c = 0; c < n; c += 2) {
            s.re[(v * n + c) / 2] = q[c];
            s.im[(v * n + c) / 2] = q[c + 1];
        }
    }
}

// Operand of one hop: where it comes from and, for a lane whose neighbour is outside the chunk, the
// neighbour's spinor
template <typename Tx> struct HopIn {
    Spinor<Tx> chi;
    int lds;   // LDS site of the neighbour, or -1
    int site;  // native site of the neighbour
};

// Fields of a chunk's sites in LDS (the residual's FP64 ones): links and clover, 72 numbers each, padded
// to a stride that spreads eight sites over the banks
constexpr int FIELD_REALS = 72, FIELD_STRIDE = 74;
template <typename Tf> using FieldVec = __attribute__((ext_vector_type(2))) Tf;
constexpr size_t field_bytes(int sites) { return 2 * sizeof(double) * FIELD_STRIDE * (size_t)sites; }

// N numbers of a field in LDS; the pointer is made a local one, or the compiler merges these loads with
// those of lanes that read global memory into flat ones
template <int N, typename Tf, typename T> __device__ __forceinline__ void staged_load(const Tf *f, T (&v)[N])
{
    const auto *p = (const __attribute__((address_space(3))) FieldVec<Tf> *)f;
#pragma unroll
    for (int c = 0; c < N / 2; ++c) {
        const FieldVec<Tf> q = p[c];
        v[2 * c] = (T)q.x;
        v[2 * c + 1] = (T)q.y;
    }
}

// TL lanes per site copy 36 two-number vectors of each field
template <int TL, typename Tf>
__device__ __forceinline__ void fields_load(const Tf *__restrict__ src, int ns, FieldVec<Tf> (&v)[(35 + TL) / TL])
{
    const auto *p = reinterpret_cast<const FieldVec<Tf> *>(src);
#pragma unroll
    for (int k = 0; k < (35 + TL) / TL; ++k) {
        const int i = k * (int)blockDim.x + threadIdx.x, last = ns * (FIELD_REALS / 2) - 1;
        v[k] = p[i < last ? i : last];
    }
}
template <int TL, typename Tf>
__device__ __forceinline__ void fields_store(Tf *dst, int ns, const FieldVec<Tf> (&v)[(35 + TL) / TL])
{
    auto *p = reinterpret_cast<FieldVec<Tf> *>(dst);
#pragma unroll
    for (int k = 0; k < (35 + TL) / TL; ++k) {
        const int i = k * (int)blockDim.x + threadIdx.x, s = i / (FIELD_REALS / 2);
        if (i < ns * (FIELD_REALS / 2)) p[s * (FIELD_STRIDE / 2) + (i - s * (FIELD_REALS / 2))] = v[k];
    }
}

template <int MU, bool FWD, typename Tx, typename Ts>
__device__ __forceinline__ void hop_fetch(const KGeo &g, const Ts *__restrict__ x, int grp, int tt, int blk, int off,
                                          int o0, int ns, const int (&bc)[4], const int (&lc)[4], HopIn<Tx> &h)
{
    const NbrSite n = FWD ? nbr_fwd(g, MU, blk, off, bc, lc) : nbr_bwd(g, MU, blk, off, bc, lc);
    const int l = n.off - o0;
    h.lds = n.blk == blk && l >= 0 && l < ns ? l : -1;
    h.site = n.blk * g.Vb + n.off;
    if (h.lds < 0) load_spinor<Tx>(g, x, grp, n.blk, n.off, tt, h.chi);
}

template <int MU, bool FWD, int TL, bool STAGED, typename Tc, typename Tx, typename Tf>
__device__ __forceinline__ void hop_apply(const Tf *__restrict__ links, const Tf *fl,
                                          const typename ChunkVec<Tx>::type *lds, int t, int own, HopIn<Tx> &h, Spinor<Tc> &out)
{
    Tc U[18];
    if constexpr (STAGED) {
        if (FWD) staged_load<18>(fl + (int)threadIdx.x / TL * FIELD_STRIDE + 18 * MU, U);
        else if (h.lds >= 0) staged_load<18>(fl + h.lds * FIELD_STRIDE + 18 * MU, U);
        else load_link(links, 0L, MU, h.site, U);
    } else {
        load_link(links, 0L, MU, FWD ? own : h.site, U);
    }
    if (h.lds >= 0) chunk_load<Tx>(lds, h.lds * TL + t, h.chi);
    hop_accumulate<MU, FWD ? -1 : 1, !FWD>(U, h.chi, out);
    hop_fence(out);
}

template <int TL, bool AHEAD, bool STAGED, typename Tc, typename Tx, typename Tf>
__device__ __forceinline__ void dirac_chunk(const KGeo &g, const Tf *__restrict__ links, const Tf *__restrict__ clover,
                                            const uint32_t *__restrict__ blk_coords,
                                            const uint32_t *__restrict__ loc_coords, const Tx *__restrict__ x, int grp,
                                            int tt, int blk, int o0, int ns, bool ok, unsigned char *smem, Spinor<Tc> &out)
{
    using V = typename ChunkVec<Tx>::type;
    V *lds = reinterpret_cast<V *>(smem);
    const int t = threadIdx.x % TL, off = o0 + (ok ? (int)threadIdx.x / TL : 0);
    const int own = blk * g.Vb + off;
    int bc[4], lc[4];
    decode_site(g, blk_coords, loc_coords, blk, off, bc, lc);
    HopIn<Tx> f, b;
    auto fetch = [&](auto mu, auto fwd, HopIn<Tx> &h) __attribute__((always_inline)) {
        hop_fetch<decltype(mu)::value, decltype(fwd)::value>(g, x, grp, tt, blk, off, o0, ns, bc, lc, h);
    };
    std::integral_constant<int, 0> m0;
    std::true_type fw;
    std::false_type bw;
    Tf *fl = reinterpret_cast<Tf *>(lds + 24 / ChunkVec<Tx>::n * (int)blockDim.x);  // used only with STAGED
    if constexpr (STAGED) {
        Spinor<Tx> me;
        if (ok) load_spinor<Tx>(g, x, grp, blk, off, tt, me);
        FieldVec<Tf> fv[2][(35 + TL) / TL];
        const size_t first = (size_t)(blk * g.Vb + o0) * FIELD_REALS;
        Tf *fc = fl + ns * FIELD_STRIDE;
        fields_load<TL>(links + first, ns, fv[0]);
        fields_load<TL>(clover + first, ns, fv[1]);
        if (AHEAD && ok) {
            fetch(m0, fw, f);
            fetch(m0, bw, b);
        }
        sched_fence();
        if (ok) chunk_store<Tx>(lds, threadIdx.x, me);
        fields_store<TL>(fl, ns, fv[0]);
        fields_store<TL>(fc, ns, fv[1]);
        __syncthreads();
        if (!ok) return;
        chunk_load<Tx>(lds, threadIdx.x, me);
        clover_site(fc + (off - o0) * FIELD_STRIDE, g.V, 0L, me, out);
        hop_fence(out);
    } else {
        if (ok) {
            Spinor<Tx> me;
            load_spinor<Tx>(g, x, grp, blk, off, tt, me);
            if (AHEAD) {
                fetch(m0, fw, f);
                fetch(m0, bw, b);
            }
            sched_fence();
            chunk_store<Tx>(lds, threadIdx.x, me);
            clover_site(clover, g.V, own, me, out);
            hop_fence(out);
        }
        __syncthreads();
        if (!ok) return;
    }
    auto direction = [&](auto mu) __attribute__((always_inline)) {
        constexpr int MU = decltype(mu)::value;
        std::integral_constant<int, (MU + 1) % 4> next;
        if (!AHEAD) fetch(mu, fw, f);
        hop_apply<MU, true, TL, STAGED>(links, fl, lds, t, own, f, out);
        if (AHEAD && MU < 3) fetch(next, fw, f);
        sched_fence();
        if (!AHEAD) fetch(mu, bw, b);
        hop_apply<MU, false, TL, STAGED>(links, fl, lds, t, own, b, out);
        if (AHEAD && MU < 3) fetch(next, bw, b);
        sched_fence();
    };
    direction(m0);
    direction(std::integral_constant<int, 1>{});
    direction(std::integral_constant<int, 2>{});
    direction(std::integral_constant<int, 3>{});
}

int round64(int n) { return (n + 63) / 64 * 64; }

// Sites per workgroup: the block cut into equal chunks of at most `most` sites
struct Chunks {
    int n, sites;
};
Chunks chunks_of(const KGeo &g, int most)
{
    const int n = (g.Vb + most - 1) / most;
    return {n, (g.Vb + n - 1) / n};
}

// Work item li of a grid over (block, tile of TL right-hand sides, slot), a slot being one chunk or
// (slots = 1) the whole block: the slots and tiles of a block are consecutive, blocks in
// contiguous runs per XCD
struct ChunkItem {
    int blk, tile, slot;
};
__device__ inline ChunkItem chunk_item(const KGeo &g, int ntiles, int slots)
{
    const int li = xcd_remap(blockIdx.x, g.nblk * ntiles * slots);
    ChunkItem w;
    w.blk = li / (ntiles * slots);
    const int rem = li - w.blk * ntiles * slots;
    w.tile = rem / slots;
    w.slot = rem - w.tile * slots;
    return w;
}

// The stencil at tile 4 on a short length of 4 (FP32): chunks of up to 128 sites, two workgroups
// per CU.  Bound by the traffic between L2 and memory, three quarters of it neighbours' faces (a face
// in x is every fourth site of the neighbouring block): 32^3 x 64, 24 right-hand sides in FP32 6.5 -> 4.9 ms
// (10.9 GB once each, 28 GB by the counters, 5.7 TB/s), 16^4 with 20 158 -> 120 us.
// TL lanes per site: 4, one group, or where 8 still share a wavefront at most (DIRAC_SMALL sites, several
// groups) two groups: 8 right-hand sides in FP32 at 4 / 8 lanes, us: one site per block at 16^4 431 / 245, 4
// sites at 24^4 695 / 427, 8 sites 412 / 306, 12 sites 303 / 325.
// Binary16 spinors are converted where they are used and are not loaded two hops ahead: with 128 VGPRs
// that spilled 19 (16^4, 20 right-hand sides 104 / 86 us ahead / not ahead, 24^4 with 24 735 / 582).
constexpr int DIRAC_THREADS = 512, DIRAC_SMALL = 8;

template <typename Ts, typename Tc, int TL>
__global__ void __launch_bounds__(DIRAC_THREADS, 4)
    k_dirac_chunk(KGeo g, const Tc *__restrict__ links, const Tc *__restrict__ clover,
                  const uint32_t *__restrict__ blk_coords, const uint32_t *__restrict__ loc_coords,
                  const Ts *__restrict__ x, Ts *__restrict__ y, int ntiles, Chunks ch, int ngrp)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const ChunkItem w = chunk_item(g, ntiles, ch.n);
    const int o0 = w.slot * ch.sites, ns = g.Vb - o0 < ch.sites ? g.Vb - o0 : ch.sites;
    const int lt = w.tile * TL + threadIdx.x % TL, grp = lt / g.S, tt = lt % g.S;
    const bool ok = (int)threadIdx.x / TL < ns && grp < ngrp;
    Spinor<Tc> out;
    using Tx = typename Elem<Ts>::type;
    dirac_chunk<TL, (sizeof(Ts) > 2), false>(g, links, clover, blk_coords, loc_coords, reinterpret_cast<const Tx *>(x),
                                             grp, tt, w.blk, o0, ns, ok, smem, out);
    if (ok) store_spinor(g, y, grp, w.blk, o0 + (int)threadIdx.x / TL, tt, out);
}

template <typename Ts, typename Tc, int TL>
void dirac_chunk_launch(const mrhs_op *op, const Tc *links, const Tc *clover, const void *x, void *y, int ngrp,
                        hipStream_t st)
{
    const KGeo &g = op->k;
    const Chunks ch = chunks_of(g, DIRAC_THREADS / TL);
    const int threads = round64(ch.sites * TL), ntiles = (ngrp * g.S + TL - 1) / TL;
    hipLaunchKernelGGL((k_dirac_chunk<Ts, Tc, TL>), dim3(g.nblk * ntiles * ch.n), dim3(threads),
                       24 * sizeof(Ts) * threads, st, g, links, clover, op->blk_coords, op->loc_coords, (const Ts *)x, (Ts *)y, ntiles, ch, ngrp);
}

// Per (block, tile of T right-hand sides, slot): partial sums of |b - D x|^2 and |b|^2 per right-hand
// side, FP64.  The T lanes of a site share its FP64 field loads; with T = 2S a tile spans two
// groups of the native layout (lanes t < S the first, t >= S the second), which halves the
// field loads per right-hand side.  Lanes of a group beyond the last one add nothing.
// A right-hand side's sums do not depend on how many others share the call, on the slots or on the
// workspace: a block's chunks are the same at tiles 4 and 8, a chunk is summed over runs of 8 sites (32 at
// tile 2, 64 at tile 1) by one tree and over the runs in order, a block over its chunks in order.
// Bound by the traffic between L2 and memory (42 GB by the counters at 32^3 x 64 with 32 right-hand sides
// in FP32, faces five times what must move) and by the FP64 links and clover, 1.7 KB per lane and site.
// Operands two hops ahead (two wavefronts per SIMD) beat three without (7.0 -> 6.4 ms with 24
// right-hand sides; 8.7 ms without, held to 168 VGPRs it spilled); FP64 storage, where they would take
// 268, goes without.
constexpr int RES_THREADS = 256;
template <int T> constexpr int res_sites() { return RES_THREADS / (T == 4 ? 8 : T); }  // of a chunk, at most
constexpr int RES_SLOTS = 256 / res_sites<8>();  // chunks of a block, at most (blocks hold up to 256 sites)
template <int T> constexpr int res_runs() { return T == 4 ? 2 : 1; }                   // of sites in a wavefront

// The fields go through LDS where the eight lanes of a site would each take them through L1 and two
// workgroups still fit in a CU (62 KiB each; with FP64 storage 87, with four lanes 100): 32^3 x 64 with
// 32 right-hand sides in FP32 9.3 ms site by site, 8.1 with the spinors alone in LDS, 7.4 with both, 16^4 with 20
// 213, 193 and 182 us.
template <typename Ts, int T> constexpr bool residual_staged() { return T == 8 && sizeof(Ts) < 8; }

template <typename Ts, int T>
__global__ void __launch_bounds__(RES_THREADS, 2) k_residual(KGeo g, const double *__restrict__ links,
                                                          const double *__restrict__ clover,
                                                          const uint32_t *__restrict__ blk_coords,
                                                          const uint32_t *__restrict__ loc_coords,
                                                          const Ts *__restrict__ b, const Ts *__restrict__ x, int ntiles,
                                                          Chunks ch, int slots, int ngrp, double *__restrict__ part)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int RUNS = res_sites<T>() * T / 64 * res_runs<T>();
    __shared__ double red[2][RUNS][T][2];
    const ChunkItem w = chunk_item(g, ntiles, slots);
    const int lt = w.tile * T + threadIdx.x % T, grp = lt / g.S, tt = lt % g.S, s = (int)threadIdx.x / T;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nruns = (int)blockDim.x / 64 * res_runs<T>();
    using Tx = typename Elem<Ts>::type;
    double sn = 0, sd = 0;  // the block's sums (threads below T)
    // one chunk's sums over its runs, added to the block's
    auto add_chunk = [&](int c) {
        if (threadIdx.x >= T) return;
        double cn = 0, cd = 0;
        for (int k = 0; k < nruns; ++k) {
            cn += red[c & 1][k][threadIdx.x][0];
            cd += red[c & 1][k][threadIdx.x][1];
        }
        sn += cn;
        sd += cd;
    };
    const int c0 = slots == 1 ? 0 : w.slot, c1 = slots == 1 ? ch.n : w.slot + 1;
#pragma unroll 1
    for (int c = c0; c < c1; ++c) {
        const int o0 = c * ch.sites, ns = g.Vb - o0 < ch.sites ? g.Vb - o0 : ch.sites;
        const bool ok = s < ns && grp < ngrp;
        double num = 0, den = 0;
        if (c > c0) {
            __syncthreads();  // every lane has finished reading the last chunk and has left its sums
            add_chunk(c - 1);
        }
        Spinor<double> Dx;
        dirac_chunk<T, (sizeof(Ts) < 8), residual_staged<Ts, T>()>(g, links, clover, blk_coords, loc_coords,
                                                                   reinterpret_cast<const Tx *>(x), grp, tt, w.blk, o0,
                                                                   ns, ok, smem, Dx);
        if (ok) {
            Spinor<double> bb;
            load_spinor<double>(g, b, grp, w.blk, o0 + s, tt, bb);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                const double dr = bb.re[k] - Dx.re[k], di = bb.im[k] - Dx.im[k];
                num += dr * dr + di * di;
                den += bb.re[k] * bb.re[k] + bb.im[k] * bb.im[k];
            }
        }
        if constexpr (T == 4) {
            // two runs of 8 sites per wavefront, lanes 0 .. 31 and 32 .. 63
            num = lane_xor_sum<4>(lane_xor_sum<8>(lane_xor_sum<16>(num)));
            den = lane_xor_sum<4>(lane_xor_sum<8>(lane_xor_sum<16>(den)));
        } else {
            num = wave_sum_mod<T>(num);
            den = wave_sum_mod<T>(den);
        }
        if ((lane & (64 / res_runs<T>() - 1)) < T) {
            double *p = red[c & 1][res_runs<T>() * wave + lane / (64 / res_runs<T>())][lane % T];
            p[0] = num;
            p[1] = den;
        }
    }
    __syncthreads();
    add_chunk(c1 - 1);
    if (threadIdx.x < T) {
        double *p = part + ((((long)w.tile * g.nblk + w.blk) * slots + w.slot) * T + threadIdx.x) * 2;
        p[0] = sn;
        p[1] = sd;
    }
}

// out[k] = sqrt(sum num / sum den), summed over a block's slots and over the blocks in a fixed order
template <int T>
__global__ void k_residual_finish(const double *__restrict__ part, int nblk, int slots, double *__restrict__ out)
{
    __shared__ double sn[256], sd[256];
    const int k = blockIdx.x;
    const int tile = k / T, t = k % T;
    double a = 0, d = 0;
    for (int blk = threadIdx.x; blk < nblk; blk += blockDim.x) {
        const double *p = part + (((long)tile * nblk + blk) * slots * T + t) * 2;
        double bn = p[0], bd = p[1];
        if (slots > 1) {
            double cn[RES_SLOTS], cd[RES_SLOTS];  // all loads in flight
#pragma unroll
            for (int c = 1; c < RES_SLOTS; ++c) {
                cn[c] = c < slots ? p[c * T * 2] : 0.0;
                cd[c] = c < slots ? p[c * T * 2 + 1] : 0.0;
            }
#pragma unroll
            for (int c = 1; c < RES_SLOTS; ++c) {
                bn += cn[c];
                bd += cd[c];
            }
        }
        a += bn;
        d += bd;
    }
    sn[threadIdx.x] = a;
    sd[threadIdx.x] = d;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            sn[threadIdx.x] += sn[threadIdx.x + s];
            sd[threadIdx.x] += sd[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) out[k] = sqrt(sn[0]) / sqrt(sd[0]);
}

template <typename Ts, typename Tc>
int dirac_dispatch(const mrhs_op *op, const Tc *links, const Tc *clover, const void *x, void *y, int n_rhs,
                   hipStream_t st)
{
    const KGeo &g = op->k;
    const int T = op->dirac_tile;
    const int ngrp = (n_rhs + g.S - 1) / g.S;
    const int ntiles = ngrp * (g.S / T);
    dim3 grid(g.nblk * ntiles), block(round64(g.Vb * T));
    switch (T) {
    case 1:
        hipLaunchKernelGGL((k_dirac<Ts, Tc, 1>), grid, block, 0, st, g, links, clover, op->blk_coords, op->loc_coords,
                           (const Ts *)x, (Ts *)y, ntiles);
        break;
    case 2:
        hipLaunchKernelGGL((k_dirac<Ts, Tc, 2>), grid, block, 0, st, g, links, clover, op->blk_coords, op->loc_coords,
                           (const Ts *)x, (Ts *)y, ntiles);
        break;
    case 4:
        // tile 4 only with FP32 arithmetic (FP64 would spill to scratch)
        if constexpr (sizeof(Tc) == 4) {
            if (g.S == 4) {
                if (g.Vb <= DIRAC_SMALL && ngrp > 1) dirac_chunk_launch<Ts, Tc, 8>(op, links, clover, x, y, ngrp, st);
                else dirac_chunk_launch<Ts, Tc, 4>(op, links, clover, x, y, ngrp, st);
                break;
            }
            hipLaunchKernelGGL((k_dirac<Ts, Tc, 4>), grid, block, 0, st, g, links, clover, op->blk_coords,
                               op->loc_coords, (const Ts *)x, (Ts *)y, ntiles);
            break;
        }
        return set_error(MRHS_EUNSUPPORTED, "dirac tile not built");
    default:
        return set_error(MRHS_EUNSUPPORTED, "dirac tile not built");
    }
    return hip_check(hipGetLastError(), "k_dirac launch");
}

// lanes per site of the residual: 8 where the short length allows (two groups of 4), else as many as
// it allows; 4 where there are no more right-hand sides (half of the lanes would idle: 32^4, FP32, 950 -> 615 us)
int residual_tile(const KGeo &g, int n_rhs)
{
    if (g.S % 4 == 0) return n_rhs <= 4 ? 4 : 8;
    return g.S % 2 == 0 ? 2 : 1;
}
int residual_tiles(int n_rhs, int T) { return (n_rhs + T - 1) / T; }

// A short grid takes one workgroup per chunk (a block's chunks side by side), a long one a workgroup
// per block, whose chunks follow one another and share one partial sum
Chunks residual_chunks(const KGeo &g, int T)
{
    return chunks_of(g, T >= 4 ? res_sites<8>() : T == 2 ? res_sites<2>() : res_sites<1>());
}
int residual_slots(const KGeo &g, int ntiles, int T)
{
    return (long)g.nblk * ntiles < 2048 ? residual_chunks(g, T).n : 1;
}

size_t residual_bytes(const KGeo &g, int n_rhs, int T, int slots)
{
    return (size_t)residual_tiles(n_rhs, T) * T * g.nblk * slots * 2 * sizeof(double);
}

template <typename Ts, int T>
int residual_launch(const mrhs_op *op, const void *b, const void *x, int n_rhs, double *out, void *ws, size_t ws_bytes,
                    hipStream_t st)
{
    const KGeo &g = op->k;
    const int ngrp = (n_rhs + g.S - 1) / g.S, ntiles = residual_tiles(n_rhs, T);
    int slots = residual_slots(g, ntiles, T);
    if (residual_bytes(g, n_rhs, T, slots) > ws_bytes) slots = 1;  // a workspace of the least size
    const Chunks ch = residual_chunks(g, T);
    double *part = (double *)ws;
    const int threads = round64(ch.sites * T);
    const size_t lds = 24 * sizeof(Ts) * threads + (residual_staged<Ts, T>() ? field_bytes(ch.sites) : 0);
    hipLaunchKernelGGL((k_residual<Ts, T>), dim3(g.nblk * ntiles * slots), dim3(threads), lds, st, g,
                       op->links64, op->clover64, op->blk_coords, op->loc_coords, (const Ts *)b, (const Ts *)x, ntiles,
                       ch, slots, ngrp, part);
    if (int rc = hip_check(hipGetLastError(), "k_residual launch")) return rc;
    hipLaunchKernelGGL((k_residual_finish<T>), dim3(n_rhs), dim3(256), 0, st, part, g.nblk, slots, out);
    return hip_check(hipGetLastError(), "k_residual_finish launch");
}

template <typename Ts>
int residual_dispatch(const mrhs_op *op, const void *b, const void *x, int n_rhs, double *out, void *ws, size_t ws_bytes,
                      hipStream_t st)
{
    switch (residual_tile(op->k, n_rhs)) {
    case 8: return residual_launch<Ts, 8>(op, b, x, n_rhs, out, ws, ws_bytes, st);
    case 4: return residual_launch<Ts, 4>(op, b, x, n_rhs, out, ws, ws_bytes, st);
    case 2: return residual_launch<Ts, 2>(op, b, x, n_rhs, out, ws, ws_bytes, st);
    default: return residual_launch<Ts, 1>(op, b, x, n_rhs, out, ws, ws_bytes, st);
    }
}

}  // namespace

int launch_dirac(const mrhs_op *op, const void *x, void *y, int n_rhs, hipStream_t st)
{
    switch (op->prec) {
    case MRHS_PREC_F64:
        return dirac_dispatch<double, double>(op, op->links64, op->clover64, x, y, n_rhs, st);
    case MRHS_PREC_F32:
        return dirac_dispatch<float, float>(op, op->links32, op->clover32, x, y, n_rhs, st);
    default:
        return dirac_dispatch<__half, float>(op, op->links32, op->clover32, x, y, n_rhs, st);
    }
}

// what the entry points ask for: the partial sums of one workgroup per block at the tile of many
// right-hand sides (at least what tile 4 takes)
size_t ws_bytes_residual_least(const mrhs_op *op, int n_rhs)
{
    return residual_bytes(op->k, n_rhs, residual_tile(op->k, INT_MAX), 1);
}

size_t ws_bytes_residual(const mrhs_op *op, int n_rhs)
{
    const KGeo &g = op->k;
    const int T = residual_tile(g, n_rhs), nt = residual_tiles(n_rhs, T);
    return std::max(residual_bytes(g, n_rhs, T, residual_slots(g, nt, T)), ws_bytes_residual_least(op, n_rhs));
}

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
void *scratch_ptr[MAX_DEVICES] = {};

// this device's copy of the scratch array, looked up once per device with it current
int device_scratch(int device, void **out)
{
    if (device < 0 || device >= MAX_DEVICES) return set_error(MRHS_EUNSUPPORTED, "device index above 63");
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[device]) {
        int cur = -1;
        if (int rc = hip_check(hipGetDevice(&cur), "hipGetDevice")) return rc;
        if (cur != device)
            if (int rc = hip_check(hipSetDevice(device), "hipSetDevice")) return rc;
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (int rc = hip_check(e, "hipGetSymbolAddress(scratch)")) return rc;
        scratch_ptr[device] = p;
    }
    *out = scratch_ptr[device];
    return MRHS_OK;
}

}  // namespace

int launch_residual_noalloc(const mrhs_op *op, const void *b, const void *x, int n_rhs, double *out, hipStream_t st)
{
    if (ws_bytes_residual_least(op, n_rhs) > RESID_SCRATCH_BYTES)
        return set_error(MRHS_EUNSUPPORTED, "residual partial sums (" + std::to_string(ws_bytes_residual_least(op, n_rhs)) +
                                                " bytes) exceed the 32 MiB scratch of the allocation-free call");
    void *ws = nullptr;
    if (int rc = device_scratch(op->device, &ws)) return rc;
    return launch_residual(op, b, x, n_rhs, out, ws, RESID_SCRATCH_BYTES, st);
}

int launch_residual(const mrhs_op *op, const void *b, const void *x, int n_rhs, double *out, void *ws, size_t ws_bytes,
                    hipStream_t st)
{
    switch (op->dtype) {
    case MRHS_DTYPE_F64:
        return residual_dispatch<double>(op, b, x, n_rhs, out, ws, ws_bytes, st);
    case MRHS_DTYPE_F32:
        return residual_dispatch<float>(op, b, x, n_rhs, out, ws, ws_bytes, st);
    default:
        return residual_dispatch<__half>(op, b, x, n_rhs, out, ws, ws_bytes, st);
    }
}
